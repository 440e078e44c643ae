"""Whole-step parity of as_train_step against the float64 reference.

Tolerances are the stated ones: fp32 tier loss 1e-4 / gradients 1e-4
(normalised max error per tensor); bf16 tier 2e-3 / 3e-2."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import random_trajs

pytestmark = pytest.mark.gpu


def test_config1_fp32():
    import gpu_util as G
    sh = synth.CONFIGS[1]
    rep = G.compare_step(sh, 0, synth.workload(1, 0), 1, 512, bf16=False, loss_tol=1e-4, grad_tol=1e-4)
    print("config1 fp32: loss rel %.2e worst grad %.2e" % (rep["loss_rel"], rep["worst_grad"]))


def test_config1_bf16():
    import gpu_util as G
    sh = synth.CONFIGS[1]
    rep = G.compare_step(sh, 0, synth.workload(1, 0), 1, 512, bf16=True, loss_tol=2e-3, grad_tol=3e-2)
    print("config1 bf16: loss rel %.2e worst grad %.2e" % (rep["loss_rel"], rep["worst_grad"]))


@pytest.mark.parametrize("bf16", [False, True])
def test_seven_targets_gqa_recompute_two_rows(bf16):
    """All seven adapters, grouped KV heads, activation recompute, two rows with ragged tails."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=3, n_q_heads=4, n_kv_heads=2, head_dim=64, d_model=128, ffn=200,
                                  lora_targets=synth.DENSE_TARGETS7, lora_rank=8, lora_alpha=16.0, recompute=1)
    trajs = random_trajs(3, 9, sh.vocab, turn_lo=10, turn_hi=40, turns=(2, 5))
    rep = G.compare_step(sh, 1, trajs, 2, 320, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4,
                         grad_tol=3e-2 if bf16 else 1e-4, recompute=1)
    rep2 = G.compare_step(sh, 1, trajs, 2, 320, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4,
                          grad_tol=3e-2 if bf16 else 1e-4, recompute=0)
    rep3 = G.compare_step(sh, 1, trajs, 2, 320, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4,
                          grad_tol=3e-2 if bf16 else 1e-4, recompute=2)
    # recompute re-runs the same kernels on the same inputs: identical bits
    assert rep["loss"] == rep2["loss"] == rep3["loss"] and rep["grads"] == rep2["grads"] == rep3["grads"]


@pytest.mark.parametrize("bf16", [False, True])
def test_long_segments_many_tiles(bf16):
    """Segments of 2048, 1024 and 1017 tokens (32 key tiles, a ragged tail), four layers, all seven adapters:
    the attention kernels' mask-free path, lazy maximum and longest-first order against the reference."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=4, n_q_heads=4, n_kv_heads=2, head_dim=64, d_model=256, ffn=512, vocab=1024,
                                  lora_targets=synth.DENSE_TARGETS7, lora_rank=16, lora_alpha=32.0)
    g = synth.rng(3, 9)

    def traj(n):
        lens = [n // 6] * 5 + [n - 5 * (n // 6)]
        return [(r, g.integers(0, sh.vocab, size=l).astype(np.int32)) for r, l in zip(synth.role_pattern(6), lens)]

    trajs = [traj(2048), traj(1024), traj(1017)]
    rep = G.compare_step(sh, 1, trajs, 2, 2048, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4)
    print("long segments %s: loss rel %.2e worst grad %.2e" % ("bf16" if bf16 else "fp32", rep["loss_rel"], rep["worst_grad"]))


def test_zero_mask_gives_exact_zero_loss_and_gradients():
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1]
    params, lora = synth.weights(sh, 0), synth.lora_weights(sh, 0)
    trajs = [[(1, t) for _, t in tr] for tr in synth.workload(1, 0)]          # every turn a user turn
    res, model, pk, ctx = G.run_step(sh, params, lora, trajs, 1, 512)
    assert res["count"] == 0 and res["loss"] == 0.0 and res["loss_sum"] == 0.0
    for Lg in model.lora_grads:
        for dA, dB in Lg.values():
            assert not dA.any().item() and not dB.any().item()


def test_lora_b_zero_equals_base_and_packed_equals_sum_of_parts():
    import gpu_util as G
    sh = synth.CONFIGS[1]
    params = synth.weights(sh, 0)
    lora0 = synth.lora_weights(sh, 0, zero_b=True)
    trajs = synth.workload(1, 0)
    res0, model0, _, _ = G.run_step(sh, params, lora0, trajs, 1, 512)
    # no adapter on o/k/v, same forward: a different target set must not change the loss when B = 0
    sh_q = sh.replace(lora_targets=("q",))
    lq = [{"q": L["q"]} for L in lora0]
    res1, _, _, _ = G.run_step(sh_q, params, lq, trajs, 1, 512)
    assert res0["loss"] == res1["loss"]
    for Lg in model0.lora_grads:
        for dA, dB in Lg.values():
            assert not dA.any().item() and dB.any().item()
    # packed row = sum over single-trajectory runs (loss_sum and count)
    lora = synth.lora_weights(sh, 0)
    full, _, _, _ = G.run_step(sh, params, lora, trajs, 1, 512)
    tot, cnt = 0.0, 0
    for tr in trajs:
        L = sum(len(t) for _, t in tr)
        r, _, _, _ = G.run_step(sh, params, lora, [tr], 1, L)
        tot, cnt = tot + r["loss_sum"], cnt + r["count"]
    assert cnt == full["count"] and abs(tot - full["loss_sum"]) <= 1e-4 * abs(full["loss_sum"])


def test_same_inputs_same_bits():
    import gpu_util as G
    sh = synth.CONFIGS[1]
    params, lora = synth.weights(sh, 0), synth.lora_weights(sh, 0)
    trajs = synth.workload(1, 0)
    a, ma, _, _ = G.run_step(sh, params, lora, trajs, 1, 512, mode=1)
    b, mb, _, _ = G.run_step(sh, params, lora, trajs, 1, 512, mode=1)
    assert a == b
    for La, Lb in zip(ma.lora_grads, mb.lora_grads):
        for k in La:
            assert torch.equal(La[k][0], Lb[k][0]) and torch.equal(La[k][1], Lb[k][1])


def test_skipping_loss_free_segments_changes_nothing():
    """Pad tails and trajectories without an assistant turn are squeezed out when the caller passes the
    flags as_pack reports; loss and gradients must agree with the run that computes everything."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, lora_targets=synth.DENSE_TARGETS7)
    trajs = random_trajs(5, 7, sh.vocab, turn_lo=10, turn_hi=30, turns=(2, 5))
    trajs[2] = [(1, t) for _, t in trajs[2]]                    # no assistant turn at all
    trajs[4] = [(0, trajs[4][0][1])]                            # a lone system turn
    params, lora = synth.weights(sh, 2), synth.lora_weights(sh, 2)
    a, ma, pk, _ = G.run_step(sh, params, lora, trajs, 3, 256, skip=True)
    b, mb, _, _ = G.run_step(sh, params, lora, trajs, 3, 256, skip=False)
    assert pk["seg_skip"].sum() >= 3 and pk["seg_skip"].sum() < len(pk["seg_skip"])
    ref = oracle.pack(trajs, 256, 3)
    lens = np.diff(ref["cu_seqlens"])
    expect = [int(ref["loss_mask"][ref["cu_seqlens"][s]:ref["cu_seqlens"][s + 1]].sum() == 0) for s in range(len(lens))]
    assert pk["seg_skip"].tolist() == expect
    assert a["count"] == b["count"] and abs(a["loss"] - b["loss"]) <= 1e-6 * abs(b["loss"])
    for La, Lb in zip(ma.lora_grads, mb.lora_grads):
        for k in La:
            for x, y in zip(La[k], Lb[k]):
                d = (x - y).abs().max().item()
                assert d <= 1e-5 * y.abs().max().item()
    rep = G.compare_step(sh, 2, trajs, 3, 256, bf16=False, loss_tol=1e-4, grad_tol=1e-4, skip=True)
    assert rep["worst_grad"] <= 1e-4


def test_per_kernel_timing_brackets_nested_launchers():
    """With per-launch timing on, a bf16 step (MFMA attention calls the transpose launcher inside its
    own bracket) must run, give the same bits, and report every class it used."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_q_heads=2, n_kv_heads=1, head_dim=64, lora_targets=synth.DENSE_TARGETS7)
    params, lora = synth.weights(sh, 0), synth.lora_weights(sh, 0)
    trajs = synth.workload(1, 0)
    a, ma, pk, ctx = G.run_step(sh, params, lora, trajs, 1, 512, mode=1)
    ctx.profile(True)
    ws = torch.empty(ctx.workspace_bytes(1, 512), dtype=torch.uint8, device="cuda")
    out = ctx.train_step(ma, pk["tokens"], pk["cu_seqlens"], pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"], 1, 512, ws,
                         seg_skip=pk["seg_skip"])
    prof = ctx.profile_read()
    ctx.profile(False)
    assert float(out["loss"].item()) == a["loss"]
    for k in ("attn_fwd", "attn_bwd", "norm", "swiglu", "rope", "lora_grad"):
        assert prof[k][0] > 0 and prof[k][1] > 0.0, (k, prof[k])
    # brackets around one class only
    ctx.profile(True, only="norm")
    out = ctx.train_step(ma, pk["tokens"], pk["cu_seqlens"], pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"], 1, 512, ws,
                         seg_skip=pk["seg_skip"])
    one = ctx.profile_read()
    ctx.profile(False)
    assert float(out["loss"].item()) == a["loss"]
    assert one["norm"][0] == prof["norm"][0] and all(v[0] == 0 for k, v in one.items() if k != "norm"), one
    ctx.profile(True)                                        # and every class again
    ctx.train_step(ma, pk["tokens"], pk["cu_seqlens"], pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"], 1, 512, ws, seg_skip=pk["seg_skip"])
    again = ctx.profile_read()
    ctx.profile(False)
    assert {k: v[0] for k, v in again.items()} == {k: v[0] for k, v in prof.items()}


def test_profile_of_adapter_products_and_of_the_one_pass_head():
    """An adapter of rank 16 adds its 16 columns of u and the 64 columns of the second segment to a forward pass; label logits and the rows' end
    are the head's two launches beside its products."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=256, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=256, vocab=8192, lora_rank=16, lora_alpha=16.0, lora_targets=("o",))
    trajs, n = random_trajs(3, 4, sh.vocab, turn_lo=20, turn_hi=30, turns=(2, 4)), 512
    _, model, pk, ctx = G.run_step(sh, synth.weights(sh, 2), synth.lora_weights(sh, 2), trajs, 1, n, mode=B.AS_BF16, skip=False)
    hcu, ws = pk["cu_seqlens"].cpu().numpy(), torch.empty(ctx.workspace_bytes(1, n), dtype=torch.uint8, device="cuda")

    def profile(call):
        ctx.profile(True)
        call()
        prof = ctx.profile_read()
        ctx.profile(False)
        return prof
    on, off = (profile(lambda: ctx.sequence_logps(model, pk["tokens"], pk["cu_seqlens"], hcu, pk["loss_mask"], 1, n, ws, adapters=a)) for a in (True, False))
    assert sum(v[2] for v in on.values()) - sum(v[2] for v in off.values()) == 2.0 * n * (16 * 128 + 64 * 256)
    step = profile(lambda: ctx.train_step(model, pk["tokens"], pk["cu_seqlens"], hcu, pk["loss_mask"], 1, n, ws))
    assert (step["gemm_devrows"][0], step["ce"][0]) == (2, 2)


@pytest.mark.parametrize("row_len", [384, 320])
def test_wide_ffn_step_runs_the_hand_scheduled_gemm(row_len):
    """ffn = 11264 with 3 row tiles makes 132 tiles of 256 x 256: the gate | up projection (one launch over both matrices) and the input gradient of
    the down projection (rank-64 adapter term as second K segment) go through the hand-scheduled kernel inside the
    step.  With rows of 384 the activation buffers hold 768 rows and the kernel covers the ragged last row tile itself
    (from the padded rows); with rows of 320 (640 rows) the ragged rest goes to the eight-wave kernel."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=2, n_q_heads=4, n_kv_heads=2, head_dim=64, d_model=256, ffn=11264, vocab=512,
                                  lora_targets=synth.DENSE_TARGETS7, lora_rank=64, lora_alpha=128.0)
    trajs = random_trajs(11, 8, sh.vocab, turn_lo=12, turn_hi=30, turns=(3, 5))
    pk = oracle.pack(trajs, row_len, 2)
    cu = pk["cu_seqlens"]
    live = sum(int(b - a) for a, b in zip(cu[:-1], cu[1:]) if pk["loss_mask"][a + 1:b].any())      # rows left after the pad tails are squeezed out
    assert live > 512 and live % 256 != 0 and (live + 255) // 256 * 256 == 768
    rep = G.compare_step(sh, 4, trajs, 2, row_len, bf16=True, loss_tol=2e-3, grad_tol=3e-2)
    print("ffn 11264, rows of %d: loss rel %.2e worst grad %.2e" % (row_len, rep["loss_rel"], rep["worst_grad"]))
    # the same step once more with per-launch timing on: the hand-scheduled kernel took launches, and the bits are the same
    params, lora = G.quantise_params(synth.weights(sh, 4), True), G.quantise_lora(synth.lora_weights(sh, 4))
    a, ma, dpk, ctx = G.run_step(sh, params, lora, trajs, 2, row_len, mode=B.AS_BF16)
    ctx.profile(True)
    ws = torch.empty(ctx.workspace_bytes(2, row_len), dtype=torch.uint8, device="cuda")
    out = ctx.train_step(ma, dpk["tokens"], dpk["cu_seqlens"], dpk["cu_seqlens"].cpu().numpy(), dpk["loss_mask"], 2, row_len, ws,
                         seg_skip=dpk["seg_skip"])
    prof = ctx.profile_read()
    ctx.profile(False)
    assert float(out["loss"].item()) == a["loss"] == rep["loss"]
    assert prof["gemm_mfma_rs"][0] >= 4, prof["gemm_mfma_rs"]                 # 2 layers x (gate | up in one launch, dX of down)


@pytest.mark.parametrize("bf16", [False, True])
def test_more_adapter_matrices_than_one_preparation_launch(bf16):
    """4 layers x 7 adapters are 56 matrices, prepared 40 per launch; widths that are no multiple of the 64 x 64 tiles."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=4, n_q_heads=2, n_kv_heads=1, head_dim=32, d_model=72, ffn=136, vocab=128,
                                  lora_targets=synth.DENSE_TARGETS7, lora_rank=5, lora_alpha=10.0)
    trajs = random_trajs(12, 4, sh.vocab, turn_lo=8, turn_hi=20, turns=(2, 4))
    G.compare_step(sh, 8, trajs, 1, 256, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4)


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("d_model,targets", [(66, ("q", "k", "v", "o", "up")), (72, ("q", "k", "v", "o", "up", "down")), (72, ("v",))])
def test_what_precedes_the_first_layer_in_one_launch(d_model, targets, full):
    """40 adapter matrices fill the launch that also makes segments, rotary table and embedding, 48 need a second, 8 and none leave room; rows of the
    embedding that are no whole 16-byte pieces; 257 tokens are one past a block of the segment table.  The step's stated fp32 tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=4, n_q_heads=2, n_kv_heads=1, head_dim=32, d_model=d_model, ffn=136, vocab=128,
                                  lora_targets=targets, lora_rank=4, lora_alpha=8.0)
    g = synth.rng(5, 9)
    trajs = [[(r, g.integers(0, sh.vocab, size=n).astype(np.int32)) for r, n in zip(synth.role_pattern(len(lens)), lens)] for lens in ([60, 70, 30, 1], [40, 56])]
    G.compare_step(sh, 8, trajs, 1, 257, bf16=False, loss_tol=1e-4, grad_tol=1e-4, full=full)


@pytest.mark.parametrize("row_len,ffn,targets,full", [(4352, 192, synth.DENSE_TARGETS7, False), (4300, 256, ("v", "gate"), False),
                                                      (4300, 192, ("down",), False), (4352, 256, (), True)])
def test_input_gradients_from_matrices_as_they_are(row_len, ffn, targets, full):
    """17 row tiles of a 2048-wide model: the input gradients of q | k | v (matrices of 512, 64 and 64 rows) and gate | up (192 or 256
    rows) are products over the matrices as they lie, with all, some or no adapter columns behind them; whole and ragged
    last row tiles.  The step's stated bf16 tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, n_q_heads=8, n_kv_heads=1, head_dim=64, d_model=2048, ffn=ffn, vocab=512,
                                  lora_targets=targets or synth.DENSE_TARGETS7, lora_rank=8, lora_alpha=16.0)
    trajs = synth.trajectories_lognormal(7, 1, row_len, sh.vocab, 400, 0.5, 64, 900, turns=(2, 5), assistant_share=0.3, token_dist="uniform")
    rep = G.compare_step(sh, 9, trajs, 1, row_len, bf16=True, loss_tol=2e-3, grad_tol=3e-2, full=full)
    print("rows of %d: loss rel %.2e worst grad %.2e" % (row_len, rep["loss_rel"], rep["worst_grad"]))


@pytest.mark.parametrize("targets,rank", [(("v",), 16), (("k", "v", "up"), 3), (("q", "v", "gate", "up", "down"), 33), (synth.DENSE_TARGETS7, 64)])
@pytest.mark.parametrize("turns", [(2, 3), (20, 30)])
def test_adapter_gradients_of_a_group_in_one_launch(targets, rank, turns):
    """Groups of one to six products of unequal, ragged widths, one and several splits of the tokens, ranks of one to four column blocks.
    The step's stated bf16 tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=1, n_q_heads=2, n_kv_heads=1, head_dim=64, d_model=136, ffn=712, vocab=128,
                                  lora_targets=targets, lora_rank=rank, lora_alpha=2.0 * rank)
    trajs = random_trajs(13, 3, sh.vocab, turn_lo=8, turn_hi=20, turns=turns)
    G.compare_step(sh, 8, trajs, 2, 640, bf16=True, loss_tol=2e-3, grad_tol=3e-2)


@pytest.mark.parametrize("bf16, rank", [(False, 16), (True, 16), (True, 33), (True, 64)])
@pytest.mark.parametrize("targets, tokens, d, heads, kv, ffn", [
    (("q", "k", "v"), 333, 512, 8, 2, 192),            # contractions of 512, 128, 128 side by side
    (("q", "v", "up"), 130, 128, 2, 1, 64),            # two of the three; one of two
    (("k", "v"), 1100, 1024, 16, 4, 1088),             # without the longest
    (synth.DENSE_TARGETS7, 70, 1024, 16, 2, 2112),     # one row tile, long contractions
    (("q", "k", "v"), 70, 256, 64, 1, 192),            # 4096, 64 and 64, split: parts in which k and v have no step
])
def test_adapter_products_side_by_side(targets, tokens, d, heads, kv, ffn, bf16, rank):
    """du of q, k, v and of gate, up as one launch each: in bf16 past rank 16 as batched GEMMs, up to it from rows."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv, head_dim=64, ffn=ffn, vocab=512, lora_rank=rank, lora_alpha=2.0 * rank,
                                  lora_targets=targets)
    g = synth.rng(6, tokens)
    cuts = [0, tokens // 3, tokens]
    trajs = [[(1, g.integers(0, sh.vocab, size=3).astype(np.int32)), (2, g.integers(0, sh.vocab, size=e - b - 3).astype(np.int32))] for b, e in zip(cuts, cuts[1:])]
    G.compare_step(sh, 2, trajs, 1, tokens, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4)
    if not bf16:
        return
    # beyond a forward pass: the input gradients of down, gate | up and o, and one launch of du for every group with an adapter
    _, model, pk, ctx = G.run_step(sh, synth.weights(sh, 2), synth.lora_weights(sh, 2), trajs, 1, tokens, mode=B.AS_BF16)
    args = (model, pk["tokens"], pk["cu_seqlens"], pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"], 1, tokens,
            torch.empty(ctx.workspace_bytes(1, tokens), dtype=torch.uint8, device="cuda"))
    launches = []
    for call in (ctx.sequence_logps, ctx.train_step):
        ctx.profile(True)
        call(*args)
        launches.append(ctx.profile_read()["gemm_mfma_skinny"][0])
        ctx.profile(False)
    assert launches[1] - launches[0] == 3 + sum(any(t in targets for t in group) for group in (("q", "k", "v"), ("o",), ("gate", "up"), ("down",)))


@pytest.mark.parametrize("tokens, rank", [(4, 16), (31, 1), (32, 16), (33, 15), (97, 16), (97, 17), (2049, 8)])
def test_adapter_gradients_around_their_32_token_steps(tokens, rank):
    """Up to rank 16 the kernel reads u and du as rows, past it as token-major copies; a last step may hold one token."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=192, vocab=256, lora_rank=rank, lora_alpha=2.0 * rank,
                                  lora_targets=synth.DENSE_TARGETS7)
    g = synth.rng(8, tokens)
    trajs = [[(1, g.integers(0, sh.vocab, size=1).astype(np.int32)), (2, g.integers(0, sh.vocab, size=tokens - 1).astype(np.int32))]]
    G.compare_step(sh, 3, trajs, 1, tokens, bf16=True, loss_tol=2e-3, grad_tol=3e-2)


@pytest.mark.parametrize("tokens, d, heads, kv, ffn, targets", [
    (17, 64, 1, 1, 64, synth.DENSE_TARGETS7),              # one 64-wide step of the contraction, a workgroup of one token
    (300, 1088, 17, 1, 2112, synth.DENSE_TARGETS7),        # more steps than waves, contractions of different lengths side by side
    (8200, 128, 2, 1, 192, synth.DENSE_TARGETS7),          # eight waves
    (300, 128, 2, 2, 200, synth.DENSE_TARGETS7),           # an FFN that is no multiple of 64: its adapters as narrow products
    (300, 128, 2, 2, 192, ("q", "v", "up")),               # two of three, one of two
])
def test_adapter_products_from_rows(tokens, d, heads, kv, ffn, targets):
    """u = x A^T and du = dY B of rank up to 16."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, d_model=d, n_q_heads=heads, n_kv_heads=kv, head_dim=64, ffn=ffn, vocab=512, lora_rank=13, lora_alpha=26.0,
                                  lora_targets=targets)
    g = synth.rng(9, tokens)
    cuts = [tokens * i // 8 for i in range(9)]
    trajs = [[(1, g.integers(0, sh.vocab, size=1).astype(np.int32)), (2, g.integers(0, sh.vocab, size=e - b - 1).astype(np.int32))] for b, e in zip(cuts, cuts[1:])]
    G.compare_step(sh, 4, trajs, 1, tokens, bf16=True, loss_tol=2e-3, grad_tol=3e-2)


@pytest.mark.parametrize("dh", [32, 128])
def test_fp32_steps_take_segments_of_so_many_tokens(dh):
    """20,480 - head_dim in backward; the message of a longer one's refusal says so."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=32, n_q_heads=1, n_kv_heads=1, head_dim=dh, ffn=32, vocab=64, lora_rank=2, lora_alpha=4.0, lora_targets=("q",))
    params, lora = synth.weights(sh, 1), synth.lora_weights(sh, 1)
    limit = 20480 - dh
    for n in (limit, limit + 1):
        trajs = [[(1, np.full(2, 5, np.int32)), (2, np.full(n - 2, 6, np.int32))]]
        if n > limit:
            with pytest.raises(B.ASError, match="segments of at most %d tokens" % limit):
                G.run_step(sh, params, lora, trajs, 1, n, mode=B.AS_FP32)
        else:
            res, model, _, _ = G.run_step(sh, params, lora, trajs, 1, n, mode=B.AS_FP32)
            assert res["count"] == n - 2 and np.isfinite(res["loss"]) and all(torch.isfinite(x).all().item() for x in model.lora_grads[0]["q"])


@pytest.mark.parametrize("tokens", [3840, 3841])
def test_attention_backward_head_dim_128_in_one_launch_and_in_two(tokens):
    """128 heads over 32: 3840 tokens are the last of a step that dQ and dK / dV share a launch for (under four rounds of dK / dV workgroups), 3841 the
    first of two launches.  The bf16 tier's tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=64, n_q_heads=128, n_kv_heads=32, head_dim=128, ffn=64, vocab=256, lora_rank=8, lora_alpha=16.0,
                                  lora_targets=("q", "k", "v"))
    g = synth.rng(14, 0)
    cuts = [0, 300, 301, 303, 559, 815] + list(range(900, 3800, 60)) + [tokens]
    trajs = [[(2, g.integers(0, sh.vocab, size=e - b).astype(np.int32))] for b, e in zip(cuts, cuts[1:])]
    G.compare_step(sh, 5, trajs, 1, tokens, bf16=True, loss_tol=2e-3, grad_tol=3e-2, skip=False)
