"""AdamW on the GPU against the float64 reference, and full fine-tuning (all weights trainable)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import random_trajs, grad_norm_err

pytestmark = pytest.mark.gpu


def test_adamw_matches_reference_over_steps():
    from paper_2503_22673_amd import binding as B
    ctx = B.Context(B.make_config(synth.CONFIGS[1]))
    g = synth.rng(0, 30)
    shapes = [(7,), (128, 344), (1000, 33), (1,)]
    w0 = [g.standard_normal(s).astype(np.float32) for s in shapes]
    masters = [torch.from_numpy(w.copy()).cuda() for w in w0]
    lowp = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") if i % 2 == 0 else None for i, s in enumerate(shapes)]
    ms = [torch.zeros_like(w) for w in masters]
    vs = [torch.zeros_like(w) for w in masters]
    wd_flags = [1, 1, 0, 1]
    ref = [(w.astype(np.float64), np.zeros(w.shape), np.zeros(w.shape)) for w in w0]
    lr, b1, b2, eps, wd = 2e-5, 0.9, 0.95, 1e-8, 0.1
    for step in range(1, 5):
        grads = [g.standard_normal(s).astype(np.float32) * (10.0 ** (step - 2)) for s in shapes]
        gd = [torch.from_numpy(x).cuda() for x in grads]
        ctx.adamw_update(masters, lowp, gd, ms, vs, wd_flags, step, lr, b1, b2, eps, wd)
        torch.cuda.synchronize()
        ref = [oracle.adamw_update(w, gr.astype(np.float64), m, v, step, lr, b1, b2, eps, wd if f else 0.0)
               for (w, m, v), gr, f in zip(ref, grads, wd_flags)]
    for i, (w, m, v) in enumerate(ref):
        assert np.max(np.abs(masters[i].cpu().numpy() - w)) <= 2e-6 * max(1.0, np.max(np.abs(w)))
        assert grad_norm_err(ms[i].cpu().numpy(), m) < 1e-5 and grad_norm_err(vs[i].cpu().numpy(), v) < 1e-5
        if lowp[i] is not None:        # round-to-nearest-even copy of the updated master
            assert torch.equal(lowp[i], masters[i].to(torch.bfloat16))


@pytest.mark.parametrize("n,shift", [(4095, 0), (4096, 0), (4097, 0), (3 * 4096, 0), (2 * 4096, 1), (70 * 1024 + 5, 0)])
def test_adamw_whole_and_partial_chunks(n, shift):
    """Chunk edges, and tensors that start off a 16-byte boundary (`shift` elements in), next to a small tensor in the same
    launch.  Reference with the float32 values of the rates: m carries two roundings of its terms' size, v three (at most
    3 x 2^-24 = 1.8e-7), w one of its own size and the update's, which is 2e-5 of it."""
    from paper_2503_22673_amd import binding as B
    ctx = B.Context(B.make_config(synth.CONFIGS[1]))
    gen = torch.Generator(device="cuda"); gen.manual_seed(n)
    new = lambda k, s: torch.empty(k + shift, device="cuda").normal_(0.0, s, generator=gen)[shift:]
    w, g, m, v = [[new(k, s) for k in (n, 9)] for s in (0.02, 1e-3, 1e-4, 1e-3)]
    for x in v:
        x.square_()
    low = [torch.zeros(n + shift, dtype=torch.bfloat16, device="cuda")[shift:], None]
    ref = [[t.double() for t in x] for x in (w, g, m, v)]
    lr, b1, b2, eps, wd = (float(np.float32(x)) for x in (2e-5, 0.9, 0.95, 1e-8, 0.1))
    step = 3
    ctx.adamw_update(w, low, g, m, v, [1, 0], step, lr, b1, b2, eps, wd)
    torch.cuda.synchronize()
    for i, decay in enumerate((wd, 0.0)):
        rw, rg, rm, rv = (x[i] for x in ref)
        size = float((b1 * rm.abs() + (1 - b1) * rg.abs()).max())
        rm, rv = b1 * rm + (1 - b1) * rg, b2 * rv + (1 - b2) * rg * rg
        rw = rw - lr * (rm / (1 - b1 ** step) / ((rv / (1 - b2 ** step)).sqrt() + eps) + decay * rw)
        assert float((m[i] - rm).abs().max()) <= 2e-7 * size and float((v[i] - rv).abs().max()) <= 2e-7 * float(rv.abs().max())
        assert float((w[i] - rw).abs().max()) <= 2e-7 * float(rw.abs().max())
    assert torch.equal(low[0], w[0].to(torch.bfloat16))


def test_adamw_first_step_closed_form_and_identity():
    from paper_2503_22673_amd import binding as B
    ctx = B.Context(B.make_config(synth.CONFIGS[1]))
    w = torch.tensor([1.0, -1.0, 0.5, 2.0], device="cuda")
    gr = torch.tensor([0.3, -2.0, 1e-3, 5.0], device="cuda")
    m, v = torch.zeros_like(w), torch.zeros_like(w)
    w0 = w.clone()
    ctx.adamw_update([w], None, [gr], [m], [v], [1], 1, 1e-2, 0.9, 0.95, 1e-8, 0.1)
    torch.cuda.synchronize()
    expect = w0 - 1e-2 * (gr / (gr.abs() + 1e-8) + 0.1 * w0)
    assert torch.allclose(w, expect, atol=1e-7)
    w2 = w.clone()
    z = torch.zeros_like(w)
    ctx.adamw_update([w], None, [z], [torch.zeros_like(w)], [torch.zeros_like(w)], [0], 1, 1e-2, 0.9, 0.95, 1e-8, 0.1)
    torch.cuda.synchronize()
    assert torch.equal(w, w2)                      # zero gradient, no decay: untouched


@pytest.mark.parametrize("bf16", [False, True])
def test_full_finetuning_step_matches_reference(bf16):
    """Every weight gradient (projections, gains, embedding with repeated tokens, head) of a small
    GQA model, two rows, against the reference."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, n_q_heads=4, n_kv_heads=2, head_dim=64, d_model=128, ffn=200, vocab=300,
                                  lora_rank=0, lora_alpha=0.0, lora_targets=(), full_ft=True)
    trajs = random_trajs(7, 8, sh.vocab, turn_lo=10, turn_hi=40, turns=(2, 5))
    rep = G.compare_step(sh, 3, trajs, 2, 320, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4,
                         full=True)
    print("full FT %s: loss rel %.2e worst grad %.2e" % ("bf16" if bf16 else "fp32", rep["loss_rel"], rep["worst_grad"]))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,d", [(5, 64), (32, 64), (33, 96), (2048, 64), (2049, 64), (4203, 72)])
def test_embedding_gradient_piece_and_tile_edges(n, d, bf16):
    """Token lists around the edges of the sum's pieces (32 positions) and of the sort's tiles (2048), one token holding
    40 % of all positions (its run crosses many pieces), the first and last id of a vocabulary that takes two sort digits,
    a width that is no multiple of a workgroup's columns.  The step's stated tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=1, n_q_heads=2, n_kv_heads=1, head_dim=32, d_model=d, ffn=64, vocab=1300,
                                  lora_rank=0, lora_alpha=0.0, lora_targets=(), full_ft=True)
    g = synth.rng(n, 31)
    ids = np.where(g.random(n) < 0.4, 700, g.integers(0, sh.vocab, size=n)).astype(np.int32)
    ids[0], ids[-1] = 0, sh.vocab - 1
    trajs = [[(1, ids[b:b + 2]), (2, ids[b + 2:b + 500])] for b in range(0, n - 4, 500)]
    if n > 4 and (n - 4) % 500:
        trajs[-1][-1] = (2, ids[(n - 5) // 500 * 500 + 2:])
    row_len = max(512, n)
    rep = G.compare_step(sh, 4, trajs, 1, row_len, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4, full=True)
    assert rep["grads"]["embed"] <= (3e-2 if bf16 else 1e-4)


@pytest.mark.parametrize("d,bf16", [(72, False), (1032, False), (100, True), (2048, True), (2304, True), (4104, True)])
def test_gain_gradients_over_row_widths(d, bf16):
    """Gain gradients that come out of the norm's backward pass (up to 1024 / 2048 float, 2048 / 4096 bf16 columns in registers)
    and those of wider rows and of rows that are no whole vectors (a pass of their own); the final norm's rows are a subset."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=1, n_q_heads=2, n_kv_heads=1, head_dim=32, d_model=d, ffn=64, vocab=96,
                                  lora_rank=0, lora_alpha=0.0, lora_targets=(), full_ft=True)
    trajs = random_trajs(d, 6, sh.vocab, turn_lo=10, turn_hi=30, turns=(2, 4))
    rep = G.compare_step(sh, 3, trajs, 1, 512, bf16=bf16, loss_tol=2e-3 if bf16 else 1e-4, grad_tol=3e-2 if bf16 else 1e-4, full=True)
    assert max(rep["grads"][k] for k in ("g_final", "L0.g1", "L0.g2")) <= (3e-2 if bf16 else 1e-4)


@pytest.mark.parametrize("row_len,Hkv,ffn,share", [(4352, 4, 256, 0.3), (11000, 4, 512, 0.9), (9000, 4, 256, 0.3), (4301, 1, 320, 0.3)])
def test_weight_gradients_from_rows_as_they_are(row_len, Hkv, ffn, share):
    """Contractions over the tokens of a 1024-wide model: q | k | v and gate | up as rows of one product, the head over its live target rows (one
    chunk, two, a second one without targets), token counts that are no multiple of a 64-token step; the last
    case has matrices of 64 and 320 rows, which go through token-major copies.  The step's stated bf16 tolerances."""
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, n_q_heads=8, n_kv_heads=Hkv, head_dim=64, d_model=1024, ffn=ffn, vocab=1024)
    trajs = synth.trajectories_lognormal(3, 1, row_len, sh.vocab, 400, 0.5, 64, 900, turns=(2, 5), assistant_share=share, token_dist="uniform")
    rep = G.compare_step(sh, 5, trajs, 1, row_len, bf16=True, loss_tol=2e-3, grad_tol=3e-2, full=True)
    print("rows of %d: loss rel %.2e worst grad %.2e" % (row_len, rep["loss_rel"], rep["worst_grad"]))


@pytest.mark.parametrize("vocab", [1024, 8448])
@pytest.mark.parametrize("targets", [0, 40])
def test_head_gradient_over_few_or_no_target_rows(vocab, targets):
    """The head's weight gradient contracts over as many target rows as the device counts.  16 tiles: every tile is split into parts,
    all or all but one of them empty; 132 tiles: unsplit.  Without targets every gradient is exactly zero, the head's over what the
    buffer held before; with 40 (one partial step of 64 rows) the step's stated bf16 tolerances hold."""
    import gpu_util as G
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=1, n_q_heads=8, n_kv_heads=4, head_dim=64, d_model=1024, ffn=256, vocab=vocab,
                                  lora_rank=0, lora_alpha=0.0, lora_targets=(), full_ft=True)
    g = synth.rng(vocab + targets, 32)
    ids = g.integers(0, vocab, size=4352).astype(np.int32)
    trajs = [[(1, ids[b:b + 544])] for b in range(0, 4352, 544)]
    if targets:
        trajs[3] = [(1, trajs[3][0][1][:300]), (2, trajs[3][0][1][300:300 + targets]), (1, trajs[3][0][1][300 + targets:])]
        rep = G.compare_step(sh, 5, trajs, 1, 4352, bf16=True, loss_tol=2e-3, grad_tol=3e-2, full=True, skip=False)
        assert rep["grads"]["head"] <= 3e-2
        return
    params = G.quantise_params(synth.weights(sh, 5), True)
    ctx = B.Context(B.make_config(sh, mode=B.AS_BF16, train_mode=B.AS_FULL))
    pk = ctx.pack(*synth.flatten_trajectories(trajs), 4352, 1)
    model = B.DeviceModel(ctx, params)
    grads = [t for k in ("embed", "head", "g_final") for t in [model.w_grads[k]]] + [t for L in model.w_grads["layers"] for t in L.values()]
    for t in grads:
        t.fill_(7.0)
    ws = torch.zeros(ctx.workspace_bytes(1, 4352), dtype=torch.uint8, device="cuda")
    out = ctx.train_step(model, pk["tokens"], pk["cu_seqlens"], pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"], 1, 4352, ws)
    torch.cuda.synchronize()
    assert int(out["count"].item()) == 0 and float(out["loss_sum"].item()) == 0.0
    for t in grads:
        assert int(torch.count_nonzero(t)) == 0
