"""SwiGLU fused with the adapter products of gate, up and down, through the whole step (its only caller): column steps around the number of
waves, tokens around the 16 of a workgroup and the 4096 from which on it is used, ranks up to its 16 and past them, adapters on some of the three
only.  Tolerances: the bf16 tier's (loss 2e-3, gradients 3e-2)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ffn, tokens, rank, targets", [
    (64, 4097, 16, synth.DENSE_TARGETS7),          # one column step; a workgroup of one token
    (192, 4110, 5, synth.DENSE_TARGETS7),          # fewer steps than waves
    (576, 4111, 16, synth.DENSE_TARGETS7),         # a step more than waves
    (1088, 4096, 16, synth.DENSE_TARGETS7),        # seventeen steps: every wave two, one of them three
    (320, 4095, 16, synth.DENSE_TARGETS7),         # a token short: the kernels one after the other
    (320, 4097, 17, synth.DENSE_TARGETS7),         # a higher rank: likewise
    (320, 4097, 16, ("q", "down")),                # forward only
    (320, 4097, 16, ("gate", "up")),               # backward only
    (320, 4097, 16, ("up", "down")),               # gate without an adapter
])
def test_step_against_the_oracle(ffn, tokens, rank, targets):
    import gpu_util as G
    sh = synth.CONFIGS[1].replace(n_layers=2, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=ffn, vocab=512, lora_rank=rank,
                                  lora_alpha=2.0 * rank, lora_targets=targets)
    g = synth.rng(4, ffn + tokens)
    cuts = [0, tokens // 2, tokens]
    trajs = [[(1, g.integers(0, sh.vocab, size=3).astype(np.int32)), (2, g.integers(0, sh.vocab, size=e - b - 3).astype(np.int32))] for b, e in zip(cuts, cuts[1:])]
    reps = [G.compare_step(sh, 2, trajs, 1, tokens, bf16=True, loss_tol=2e-3, grad_tol=3e-2, recompute=mode) for mode in (0, 2)]
    assert reps[0]["loss"] == reps[1]["loss"] and reps[0]["grads"] == reps[1]["grads"]          # the rewritten product has the forward's bits


@pytest.mark.parametrize("tokens, targets", [(300, ("gate", "up", "down")), (4100, ("gate", "up", "down")), (4100, ("gate", "down"))])
def test_gates_whose_exponential_is_near_the_largest_float(tokens, targets):
    """Gates of -88: 1 + exp(88) is 1.7e38, and its reciprocal no normal float any more, but SiLU(-88) = -5.3e-37 is one, and so is what comes of it
    with large up and down projections.  Every token's hidden row is the same, so that its gate is -88 to 3e-7 (exp: 3e-5 of its value); the other
    operands and the tolerance are the step's."""
    import gpu_util as G
    import oracle
    from helpers import grad_norm_err
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn=192, vocab=512, lora_rank=8, lora_alpha=16.0,
                                  lora_targets=targets)
    params, lora = synth.weights(sh, 6), synth.lora_weights(sh, 6)
    W = params["layers"][0]
    params["embed"][:] = 0.0
    params["embed"][:, 0] = 32.0                             # normalised: 8 in the first column, 0 in the others
    W["wo"][:] = 0.0
    W["g2"][:] = 1.0
    W["wgate"][:, 0] = -11.0
    W["wup"] *= 2.0 ** 60
    W["wdown"] *= 2.0 ** 50                                  # the layer's output is 1e-6 of its input all the same
    lora[0]["gate"] = (1e-7 * lora[0]["gate"][0], lora[0]["gate"][1])     # the gate stays what it is
    params, lora = G.quantise_params(params, True), G.quantise_lora(lora)
    trajs = [[(1, np.full(3, 7, np.int32)), (2, np.full(tokens - 3, 7, np.int32))]]           # one label: the tokens' gradients add up
    res, model, pk, ctx = G.run_step(sh, params, lora, trajs, 1, tokens, mode=B.AS_BF16)
    f, want = oracle.train_step(oracle.config_from_shape(sh), params, lora, pk["tokens"].cpu().numpy(), pk["cu_seqlens"].cpu().numpy(), pk["loss_mask"].cpu().numpy())
    assert f["count"] == res["count"] == tokens - 3
    errs = {(t, k): grad_norm_err(G.to_np(model.lora_grads[0][t][k]), want["lora"][0][t][k]) for t in targets for k in (0, 1)}
    assert max(errs.values()) <= 3e-2, errs
