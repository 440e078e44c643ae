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
