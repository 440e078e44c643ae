"""Float products: the kernels the size rule picks (16x16 and 32x32 results per workgroup with the contraction over four to sixteen waves, 32x32
and 64x64 tiles of FMAs, which variant 1 asks for), at the edges of their tiles and of the 16-wide chunks, rows that are and are not whole 16-byte pieces, one and two segments."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("M,N,K1,K2", [(1, 1, 1, 0), (15, 17, 5, 0), (16, 16, 16, 8), (33, 31, 63, 3), (478, 384, 128, 8), (141, 128, 1024, 0), (300, 8, 344, 0),
                                       (2049, 270, 100, 12), (1025, 1030, 257, 0), (4100, 1100, 68, 4), (999, 1001, 300, 0), (1003, 514, 1001, 16),
                                       (1003, 514, 1000, 16), (2011, 520, 516, 0)])
def test_float_products(M, N, K1, K2, pad, variant):
    from paper_2503_22673_amd import binding as B
    import perf.cases as cases
    ctx = B.Context(cases._config(dict(arch="tiny", layers=1, train="lora", fp32=True)))
    gen = torch.Generator(device="cuda"); gen.manual_seed(M + N)
    new = lambda r, c: torch.empty(r, c + 4 * pad + pad, device="cuda").normal_(generator=gen)      # noqa: E731
    A1, B1, R = new(M, K1), new(N, K1), new(M, N)
    A2, B2 = (new(M, K2), new(N, K2)) if K2 else (None, None)
    out = torch.full((M + 2, N + 3), 7.0, device="cuda")
    ld = lambda t: t.shape[1] if t is not None else 0                                              # noqa: E731
    ctx.check(B.lib.as_op_gemm(ctx.handle, B.AS_FP32, variant, M, N, B._ptr(A1), ld(A1), B._ptr(B1), ld(B1), K1, B._ptr(A2), ld(A2), B._ptr(B2), ld(B2), K2, C.c_float(0.5),
                               B._ptr(R), ld(R), B._ptr(out), N + 3, 0, None, 0, B._stream()))
    torch.cuda.synchronize()
    ref, size = A1[:, :K1].double() @ B1[:, :K1].double().T, A1[:, :K1].double().abs() @ B1[:, :K1].double().abs().T
    if K2:
        ref += A2[:, :K2].double() @ B2[:, :K2].double().T
        size += A2[:, :K2].double().abs() @ B2[:, :K2].double().abs().T
    ref, size = 0.5 * ref + R[:, :N].double(), 0.5 * size + R[:, :N].double().abs()
    # a float sum of K products in any order is off by at most K roundings of the sum of their magnitudes; alpha and R are two more
    assert ((out[:M, :N].double() - ref).abs() <= (K1 + K2 + 3) * 2.0 ** -24 * size).all()
    assert (out[M:] == 7.0).all() and (out[:, N:] == 7.0).all()


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("d,hq,hkv,ffn,vocab,rank", [(128, 4, 2, 328, 301, 5), (96, 3, 1, 200, 1003, 12)])
def test_float_step_at_odd_widths(d, hq, hkv, ffn, vocab, rank, full):
    """gate | up and q | k | v side by side, input gradients over the weights as they lie, adapter gradients 16 columns at a time, where no
    width is a whole tile"""
    import gpu_util as G
    import synth
    from helpers import random_trajs
    sh = synth.CONFIGS[1].replace(n_layers=2, n_q_heads=hq, n_kv_heads=hkv, head_dim=32, d_model=d, ffn=ffn, vocab=vocab, lora_targets=synth.DENSE_TARGETS7, lora_rank=rank)
    trajs = random_trajs(8, 7, sh.vocab, turn_lo=8, turn_hi=30, turns=(2, 5))
    G.compare_step(sh, 8, trajs, 2, 253, bf16=False, loss_tol=1e-4, grad_tol=1e-4, full=full)


def test_float_step_over_many_tokens():
    """some input gradients over transposed copies of the weights, as the size rule has it, some over the weights as they lie"""
    import gpu_util as G
    import synth
    from helpers import random_trajs
    sh = synth.CONFIGS[1].replace(n_layers=1, n_q_heads=8, n_kv_heads=2, head_dim=32, d_model=256, ffn=704, vocab=301, lora_targets=synth.DENSE_TARGETS7, lora_rank=5)
    G.compare_step(sh, 8, random_trajs(8, 90, sh.vocab, turn_lo=8, turn_hi=30, turns=(2, 5)), 2, 2100, bf16=False, loss_tol=1e-4, grad_tol=1e-4)
