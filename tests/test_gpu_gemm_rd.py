"""The persistent 256x256 kernel on the GPU: workgroups that take one tile and several in turn, contractions of one to four 64-wide steps
(the ring of tiles under way is then shorter than it is deep), an adapter segment, a ragged last row of tiles, both result types."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out_f32,with_residual", [(False, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K1,K2,split", [(2817, 2816, 192, 0, False), (4353, 4096, 64, 0, False), (4353, 4096, 64, 64, False), (9001, 8192, 128, 0, False),
                                             (12289, 4352, 256, 128, False), (4353, 4096, 1024, 64, True),
                                             (4300, 4096, 8192, 64, True), (4300, 4096, 2048, 128, True), (3900, 4352, 2240, 0, True),
                                             (4353, 4096, 1024, 1024, True), (4300, 4096, 1024, 1088, True), (4353, 4096, 1088, 1024, True)])
def test_large_products(M, N, K1, K2, split, out_f32, with_residual):
    # more than half a round of tiles with whole 64-wide steps: always this kernel; split: not below 32 steps, then 16 tiles behind a full
    # round, their contraction in 16, 4 and 4 parts; segments of one length, or one step apart: in two, the second one beginning where
    # segment 1 does, or with the last step before it
    from paper_2503_22673_amd import binding as B
    import perf.cases as cases
    ctx = B.Context(cases._config(dict(arch="1b", layers=1, train="lora")))
    gen = torch.Generator(device="cuda"); gen.manual_seed(M + N + K1)
    new = lambda r, c: torch.empty(r, c, device="cuda").normal_(generator=gen).to(torch.bfloat16)      # noqa: E731
    A1, B1, R = new(M, K1), new(N, K1), new(M, N) if with_residual else None
    A2, B2 = (new(M, K2), new(N, K2)) if K2 else (None, None)
    scratch = torch.empty(B.GEMM_TAIL_SCRATCH_BYTES, dtype=torch.uint8, device="cuda") if split else None
    out = ctx.op_gemm(A1, B1, A2, B2, alpha=0.5, R=R, out_f32=out_f32, mode=B.AS_BF16, tail_scratch=scratch)
    ref, size = A1.double() @ B1.double().T, A1.double().abs() @ B1.double().abs().T
    if K2:
        ref += A2.double() @ B2.double().T
        size += A2.double().abs() @ B2.double().abs().T
    ref, size = 0.5 * ref, 0.5 * size
    if with_residual:
        ref += R.double(); size += R.double().abs()
    # exact products of N(0, 1) values: K additions in float whose roundings, of sums of size sqrt(K), add up like a random walk, 2^-24 K, and
    # at worst one after the other, K + 3 times the last place of the magnitudes' sum; one rounding to the result's type
    bound = ((K1 + K2 + 3) * 2.0 ** -23 * size).clamp_max(1e-5 * (K1 + K2) ** 0.5) + (0.0 if out_f32 else 2.0 ** -8) * ref.abs()
    assert ((out.double() - ref).abs() <= bound).all()
