"""The persistent 256x256 kernel in every layout and over rows counted on the device, its tiles split where few are left for a round: every
entry against float64, the rest of the result untouched."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def _env():
    from paper_2503_22673_amd import binding as B
    import perf.cases as cases
    return B, B.Context(cases._config(dict(arch="1b", layers=1, train="lora")))


def _new(seed):
    gen = torch.Generator(device="cuda"); gen.manual_seed(seed)
    return lambda *s: torch.empty(s, device="cuda").normal_(generator=gen).to(torch.bfloat16)


def _run(B, ctx, layout, A, Bs, out, M, N, K, ldb, alpha=1.0, R=None, accumulate=0, rows=None, row_off=0, off=None, groups=0, stride=0, cap=0, k=None, scratch=True, b_rows=None):
    hb = (C.c_void_p * len(Bs))(*[b.data_ptr() for b in Bs])
    hr = (C.c_int64 * len(Bs))(*(b_rows or [0] * len(Bs)))
    ws = torch.full((B.GEMM_TAIL_SCRATCH_BYTES // 4,), float("nan"), device="cuda") if scratch else None
    ctx.check(B.lib.as_op_gemm_layout(ctx.handle, layout, M, N, K, B._ptr(A), A.stride(0), hb, hr, len(Bs), ldb, C.c_float(alpha), B._ptr(R), R.stride(0) if R is not None else 0,
                                      B._ptr(out), out.stride(0), int(out.dtype == torch.float32), accumulate, B._ptr(rows), row_off, B._ptr(off), groups, stride, cap,
                                      B._ptr(k), B._ptr(ws), B.GEMM_TAIL_SCRATCH_BYTES if scratch else 0, B._stream()))
    torch.cuda.synchronize()


def _same(got, ref, size, K, f32):
    # exact products of N(0, 1) values: K additions in float whose roundings, of sums of size sqrt(K), add up like a random walk, 2^-24 K, and
    # at worst one after the other, K + 3 times the last place of the magnitudes' sum; one rounding to the result's type
    bound = (2.0 ** -23 * (K + 3) * size).clamp_max(1e-5 * max(K, 1) ** 0.5) + (0.0 if f32 else 2.0 ** -8) * ref.abs()
    worst = ((got.double() - ref).abs() / bound.clamp_min(1e-30)).max().item() if ref.numel() else 0.0
    assert worst <= 1.0, worst


def _stack(new, layout, N, K, rows, groups=1):
    """B of every group as its matrices lie, and as [groups, K, N]"""
    if layout == 0:
        b = new(groups, N, K)
        return [b], b.transpose(1, 2), K, groups and N * K
    bs = [new(groups, r, N) for r in rows]
    return bs, torch.cat(bs, 1), N, rows[0] * N


K_LONG = 8192                                                          # 128 steps: from here on the device-side counts split tiles
ROWS = {0: None, 1: [2112, 4096, 1984]}


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("out_f32,with_residual", [(False, True), (True, False)])
@pytest.mark.parametrize("N,live", [(256, 0), (256, 1), (256, 257), (256, 5000), (4096, 2048), (4096, 2049), (4096, 4097), (4096, 4353)])
def test_rows_counted_on_the_device(layout, out_f32, with_residual, N, live):
    """one tile in sixteen parts, 128 tiles in two, 144 whole, 272 and 288 with 16 and 32 behind a full round; rows before and behind the
    live ones stay as they are"""
    B, ctx = _env()
    M, row_off, new = 5000, 3, _new(N + live)
    A, R = new(M + row_off, K_LONG), new(M + row_off, N) if with_residual else None
    Bs, b, ldb, _ = _stack(new, layout, N, K_LONG, ROWS[layout])
    out = torch.full((M + row_off, N), 7.0, dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
    rows = torch.tensor([row_off + live], dtype=torch.int32, device="cuda")
    # (rows are 16-byte aligned whatever row the pointers are moved to)
    _run(B, ctx, layout, A[row_off:], Bs, out[row_off:], M, N, K_LONG, ldb, 0.5, R[row_off:] if with_residual else None, rows=rows, row_off=row_off, b_rows=ROWS[layout])
    lo, hi = row_off, row_off + live
    a = A[lo:hi].double()
    ref, size = 0.5 * (a @ b[0].double()), 0.5 * (a.abs() @ b[0].double().abs())
    if with_residual:
        ref += R[lo:hi].double(); size += R[lo:hi].double().abs()
    _same(out[lo:hi], ref, size, K_LONG, out_f32)
    assert (out[:lo] == 7.0).all() and (out[hi:] == 7.0).all()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("N,off", [(256, (0, 700, 700, 701, 1300)), (1024, (5, 700, 700, 701, 4300)), (4096, (0, 700, 700, 701, 5000)), (4096, (0, 3, 256, 4000, 4990))])
def test_rows_of_all_groups(layout, N, off):
    """ragged and empty groups in one launch, the matrices of a group side by side; under half a round in all, and 64 and 48 tiles behind a full one"""
    B, ctx = _env()
    cap, G, new = max(off[-1], 1300) + (10 if off[-1] == 4990 else 0), len(off) - 1, _new(N + off[1])
    A = new(cap, K_LONG)
    Bs, b, ldb, stride = _stack(new, layout, N, K_LONG, [4096, 4096] if layout else None, G)
    out = torch.full((cap, N), 7.0, dtype=torch.bfloat16, device="cuda")
    _run(B, ctx, layout, A, Bs, out, cap, N, K_LONG, ldb, off=torch.tensor(off, dtype=torch.int32, device="cuda"), groups=G, stride=stride, cap=cap, b_rows=[4096, 4096] if layout else None)
    for e in range(G):
        a, w = A[off[e]:off[e + 1]].double(), b[e].double()
        _same(out[off[e]:off[e + 1]], a @ w, a.abs() @ w.abs(), K_LONG, False)
    assert (out[:off[0]] == 7.0).all() and (out[off[-1]:] == 7.0).all()


@pytest.mark.parametrize("with_residual", [False, True])
@pytest.mark.parametrize("M,rows", [(4353, [2048]), (4352, [576, 64, 1408]), (4300, [64, 1984]), (1000, [64, 64, 64]), (256, [64])])
def test_matrices_below_one_another(M, rows, with_residual):
    """plain rows, 16 tiles behind a full round in four parts that begin and end inside the matrices; few tiles and steps"""
    B, ctx = _env()
    N, K, new = 4096, sum(rows), _new(M + len(rows))
    A, R = new(M, K), new(M, N) if with_residual else None
    Bs, b, ldb, _ = _stack(new, 1, N, K, rows)
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    _run(B, ctx, 1, A, Bs, out, M, N, K, ldb, 0.5, R, b_rows=rows)
    ref, size = 0.5 * (A.double() @ b[0].double()), 0.5 * (A.double().abs() @ b[0].double().abs())
    if with_residual:
        ref += R.double(); size += R.double().abs()
    _same(out, ref, size, K, False)


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("M,N,K,live", [(2048, 2048, 4096, None), (2048, 2048, 4096, 0), (2048, 2048, 4096, 1), (2048, 2048, 4096, 65), (2048, 2048, 4096, 4095), (1024, 2048, 8192, 100),
                                        (4352, 4096, 2048, 130), (4352, 4096, 2048, None)])
def test_contraction_counted_on_the_device(M, N, K, live, accumulate):
    """64 and 32 tiles in three and six parts, 16 behind a full round; no live row, fewer steps than parts, all"""
    B, ctx = _env()
    new = _new(M + (live or 0))
    A, W = new(K, M), new(K, N)
    n = K if live is None else live
    A[n:] = 0; W[n:] = 0
    out = torch.full((M, N), 7.0, device="cuda")
    _run(B, ctx, 2, A, [W], out, M, N, K, N, 0.5, accumulate=accumulate, k=None if live is None else torch.tensor([live], dtype=torch.int32, device="cuda"))
    a, w = A[:n].double().T.contiguous(), W[:n].double()
    ref, size = 0.5 * (a @ w) + 7.0 * accumulate, 0.5 * (a.abs() @ w.abs()) + 7.0 * accumulate
    _same(out, ref, size, n, True)


def test_what_the_kernel_does_not_take():
    B, ctx = _env()
    new = _new(1)
    A, W, out = new(512, 192), new(256, 192), torch.empty(512, 256, device="cuda")
    for kw in (dict(M=255), dict(N=128), dict(K=96), dict(layout=2)):
        a = dict(layout=0, M=512, N=256, K=192); a.update(kw)
        with pytest.raises(B.ASError):
            _run(B, ctx, a["layout"], A, [W], out, a["M"], a["N"], a["K"], 192)
