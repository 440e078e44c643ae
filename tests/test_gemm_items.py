"""How the persistent 256x256 GEMM deals a product out to its workgroups (csrc/gemm_items.h), compiled for the host: every tile and every
step of its contraction exactly once, every address the loop forms inside its operand, loads that nobody reads among them, and the
generated loops run over the items of small launches."""
import os
import subprocess

import numpy as np
import pytest

from test_gemm_rd_loop import _lines, _Workgroup

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NT, NN, TN = 0, 1, 2
NAMES = {NT: "nt", NN: "nn", TN: "tn"}
FIELDS = "wg item row0 col0 row_lo row_hi pid kpart nt0 nt n1 n2 two chain lim".split()
BASES = "a0 a1 b0 b1 b2 b3 bf an bn".split()
LAUNCH = "tiles_m tiles_n tiles first_split parts items nt0 nt tail_first".split()


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("items") / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan", "-static-libubsan",
                        "-I" + os.path.join(ROOT, "paper_2503_22673_amd", "csrc"), os.path.join(ROOT, "tests", "gemm_items_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(**kw):
        p = subprocess.run([exe], input=" ".join("%s=%d" % kv for kv in kw.items()) + "\n", capture_output=True, text=True, timeout=120)
        assert p.returncode == 0, p.stderr[-2000:]
        return p.stdout.splitlines()
    return run


def _launch(driver, **kw):
    lines = driver(**kw)
    assert lines[-1] == "end"
    g = dict(zip(LAUNCH, map(int, lines[0].split()[1:])))
    items = []
    for ln in lines[1:-1]:
        v = [int(x) for x in ln.split()[1:]]
        it = dict(zip(FIELDS, v))
        it.update(zip(BASES, np.asarray(v[len(FIELDS):], np.int64).reshape(4, len(BASES)).T))
        items.append(it)
    assert [it["item"] for it in sorted(items, key=lambda it: it["item"])] == list(range(g["items"]))
    return g, items


def test_rule_of_the_split_last_round(driver):
    """Segments of up to 96 steps each, every rest of a round: parts that fit the scratch and the round, of at least eight steps; more than two
    only where the last one begins inside segment 0, two at its end at the latest (as many as 20,608 of these shapes do)"""
    split, at_segment_1, bad = map(int, driver(rules=96)[0].split()[1:])
    assert bad == 0 and split > 500_000 and at_segment_1 > 20_000


class _Operands:
    """operands far apart, with their extents: (first element, row stride, rows, columns)"""

    def __init__(self, layout, M, N, K1, K2=0, rows=(), cap=0, groups=0, cgs=()):
        self.layout, self.M, self.N, self.K1, self.K2, self.cap = layout, M, N, K1, K2, cap or M
        self.first = [0] + list(rows)                                  # contraction rows at which the matrices of B begin
        self.lda, self.ldb = (1032 if layout == TN else K1 + 24), (776 if layout != NT else K1 + 8)
        self.lda2, self.ldb2 = K2 * max(1, len(cgs)) + 16, (self.ldb if layout == NN else K2 + 40)
        A, Bs, A2, B2 = 1 << 40, [2 << 40, 3 << 40, 4 << 40], 5 << 40, 6 << 40
        self.cgs, self.groups = list(cgs), groups
        ends = self.first[1:] + [K1]
        self.stride = (ends[0] * self.ldb if layout == NN else N * self.ldb) if groups else 0
        self.extent = {"A": (A, self.lda, K1, M) if layout == TN else (A, self.lda, self.cap, K1), "A2": (A2, self.lda2, self.cap, K2 * max(1, len(cgs)))}
        for i, (b, e) in enumerate(zip(self.first, ends)):
            r = e - b if layout != NT else N
            self.extent["B%d" % i] = (Bs[i], self.ldb, r * max(1, groups), N if layout != NT else K1)
        self.extent["Bx"] = (B2, self.ldb2, K2 if layout == NN else N, N if layout == NN else K2)
        self.args = dict(layout=layout, M=M, N=N, K1=K1, K2=K2, A=A, A2=A2, B0=Bs[0], B1=Bs[1], B3=Bs[2], B2=B2, lda=self.lda, ldb=self.ldb, lda2=self.lda2, ldb2=self.ldb2,
                         nn=len(self.first) if layout == NN else 0, nb0=self.first[1] if len(self.first) > 1 else 0, nb1=self.first[2] if len(self.first) > 2 else 0,
                         rows_cap=cap, grp_b_stride=self.stride)
        if cgs:                                                        # column groups: a matrix each
            for i, end in enumerate(cgs):
                w = end - (cgs[i - 1] if i else 0)
                self.extent["B%d" % i], self.extent["Bx%d" % i] = ((10 + i) << 40, self.ldb, w, K1), ((20 + i) << 40, self.ldb2, w, K2)
                self.args.update({"cg_end%d" % i: end, "cg_B%d" % i: (10 + i) << 40, "cg_C%d" % i: (20 + i) << 40, "cg_a%d" % i: i * K2})
            self.args["ncg"] = len(cgs)

    def inside(self, byte, rows, cols, name):
        """[rows x cols] elements from a byte address lie inside the operand; returns row and column of the first"""
        base, ld, R, C = self.extent[name]
        assert byte >= base and byte % 2 == 0, (name, byte)
        r, c = divmod((int(byte) - base) // 2, ld)
        assert r + rows <= R and c + cols <= C, "%s: rows %d + %d of %d, columns %d + %d of %d" % (name, r, rows, R, c, cols, C)
        return r, c


def _check(driver, ops, live=0, off=None, **kw):
    """coverage and addresses of a whole launch; off: first row of every group"""
    if off is not None:
        kw.update({"off%d" % i: v for i, v in enumerate(off)})
        kw["grp_n"] = ops.groups
    kw.setdefault("tiles_m", (ops.cap if off is not None else ops.M) // 256 + (len(off) if off is not None else 1) if live == 1 else -(-ops.M // 256))
    kw.setdefault("grid", 256)
    g, items = _launch(driver, live=live, tiles_n=ops.N // 256, **ops.args, **kw)
    steps, at = {}, {}
    for it in items:
        assert 0 <= it["row0"] <= ops.cap - 256 or live == 0 and "spare" in kw, it
        assert it["row_lo"] < it["row_hi"] and it["row0"] <= it["row_lo"] < it["row0"] + 256
        lo = g["nt"] * it["kpart"] // g["parts"] if it["kpart"] >= 0 else 0
        steps.setdefault(it["pid"], []).append((lo, it["nt"]))
        at.setdefault(it["pid"], set()).add((it["row0"], it["row_lo"], it["row_hi"], it["col0"]))
        grp = sum(1 for o in off[1:-1] if o <= it["row_lo"]) if off is not None else 0
        while off is not None and not off[grp] <= it["row_lo"] < off[grp + 1]:
            grp += 1
        cg = sum(1 for e in ops.cgs if e <= it["col0"])
        colg = it["col0"] - (ops.cgs[cg - 1] if cg else 0)
        for wave in range(4):
            a = lambda n: int(it[n][wave])                             # noqa: E731
            for t in range(it["nt"]):
                seg1, k = t >= it["nt0"], (lo + t) * 64
                assert seg1 == (lo + t >= g["nt0"])
                if ops.layout == TN:
                    assert ops.inside(a("a0") + t * 128 * ops.lda, 16, 256, "A") == (k + wave * 16, it["row0"])
                    assert ops.inside(a("b0") + t * 128 * ops.ldb, 16, 256, "B0") == (k + wave * 16, it["col0"])
                    continue
                k1 = k - ops.K1
                want_a = (it["row0"] + wave * 64, k1 + (ops.args.get("cg_a%d" % cg, 0) if ops.cgs else 0)) if seg1 else (it["row0"] + wave * 64, k)
                assert ops.inside(a("a1" if seg1 else "a0") + t * 128, 64, 64, "A2" if seg1 else "A") == want_a
                if ops.layout == NT:
                    name = ("Bx%d" % cg if ops.cgs else "Bx") if seg1 else "B%d" % cg
                    assert ops.inside(a("b1" if seg1 else "b0") + t * 128, 64, 64, name) == (grp * ops.N + colg + wave * 64, k1 if seg1 else k)
                    continue
                i = sum(1 for f in ops.first[1:] if f <= k)
                base = "b1" if seg1 else "b0" if t < it["n1"] else "b2" if t < it["n2"] else "b3"
                if not seg1 and len(ops.first) < 3 and base == "b3":
                    raise AssertionError("a matrix that is not there")
                ends = ops.first[1:] + [ops.K1]
                assert ops.inside(a(base) + t * 128 * ops.ldb, 16, 256, "Bx" if seg1 else "B%d" % i) == \
                    ((k1 + wave * 16, it["col0"]) if seg1 else (grp * (ends[i] - ops.first[i]) + k - ops.first[i] + wave * 16, it["col0"]))
            if it["nt"] == 0:
                continue
            for t in (it["nt"], it["nt"] + 1):                         # loads behind the last step
                s = min(t, it["lim"])
                ops.inside(a("an") + s * (128 * ops.lda if ops.layout == TN else 128), *((16, 256) if ops.layout == TN else (64, 64)), "A")
                b = a("bn") + s * (128 if ops.layout == NT else 128 * ops.ldb)
                name = [n for n, (base, ld, R, C) in ops.extent.items() if n[0] == "B" and base <= b < base + 2 * ld * R]
                assert len(name) == 1 and name[0][:2] != "Bx", "a load behind the last step lies outside of every matrix of segment 0: %#x" % b
                ops.inside(b, *((64, 64) if ops.layout == NT else (16, 256)), name[0])
    assert g["nt"] == (ops.K1 + ops.K2) // 64 or "k_dev" in kw
    for pid, parts in steps.items():                                   # one after the other, the whole contraction
        assert len(at[pid]) == 1
        end = 0
        for lo, n in sorted(parts):
            assert lo == end
            end = lo + n
        assert end == g["nt"]
    # every row and column of the result in one tile
    seen = np.zeros((ops.cap if off is not None else ops.M, ops.N // 256), np.int64)
    for (row0, lo, hi, col0), in at.values():
        seen[lo:min(hi, row0 + 256), col0 // 256] += 1
    live_rows = np.zeros(len(seen), np.int64)
    if off is not None:
        live_rows[off[0]:off[-1]] = 1
    else:
        live_rows[:max(0, min(ops.M, kw["m_dev"] - kw.get("m_off", 0))) if "m_dev" in kw else ops.M] = 1
    assert (seen == live_rows[:, None]).all()
    return g, items


_PRODUCTS = [(NT, 128, 0, ()), (NT, 192, 64, ()), (NT, 128, 128, ()), (NT, 128, 192, ()), (NT, 64, 192, ()), (NN, 128, 0, ()), (NN, 256, 64, (64, 128)), (NN, 128, 128, (64,)),
             (NN, 192, 256, (64, 128)), (NN, 128, 128, ()), (NN, 64, 320, ()), (TN, 320, 0, ())]


@pytest.mark.parametrize("M,live,parts,layout,K1,K2,rows", [(M, live, parts) + p for M, live in ((768, 0), (1000, 2), (256, 0)) for parts in (1, 2, 3, 5) for p in _PRODUCTS
                                                            if parts <= (p[1] + p[2]) // 64 and (p[0] != TN or M % 256 == 0)])
def test_every_address_of_a_split_product(driver, M, live, parts, layout, K1, K2, rows):
    """Parts of a contraction over two segments and over up to three matrices below one another, whatever begins where: parts without a
    step of segment 0 too, whose loads behind the last step fall back on that segment"""
    split = {} if parts == 1 else dict(tail_first=0, tail_parts=parts, scratch=1)
    _check(driver, _Operands(layout, M, 768, K1, K2, rows), live, grid=4, **split)


@pytest.mark.parametrize("K1,K2", [(1024, 1024), (1024, 1088), (2048, 64), (1088, 1024), (8192, 64)])
def test_split_last_round(driver, K1, K2):
    """One full round and 16 tiles behind it, split as the launcher says; segments of the same length, and one step more in the second one, put
    the second of two parts where segment 1 begins"""
    g, items = _check(driver, _Operands(NT, 4353 - 257, 4352, K1, K2), scratch=1, tail=1)
    assert g["first_split"] == 256 and g["items"] == 256 + 16 * g["parts"] and {it["nt0"] for it in items if it["kpart"] == 1} == ({0} if K2 >= K1 else {min(g["nt0"] - g["nt"] // g["parts"], g["nt"] * 2 // g["parts"] - g["nt"] // g["parts"])})


def test_column_groups(driver):
    _check(driver, _Operands(NT, 700, 1024, 192, 64, cgs=(512, 768, 1024)), 2, grid=5)
    _check(driver, _Operands(NT, 768, 768, 192, 192, cgs=(512, 768)), 0, grid=5, tail_first=0, tail_parts=3, scratch=1)


@pytest.mark.parametrize("layout,rows", [(NT, ()), (NN, (128, 256)), (NN, ())])
@pytest.mark.parametrize("scratch", [0, 1])
@pytest.mark.parametrize("live", [0, 1, 255, 256, 257, 1280, 1536])
def test_rows_counted_on_the_device(driver, layout, rows, scratch, live):
    """no row, one, around a tile, all; split where their tiles fill at most half a round"""
    _check(driver, _Operands(layout, 1536, 512, 384, 0, rows), 1, m_dev=live + 300, m_off=300, scratch=scratch)


@pytest.mark.parametrize("layout,rows", [(NT, ()), (NN, (192,)), (NN, ())])
@pytest.mark.parametrize("scratch", [0, 1])
@pytest.mark.parametrize("off", [(0, 0, 0, 0, 0), (0, 256, 256, 1000, 1300), (40, 300, 300, 1000, 1290), (0, 1, 1, 2, 1300), (1299, 1300, 1300, 1300, 1300)])
def test_rows_of_groups(driver, layout, rows, scratch, off):
    """empty groups, one row, ragged tiles, a last tile moved up; the groups' matrices one after the other"""
    _check(driver, _Operands(layout, 1300, 512, 384, 0, rows, cap=1300, groups=4), 1, off=list(off), scratch=scratch)


def test_rows_of_groups_behind_full_rounds(driver):
    """293 tiles and more: the last round's split, the others whole"""
    off = [0, 5000, 5001, 5001, 11000, 18000]
    g, _ = _check(driver, _Operands(NT, 18000, 1024, 256, 0, cap=18000, groups=5), 1, off=off, scratch=1)
    assert g["tiles"] > 256 and g["first_split"] == 256 and g["parts"] > 1


@pytest.mark.parametrize("k_dev,parts", [(0, 1), (1, 1), (64, 2), (65, 2), (130, 5), (1000, 4)])
def test_contraction_counted_on_the_device(driver, k_dev, parts):
    """fewer live steps than parts: some parts have none"""
    kw = dict(tail_first=0, tail_parts=parts, scratch=1) if parts > 1 else {}
    g, _ = _check(driver, _Operands(TN, 512, 512, 1024), k_dev=k_dev, grid=3, **kw)
    assert g["nt"] == (k_dev + 63) // 64


# ------------------------------------------------------------------ the loops over these items

class _Bounded(_Workgroup):
    """the replay's workgroup, with every load inside its operand"""

    def __init__(self, ops):
        super().__init__(_lines(NAMES[ops.layout]), NAMES[ops.layout])
        self.ops, self.A, self.lda, self.ldb, self.lda2, self.ldb2 = ops, ops.extent["A"][0], ops.lda, ops.ldb, ops.lda2, ops.ldb2
        base = _Workgroup(_lines(NAMES[ops.layout]), NAMES[ops.layout])
        for at, (old, new) in enumerate(((base.lda, ops.lda), (base.ldb, ops.ldb), (base.lda2, ops.lda2), (base.ldb2, ops.ldb2))):
            for o in range(2):                                         # lane offsets: rows of the old stride become rows of the new one
                self.vin[24 + 2 * at + o] = base.vin[24 + 2 * at + o] // (2 * old) * (2 * new) + base.vin[24 + 2 * at + o] % (2 * old)

    def load(self, t):
        src = (self.sget(t[1])[:, None] + self.addr[:, int(t[0][1:])]) // 2
        ok = np.zeros(src.shape, bool)
        for base, ld, R, C in self.ops.extent.values():
            e = src - base // 2
            ok |= (e >= 0) & (e < ld * R) & (e % ld + 8 <= C)
        assert ok.all(), "a load outside of every operand"
        super().load(t)


@pytest.mark.parametrize("layout,K1,K2,rows,parts", [(NT, 128, 128, (), 2), (NT, 128, 192, (), 2), (NT, 64, 192, (), 2), (NT, 192, 64, (), 3), (NN, 128, 128, (), 2), (NN, 128, 128, (64,), 2),
                                                     (NN, 192, 256, (64, 128), 3), (NN, 256, 0, (64, 128), 2), (TN, 320, 0, (), 2), (NT, 128, 0, (), 1), (NN, 64, 64, (), 1)])
def test_loops_over_the_items_of_a_product(driver, layout, K1, K2, rows, parts):
    """The committed loops over what the workgroups of a launch take in turn: the right fragments for every product, nothing read outside
    the operands, parts without a step of segment 0 among them"""
    ops = _Operands(layout, 512, 512, K1, K2, rows)
    split = {} if parts == 1 else dict(tail_first=0, tail_parts=parts, scratch=1)
    g, items = _launch(driver, live=0, tiles_m=2, tiles_n=2, grid=3, **ops.args, **split)
    assert sum(it["nt"] for it in items) == 4 * (K1 + K2) // 64
    for wg in range(3):
        mine = [it for it in items if it["wg"] == wg]
        run, fresh = _Bounded(ops), True
        for n, it in enumerate(mine):
            d = dict(it, rows=[f // 64 for f in ops.first[1:]], lo=g["nt"] * it["kpart"] // g["parts"] if it["kpart"] >= 0 else 0)
            nx = mine[n + 1] if it["chain"] else None
            run.multiply(d, nx, fresh)
            fresh = not it["chain"]
