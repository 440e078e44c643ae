"""The loops of the persistent projection GEMM (gemm_rd_loop.inc, gemm_rd_nn_loop.inc, gemm_rd_tn_loop.inc) run on the CPU, on element
numbers instead of values: four waves in lockstep, LDS per 2 bytes with the barrier interval and wave of the last write and read,
loads to LDS landing only when a counter wait covers them.  Two tiles one after the other, as the kernel chains them."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from test_attn_tile_generators import CSRC, _clobbers, _fixed_registers, _macro, _regs

LOOPS = {"nt": ("gemm_rd_loop.inc", "GEMM_RD_LOOP"), "nn": ("gemm_rd_nn_loop.inc", "GEMM_RD_NN_LOOP"), "tn": ("gemm_rd_tn_loop.inc", "GEMM_RD_TN_LOOP")}
HALF = 32768


def _lines(layout):
    return _macro(os.path.join(CSRC, LOOPS[layout][0]), LOOPS[layout][1] + "_ASM")


class _Workgroup:
    BS, A2, B2 = [2 << 40, 3 << 40, 4 << 40], 5 << 40, 6 << 40         # operand bases, far apart

    def __init__(self, lines, layout):
        self.lines, self.layout = lines, layout
        self.A = (1 << 40) - (300_000 if layout == "tn" else 1_200_000)         # a multiple of 2^32 lies inside what is read
        self.lda, self.ldb, self.lda2, self.ldb2 = 1032, 776, 328, 776 if layout == "nn" else 264
        self.lds = np.full(5 * HALF // 2, -1, np.int64)
        self.w_at, self.w_by, self.r_at, self.r_by = (np.full(5 * HALF // 2, -1) for _ in range(4))
        self.interval, self.vm, self.lg = 0, [], []
        self.v, self.addr = np.full((4, 256, 64, 2), -1, np.int64), np.full((4, 256, 64), -1, np.int64)
        lane, wave = np.arange(64)[None, :] + np.zeros((4, 1), np.int64), np.arange(4)[:, None]
        l15, q, r, lrow, lch, l31, hh, wm, wn = lane & 15, lane >> 4, (lane >> 2) & 3, lane >> 3, lane & 7, lane & 31, lane >> 5, wave >> 1, wave & 1
        rows_b, rows_a = layout != "nt", layout == "tn"
        vin = []                                                      # the kernel's formulas
        for w, rows in ((wm, rows_a), (wn, rows_b)):
            for k in range(4):
                vin.append(w * 256 + (8 * q + r) * 512 + (k ^ r) * 64 + (lane & 3) * 8 if rows else w * 16384 + l15 * 128 + ((4 * (k & 1) + q) ^ (l15 >> 1)) * 16)
        off = lambda ld, rows, o: (hh * ld + ((l31 >> 2) ^ (2 * o + hh)) * 32 + (l31 & 3) * 8 if rows else lrow * ld + (lch ^ ((lrow >> 1) | (o * 4))) * 8) * 2      # noqa: E731
        for ld, rows in ((self.lda, rows_a), (self.ldb, rows_b), (self.lda2, False), (self.ldb2, False)):
            vin += [off(ld, rows, o) for o in range(2)]
        self.vin = {16 + i: x for i, x in enumerate(vin)}
        self.half = 0

    def item(self, row0, col0, nt, nt0, rows=(), lo=0):
        """nt steps, nt0 of them in segment 0, the first one being step lo of the whole contraction; rows: first steps, in the whole
        contraction, of the matrices below the first one (nn)"""
        w, k_skip = np.arange(4), lo * 64
        d = dict(row0=row0, col0=col0, nt=nt, nt0=nt0, rows=list(rows), lo=lo, n1=nt0, n2=nt0, b2=w * 0, b3=w * 0)
        d["two"] = nt0 >= 2
        if self.layout == "tn":
            d["a0"] = d["a1"] = self.A + 2 * ((k_skip + w * 16) * self.lda + row0)
            d["b0"] = d["b1"] = self.BS[0] + 2 * ((k_skip + w * 16) * self.ldb + col0)
            d["bf"] = d["b0"]
            return d
        d["a0"] = self.A + 2 * ((row0 + w * 64) * self.lda + k_skip)
        d["a1"] = self.A2 + 2 * ((row0 + w * 64) * self.lda2 - nt0 * 64)
        if self.layout == "nn":
            row_w = w * 16 * self.ldb + col0
            first = [0] + [64 * x for x in rows] + [0] * (2 - len(rows))
            d["b0"], d["b2"], d["b3"] = (self.BS[i] + 2 * (row_w + (k_skip - first[i]) * self.ldb) for i in range(3))
            d["b1"] = self.B2 + 2 * (row_w - nt0 * 64 * self.ldb)
            if len(rows) > 0:
                d["n1"] = rows[0] - lo
            if len(rows) > 1:
                d["n2"] = rows[1] - lo
        else:
            d["b0"] = self.BS[0] + 2 * ((col0 + w * 64) * self.ldb + k_skip)
            d["b1"] = self.B2 + 2 * ((col0 + w * 64) * self.ldb2 - nt0 * 64)
        d["bf"] = d["b0"] if d["n1"] > 0 else d["b2"] if d["n2"] > 0 else d["b3"]
        d["two"] = nt0 >= 2 and (d["n1"] if d["n1"] > 0 else d["n2"] if d["n2"] > 0 else nt0) >= 2
        return d

    def multiply(self, d, nx, fresh):
        """one item, with the loads of the next one's first steps behind it (nx None: its own again)"""
        tn, rows_b = self.layout == "tn", self.layout != "nt"
        step_a, step_b, n = 128 * self.lda if tn else 128, 128 * self.ldb if rows_b else 128, nx or d
        sa, sb = (4 if tn else 16) * self.lda, (4 if rows_b else 16) * self.ldb
        vals = [d["a0"], d["b0"], d["a1"], d["b1"], n["a0"] - d["nt"] * step_a, n["bf"] - d["nt"] * step_b, sa, sb, 16 * self.lda2, 16 * self.ldb2,
                d["nt0"], d["nt"], d["nt"] + (1 if nx or d["two"] else 0), self.half * HALF, np.arange(4) * 8192, int(fresh),
                d["b2"], d["b3"], d["n1"], d["n2"], 128 * self.ldb, 128 * self.lda]
        self.op = {32 + i: np.broadcast_to(np.asarray(x, np.int64), 4) for i, x in enumerate(vals)}
        self.s, self.scc, self.vcc, self.m0 = np.zeros((4, 106), np.int64), np.zeros(4, bool), np.zeros(4, np.int64), np.zeros(4, np.int64)
        self.d, self.mfma = d, 0
        self.run()
        assert self.mfma == 128 * d["nt"]
        self.half = (self.half + 2 * d["nt"]) % 5
        # the epilogue: each wave writes and reads its quarter of the free half stage
        for w in range(4):
            c = ((self.half + 4) % 5 * HALF + w * 8192) // 2 + np.arange(4096)
            assert not ((self.r_by[c] != w) & (self.r_at[c] == self.interval)).any(), "the free half stage is still read"
            assert not any(fn.cells is not None and np.isin(fn.cells[w], c).any() for fn in self.vm), "a load is under way into the free half stage"
            self.lds[c], self.w_at[c], self.w_by[c], self.r_at[c], self.r_by[c] = -1, self.interval, w, self.interval, w

    # ---- registers
    def sget(self, t):
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", t)
        if m:
            return (self.s[:, int(m.group(1))] & 0xffffffff) | (self.s[:, int(m.group(2))] << 32)
        if t.startswith("%"):
            return self.op[int(t[1:])]
        return self.m0 if t == "m0" else self.vcc if t == "vcc" else self.s[:, int(t[1:])] if t.startswith("s") else np.full(4, int(t))

    def sset(self, t, x):
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", t)
        if m:
            self.s[:, int(m.group(1))], self.s[:, int(m.group(2))] = x & 0xffffffff, (x >> 32) & 0xffffffff
        elif t == "vcc":
            self.vcc = x
        elif t == "m0":
            self.m0 = x + 0
        else:
            self.s[:, int(t[1:])] = (x + (1 << 31)) % (1 << 32) - (1 << 31)          # signed 32 bits

    def scalar(self, op, t):
        u = lambda x: np.asarray(x) & 0xffffffff                                      # noqa: E731
        a, b = (self.sget(x) for x in (t + ["0"])[:3][-2:]) if op not in ("s_cmp_lt_i32", "s_cmp_ge_i32", "s_cmp_eq_u32") else (self.sget(x) for x in t)
        if op in ("s_mov_b32", "s_mov_b64"):
            self.sset(t[0], self.sget(t[1]))
        elif op == "s_min_i32":
            self.scc = a < b
            self.sset(t[0], np.minimum(a, b))
        elif op == "s_mul_i32":
            self.sset(t[0], a * b)
        elif op == "s_mul_hi_u32":
            self.sset(t[0], (u(a) * u(b)) >> 32)
        elif op in ("s_add_u32", "s_addc_u32"):
            x = u(a) + u(b) + (self.scc if op == "s_addc_u32" else 0)
            self.scc = x >> 32 != 0
            self.sset(t[0], x)
        elif op in ("s_add_i32", "s_sub_i32"):
            x = a + (1 if op == "s_add_i32" else -1) * b
            self.scc = abs(x) >= 1 << 31
            self.sset(t[0], x)
        elif op == "s_lshl_b32":
            self.scc = u(u(a) << b) != 0
            self.sset(t[0], u(a) << b)
        elif op.startswith("s_cmp"):
            self.scc = a < b if "lt" in op else a >= b if "ge" in op else a == b
        elif op in ("s_cselect_b32", "s_cselect_b64"):
            self.sset(t[0], np.where(self.scc, a, b))
        else:
            raise AssertionError("unknown instruction %s" % op)

    def push(self, queue, regs, done=lambda: None, cells=None):
        def fn():
            done()
        fn.regs, fn.cells = regs, cells
        queue.append(fn)

    def run(self):
        at, jumps, here, m0_set = 0, 0, 0, -9
        label = {ln[:-1]: i for i, ln in enumerate(self.lines) if ln.endswith(":")}
        while at < len(self.lines):
            ln = self.lines[at]
            at, here = at + 1, here + 1
            if ln.endswith(":"):
                continue
            op, _, rest = ln.partition(" ")
            m = re.search(r"offset:(\d+)", rest)
            off = int(m.group(1)) if m else 0
            t = [x.strip() for x in re.split(r",\s*(?![^\[]*\])", rest.split(" offset")[0])]
            if op == "s_waitcnt":
                for name, queue in (("vmcnt", self.vm), ("lgkmcnt", self.lg)):
                    m = re.search(name + r"\((\d+)\)", rest)
                    while m and len(queue) > int(m.group(1)):
                        queue.pop(0)()
            elif op == "s_barrier":
                assert not self.lg, "LDS operations outstanding at the barrier"
                self.interval += 1
            elif op == "s_nop":
                pass
            elif op in ("s_cbranch_scc1", "s_cbranch_scc0"):
                assert (self.scc == self.scc[0]).all()
                if self.scc[0] == (op == "s_cbranch_scc1"):
                    at = label[t[0]]
                jumps += 1
                assert jumps < self.d["nt"] + 4, "the loop does not end"
            elif op.startswith("s_"):
                self.scalar(op, t)
                m0_set = here if t[0] == "m0" else m0_set
            elif op == "v_add_u32":
                self.addr[:, int(t[0][1:])] = self.sget(t[1])[:, None] + self.vin[int(t[2][1:])]
            elif op == "v_mov_b32":
                self.addr[:, int(t[0][1:])] = self.vin[int(t[1][1:])]
            elif op == "v_cndmask_b32":
                self.addr[:, int(t[0][1:])] = np.where(self.vcc[:, None] != 0, self.vin[int(t[2][1:])], self.vin[int(t[1][1:])])
            elif op == "global_load_lds_dwordx4":
                assert here - m0_set > 1, "m0 written right in front of the load that reads it"
                self.load(t)
            elif op in ("ds_read_b128", "ds_read_b64_tr_b16"):
                self.read(t, off, op != "ds_read_b128")
            elif op.startswith("v_mfma"):
                self.check(t)
            else:
                raise AssertionError("unknown instruction %s" % ln)
        assert not self.lg, "LDS reads left behind the loop"

    def load(self, t):
        src = (self.sget(t[1])[:, None] + self.addr[:, int(t[0][1:])]) // 2
        c = (self.m0[:, None, None] + np.arange(64)[None, :, None] * 16) // 2 + np.arange(8)
        assert (c >= 0).all() and (c < len(self.lds)).all() and (self.m0 % 16 == 0).all()
        for w in range(4):
            assert not ((self.r_by[c[w]] != w) & (self.r_at[c[w]] == self.interval)).any(), "a half stage is loaded while another wave reads it"
            assert not any(fn.cells is not None and np.isin(fn.cells[w], c[w]).any() for fn in self.vm), "two loads under way into one place"
            self.lds[c[w]] = -1

        def done():
            for w in range(4):
                self.lds[c[w]] = src[w][:, None] + np.arange(8)
                self.w_at[c[w]], self.w_by[c[w]] = self.interval, w
        self.push(self.vm, [], done, c)
        assert len(self.vm) <= 63

    def read(self, t, off, transposing):
        d = [int(r[1:]) for r in _regs(t[0])]
        assert not any(set(fn.regs) & set(d) for fn in self.lg), "a register is taken again while a read into it is under way"
        n = 4 if transposing else 8
        at = self.addr[:, int(t[1][1:])] + off
        assert len(d) * 2 == n and (at >= 0).all() and (at % (2 * n) == 0).all() and (at + 2 * n <= 5 * HALF).all()
        c = at[..., None] // 2 + np.arange(n)
        got = np.zeros(c.shape, np.int64)
        for w in range(4):
            assert not ((self.w_by[c[w]] != w) & (self.w_at[c[w]] == self.interval)).any(), "a half stage is read while another wave's load may be landing"
            mixed = (self.r_at[c[w]] == self.interval) & (self.r_by[c[w]] != w)
            self.r_at[c[w]], self.r_by[c[w]] = self.interval, np.where(mixed, 4, w)
            got[w] = self.lds[c[w]]
        if transposing:                                                # lane 4 r + k of sixteen receives element k of the lanes r, r + 4, r + 8, r + 12
            got = got.reshape(4, 4, 4, 4, 4).transpose(0, 1, 3, 4, 2).reshape(got.shape)
        self.v[:, d] = -1

        def done():
            for i, r in enumerate(d):
                self.v[:, r] = got[:, :, 2 * i:2 * i + 2]
        self.push(self.lg, d, done)

    def check(self, t):
        """the MFMA's operands and accumulator are those of its block"""
        d = self.d
        step, slot = divmod(self.mfma, 128)
        s, i, j = slot // 64, slot % 64 // 8, slot % 8
        self.mfma += 1
        base = 16 * (4 * (i // 2) + j // 2) + 4 * (2 * (i % 2) + j % 2)
        assert t[0] == "a[%d:%d]" % (base, base + 3) and t[3] == ("0" if step == 0 and s == 0 else t[0])
        lane, wave = np.arange(64)[None, :, None], np.arange(4)[:, None, None]
        k = (step * 64 if step < d["nt0"] else (step - d["nt0"]) * 64) + s * 32 + 8 * (lane >> 4) + np.arange(8)      # within its segment
        row, col = d["row0"] + (wave >> 1) * 128 + i * 16 + (lane & 15), d["col0"] + (wave & 1) * 128 + j * 16 + (lane & 15)
        if step >= d["nt0"]:
            a = self.A2 // 2 + row * self.lda2 + k
            b = self.B2 // 2 + (k * self.ldb2 + col if self.layout == "nn" else col * self.ldb2 + k)
        else:
            k = k + d["lo"] * 64
            a = self.A // 2 + (k * self.lda + row if self.layout == "tn" else row * self.lda + k)
            piece = sum(step + d["lo"] >= r for r in d["rows"])
            kb = k - (64 * d["rows"][piece - 1] if piece else 0)
            b = self.BS[piece] // 2 + (kb * self.ldb + col if self.layout != "nt" else col * self.ldb + kb)
        for want, tok, what in ((b, t[1], "B"), (a, t[2], "A")):
            got = self.v[:, [int(r[1:]) for r in _regs(tok)]].transpose(0, 2, 1, 3).reshape(4, 64, 8)
            assert (got == want).all(), "step %d, slice %d, block (%d, %d): not the fragment of %s" % (step, s, i, j, what)


def _chain(lines, layout, items, chained=True):
    wg = _Workgroup(lines, layout)
    its = [wg.item(**it) for it in items]
    for n, it in enumerate(its):
        nx = its[n + 1] if chained and n + 1 < len(its) and its[n + 1]["two"] else None
        wg.multiply(it, nx, n == 0 or not chained or not it["two"])


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_every_product_gets_its_elements(layout):
    """Items one after the other: one step and more, odd and even counts, with and without a second segment, parts of a split
    contraction, (nn) two and three matrices below one another also where a part begins or ends inside them; an item of one step, after
    which nothing is under way for the next."""
    at = lambda n, **kw: dict(row0=512 * n, col0=256 * (n + 1), **kw)             # noqa: E731
    shapes = [[dict(nt=3, nt0=3), dict(nt=2, nt0=2), dict(nt=6, nt0=6)], [dict(nt=2, nt0=2), dict(nt=1, nt0=1), dict(nt=4, nt0=4)]]
    if layout == "tn":
        shapes += [[dict(nt=3, nt0=3, lo=2), dict(nt=2, nt0=2)]]
    else:
        shapes += [[dict(nt=5, nt0=3), dict(nt=4, nt0=2, lo=3)], [dict(nt=3, nt0=2), dict(nt=2, nt0=1), dict(nt=2, nt0=2)]]
    if layout == "nn":
        shapes += [[dict(nt=6, nt0=5, rows=[2]), dict(nt=6, nt0=6, rows=[1, 4])], [dict(nt=5, nt0=4, rows=[2, 4], lo=3), dict(nt=3, nt0=3, rows=[1, 2], lo=4)],
                   [dict(nt=3, nt0=3, rows=[5, 8], lo=0), dict(nt=3, nt0=3, rows=[5, 8], lo=3), dict(nt=3, nt0=3, rows=[5, 8], lo=6)]]
    for sh in shapes:
        _chain(_lines(layout), layout, [at(n, **it) for n, it in enumerate(sh)])
        _chain(_lines(layout), layout, [at(n, **it) for n, it in enumerate(sh)], chained=False)


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_mistakes_are_caught(layout):
    """every wait, barrier and read of the loop left out by itself, and loads or addresses moved: each one fails the run above"""
    lines = _lines(layout)
    on = [i for i, ln in enumerate(lines) if ln.endswith(":")][0]
    out = []
    for i, ln in enumerate(lines[:-4]):
        # a wait that a stricter one follows at once is none of its own
        if i > on and (ln == "s_barrier" or ln.startswith("s_waitcnt") and not lines[i + 1].startswith("s_waitcnt")) or ln.startswith("s_waitcnt vmcnt(16)"):
            out.append(lines[:i] + lines[i + 1:])
    reads = [i for i, ln in enumerate(lines) if ln.startswith("ds_read")]
    loads = [i for i, ln in enumerate(lines) if ln.startswith("global_load")]
    for i in reads[::7] + loads[::5]:
        out.append(lines[:i] + lines[i + 1:])
    for i in reads[3::9]:
        out.append(lines[:i] + [re.sub(r"offset:(\d+)", lambda m: "offset:%d" % (int(m.group(1)) ^ 2048), lines[i])] + lines[i + 1:])
    for i in [i for i, ln in enumerate(lines) if ln.startswith("s_add_i32 m0, m0")][::6]:
        out.append(lines[:i] + ["s_add_i32 m0, m0, 2048"] + lines[i + 1:])
    items = [dict(row0=0, col0=0, nt=3, nt0=3), dict(row0=256, col0=512, nt=3, nt0=3)]
    missed = []
    for n, text in enumerate(out):
        try:
            _chain(text, layout, items)
            missed.append(n)
        except AssertionError:
            pass
    assert not missed, missed


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_committed_loops_are_current(layout, tmp_path):
    committed, out = os.path.join(CSRC, LOOPS[layout][0]), tmp_path / "loop.inc"
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_gemm_rd_loop.py"), str(out), layout], check=True, capture_output=True)
    assert out.read_text() == open(committed).read()
    clob = _clobbers(committed, LOOPS[layout][1] + "_CLOBBERS")
    assert {r for r in _fixed_registers(_lines(layout)) if not r.startswith("a")} <= clob
