#!/usr/bin/env python3
"""Writes gemm_rd_loop.inc, gemm_rd_nn_loop.inc and gemm_rd_tn_loop.inc: the main loops of gemm_mfma_rd_kernel (gemm.hip), one tile's
contraction as one inline-asm block each.  Run by hand after a change (python gen_gemm_rd_loop.py); the generated files are committed.

One K step (64 wide) of one wave (a 128 x 128 block of a 256 x 256 tile, four waves, one per SIMD) is two slices of 8 x 8
v_mfma_f32_16x16x32_bf16 of 16 clocks each: 128 slots, slot 64 s + 8 i + j multiplies row block i with column block j.  What was
measured about a slot: it takes three scalar instructions, two vector ones, a wait, an LDS read, a load to registers or a load to LDS
without a clock more, but a ds_write_b128 costs 12 and a ds_write_b64 four.  So tiles go from global memory straight into LDS.

LDS is a ring of five half stages of 32 KB (256 rows x 64 of A, then of B, of one step; 160 KB), filled in the order A_0 B_0 A_1 B_1
...; half stage h lies at h % 5.  In step t, slots:
  1 .. 31    reads of slice 1 of step t (the registers of slice 1 are free since the step before)
  0 .. 42    loads of A_(t+2), into the half stage of B_(t-1)
  44         barrier: every wave has read A_t and B_t
  46 .. 95   loads of B_(t+2), into the half stage of A_t
  96         barrier: this wave's loads of A_(t+1) and B_(t+1) have landed (vmcnt(16): all but A_(t+2), B_(t+2)), and so have all others'
  97 .. 127  reads of slice 0 of step t + 1
so a load has 0.95 to 1.7 steps to arrive.  Behind the last step of a tile the loads go on with the first two steps of the next tile
that the workgroup takes: at its end A_0 B_0 A_1 B_1 of that one are in LDS or under way, in order, A_0 and B_0 landed for all, and the
fifth half stage (that of B_(nt-1)) is free for the epilogue, each wave's quarter of it for that wave: its own loads of A_2 fill it next.
`first` says that there was no such tile before: the block then loads those four itself.

Vector registers: v[0:31], v[32:63] column (B) and row (A) fragments of slice 0, 8 blocks of 4; v[64:127] of slice 1; v[128:131], v[132:135]
LDS read addresses of A, B in this step's half stages; v[136:139] this lane's global offsets of the tile being loaded: A even / odd
load, B even / odd.  Scalar: s[40:41], s[42:43] running bases of the loads of A, B, s44, s45 their strides between loads, s46, s47 LDS
offsets of A_t, B_t, s48 step, s70, s71 LDS offsets the loads of A, B go to, s72 the caller's m0, s60 .. s66 temps.  The accumulators are
a[0:255]: the 32 x 32 block (i, j) of the kernel's array is a[16 (4 i + j) ..], its 16 x 16 block (a, b) four registers at 4 (2 a + b) of
those.  The blocks come out transposed (B fragment first): a lane owns row lane % 16 and four consecutive columns, 4 (lane / 16) ...

LDS layouts: rows of 64 of the contraction (128 bytes) with 16-byte chunk c of row r at c ^ (r / 2 % 8);
NN: B as [K rows, N columns], 64 rows of 512 bytes, 64-byte unit u of row r at u ^ (r % 4), fragments through two transposing reads of
8 bytes a lane; TN: A that way too.  A load instruction fills 1 KB in lane order, so the permutation is in the addresses it reads.
Bases of B in NN: up to three matrices below one another, the second segment's and the next tile's, each minus its first row.
"""
import os

(A_R0, A_R1, A_R2, A_R3, B_R0, B_R1, B_R2, B_R3, OA0E, OA0O, OB0E, OB0O, OA1E, OA1O, OB1E, OB1O,
 PA0, PB0, PA1, PB1, PAN, PBN, SA0, SB0, SA1, SB1, NT0, NT, LIM, OFF0, LDSW, FIRST, PB2, PB3, N1, N2, SK, KA) = range(16, 54)
HALF, RING = 32768, 5 * 32768
A_LOADS = [6 * n for n in range(8)]
B_LOADS = [46 + 7 * n for n in range(8)]
ADVANCE = 2       # slots from a load to the step of its base and of m0
FREE_SLOT, LAND_SLOT = 45, 96
READ_ORDER = [("a", 0)] + [("b", j) for j in range(8)] + [("a", i) for i in range(1, 8)]
READ_SLICE1 = [1 + 2 * k for k in range(16)]
READ_NEXT = [97 + 2 * k for k in range(16)]
LAYOUT = "nt"


def op(n):
    return "%%%d" % n


def frag(which, s, idx):
    return 64 * s + (32 if which == "a" else 0) + 4 * idx


def transposed(which):
    return LAYOUT == "tn" or LAYOUT == "nn" and which == "b"


def text_read(s, which, idx):
    base, areg = frag(which, s, idx), 128 if which == "a" else 132
    if transposed(which):
        return ["ds_read_b64_tr_b16 v[%d:%d], v%d offset:%d" % (base + 2 * q, base + 2 * q + 1, areg + idx // 2, s * 16384 + q * 2048 + (idx & 1) * 32)
                for q in range(2)]
    return ["ds_read_b128 v[%d:%d], v%d offset:%d" % (base, base + 3, areg + s, idx * 2048)]


def read_addresses():
    """LDS read addresses in the half stages at s46, s47"""
    out = ["v_add_u32 v%d, s46, %s" % (128 + k, op(A_R0 + k)) for k in range(4 if transposed("a") else 2)]
    return out + ["v_add_u32 v%d, s47, %s" % (132 + k, op(B_R0 + k)) for k in range(4 if transposed("b") else 2)]


def ring_next(reg, by):
    """reg += by half stages, around the ring"""
    return ["s_add_i32 %s, %s, %d" % (reg, reg, by * HALF), "s_sub_i32 s66, %s, %d" % (reg, RING),
            "s_cmp_lt_i32 %s, %d" % (reg, RING), "s_cselect_b32 %s, %s, s66" % (reg, reg)]


def a_dest():
    """s70: where the loads of A_(t+2) go, four half stages behind A_t (at s46)"""
    return ["s_mov_b32 s70, s46"] + ring_next("s70", 4) + ["s_add_i32 s70, s70, %s" % op(LDSW)]


def bases(which, ahead):
    """Base, stride and lane offsets of the loads of step s48 + ahead (past the end: the next tile's first steps).  From the first
    compare to the last select nothing else may touch scc."""
    a = which == "a"
    lo, hi, st, ve, vo = ("s40", "s41", "s44", "v136", "v137") if a else ("s42", "s43", "s45", "v138", "v139")
    p0, p1, pn, s0, s1 = (PA0, PA1, PAN, SA0, SA1) if a else (PB0, PB1, PBN, SB0, SB1)
    e0, o0, e1, o1 = (OA0E, OA0O, OA1E, OA1O) if a else (OB0E, OB0O, OB1E, OB1O)
    out = ["s_add_i32 s60, s48, %d" % ahead, "s_min_i32 s60, s60, %s" % op(LIM)]
    step = KA if a else SK
    if transposed(which):
        out += ["s_mul_i32 s61, s60, %s" % op(step), "s_mul_hi_u32 s67, s60, %s" % op(step)]
    else:
        out += ["s_lshl_b32 s61, s60, 7", "s_mov_b32 s67, 0"]
    past = ["s_cmp_lt_i32 s60, %s" % op(NT), "s_cselect_b64 s[62:63], s[62:63], %s" % op(pn)]
    if LAYOUT == "tn":
        out += ["s_mov_b32 %s, %s" % (st, op(s0)), "s_mov_b64 s[62:63], %s" % op(p0)] + past
    elif transposed(which):
        out += ["s_mov_b32 %s, %s" % (st, op(s0)),
                "s_cmp_lt_i32 s60, %s" % op(N1), "s_cselect_b64 s[62:63], %s, %s" % (op(p0), op(PB2)),
                "s_cmp_lt_i32 s60, %s" % op(N2), "s_cselect_b64 s[62:63], s[62:63], %s" % op(PB3),
                "s_cmp_lt_i32 s60, %s" % op(NT0), "s_cselect_b64 s[62:63], s[62:63], %s" % op(p1)] + past
    else:
        out += ["s_cmp_lt_i32 s60, %s" % op(NT0), "s_cselect_b64 s[62:63], %s, %s" % (op(p0), op(p1)),
                "s_cselect_b32 %s, %s, %s" % (st, op(s0), op(s1)), "s_cselect_b64 s[64:65], 0, -1"] + past + \
               ["s_cselect_b32 %s, %s, %s" % (st, st, op(s0)), "s_cselect_b64 vcc, s[64:65], 0"]
    out += ["s_add_u32 %s, s62, s61" % lo, "s_addc_u32 %s, s63, s67" % hi]
    if LAYOUT == "tn" or transposed(which):
        out += ["v_mov_b32 %s, %s" % (ve, op(e0)), "v_mov_b32 %s, %s" % (vo, op(o0))]
    else:
        out += ["v_cndmask_b32 %s, %s, %s, vcc" % (ve, op(e0), op(e1)), "v_cndmask_b32 %s, %s, %s, vcc" % (vo, op(o0), op(o1))]
    return out


def text_load(which, n):
    """load n of a wave's eight, and the step to the next (m0 and the base are set in earlier slots)"""
    lo, hi, st, v = ("s40", "s41", "s44", 136) if which == "a" else ("s42", "s43", "s45", 138)
    out = ["global_load_lds_dwordx4 v%d, s[%s:%s]" % (v + (n & 1), lo[1:], hi[1:])]
    return out + ["s_add_u32 %s, %s, %s" % (lo, lo, st), "s_addc_u32 %s, %s, 0" % (hi, hi), "s_add_i32 m0, m0, 1024"]


def acc(i, j):
    base = 16 * (4 * (i // 2) + j // 2) + 4 * (2 * (i % 2) + j % 2)
    return "a[%d:%d]" % (base, base + 3)


def step_ops():
    """the operations of one step: 128 slots, each the MFMA and what is issued behind it"""
    slots = [[("mfma", g // 64, (g % 64) // 8, g % 8)] for g in range(128)]
    for k, (which, idx) in enumerate(READ_ORDER):
        slots[READ_SLICE1[k]].append(("read", 1, which, idx))
        slots[READ_NEXT[k]].append(("read", 0, which, idx))
    for n in range(8):
        for which, at in (("a", A_LOADS[n]), ("b", B_LOADS[n])):
            slots[at].append(("load", which, n))
            slots[at + ADVANCE].append(("other", text_load(which, n)[1:]))
    slots[FREE_SLOT].append(("barrier", None))
    slots[LAND_SLOT].append(("barrier", 16))

    def spread(groups, at):
        """groups of instructions into slots, one group each; a group stays together"""
        assert len(groups) == len(at), (len(groups), len(at))
        for slot, group in zip(at, groups):
            slots[slot].append(("other", group))
    spread([["s_add_i32 s71, s46, %s" % op(LDSW)], ["s_mov_b32 m0, s71"]], (31, A_LOADS[7] + ADVANCE))
    # behind the first barrier: the next step's half stages
    spread([ring_next("s46", 2), ring_next("s47", 2)], (50, 57))
    ad = a_dest()
    spread([ad[:1], ad[1:5], ad[5:]], (62, 64, 65))
    ra = read_addresses()
    spread([[x] for x in ra], (68, 69, 70, 71, 75, 76, 77, 78)[:len(ra)])
    # behind the last load: where the next step's loads of A and B begin, two instructions a slot (the carry stays beside its sum)
    at = 98
    for which in "ab":
        t = bases(which, 3)
        while t:
            take = 1 if len(t) > 1 and t[1].startswith("s_addc") or t[0].startswith("v_") else 2
            if t[0].startswith("s_add_u32"):
                take = 2
            slots[at].append(("other", t[:take]))
            t, at = t[take:], at + 1
    assert at <= 127
    spread([["s_mov_b32 m0, s70"]], (125,))
    return slots


class Waits:
    """replays LDS operations; says which counter wait an operation needs"""

    def __init__(self):
        self.issued = self.done = 0
        self.src = {}

    def read(self, key, count):
        self.issued += count
        self.src[key] = self.issued

    def need(self, idx):
        if idx <= self.done:
            return []
        younger = min(self.issued - idx, 15)               # what the counter can express
        self.done = self.issued - younger
        return ["s_waitcnt lgkmcnt(%d)" % younger]


def emit_step(w, zero):
    """one step's text; zero: the accumulators start with this step"""
    out = []
    for ops in step_ops():
        for o in ops:
            if o[0] == "mfma":
                _, s, i, j = o
                for key in (("a", s, i), ("b", s, j)):
                    out += w.need(w.src[key])
                a, b = frag("a", s, i), frag("b", s, j)
                out.append("v_mfma_f32_16x16x32_bf16 %s, v[%d:%d], v[%d:%d], %s" % (acc(i, j), b, b + 3, a, a + 3, "0" if zero and s == 0 else acc(i, j)))
            elif o[0] == "read":
                _, s, which, idx = o
                text = text_read(s, which, idx)
                w.read((which, s, idx), len(text))
                out += text
            elif o[0] == "load":
                out += text_load(o[1], o[2])[:1]
            elif o[0] == "barrier":
                if o[1] is None:
                    out += w.need(w.issued)                # this wave has read the step
                else:
                    out.append("s_waitcnt vmcnt(%d)" % o[1])
                out.append("s_barrier")
            else:
                out += o[1]
    return out


def generate(layout, out_path=None):
    global LAYOUT
    LAYOUT = layout
    name = "rd" if layout == "nt" else "rd_" + layout
    e = ["s_mov_b32 s72, m0", "s_mov_b32 s46, %s" % op(OFF0), "s_mov_b32 s47, s46"] + ring_next("s47", 1)
    e += ["s_cmp_eq_u32 %s, 0" % op(FIRST), "s_cbranch_scc1 L_%s_on_%%=" % name]
    # no tile before this one: nothing of an earlier one may still be landing or be read
    e += ["s_waitcnt vmcnt(0) lgkmcnt(0)", "s_barrier"]
    for t in range(2):
        for which in "ab":
            e += ["s_mov_b32 s48, 0"] + bases(which, t)
            e += ["s_mov_b32 s70, %s" % ("s46" if which == "a" else "s47")] + (ring_next("s70", 2) if t else []) + ["s_add_i32 m0, s70, %s" % op(LDSW), "s_nop 0"]
            for n in range(8):
                e += text_load(which, n) + ["s_nop 0"]
    e += ["s_waitcnt vmcnt(16)", "s_barrier", "L_%s_on_%%=:" % name, "s_mov_b32 s48, 0"]
    e += read_addresses()
    w = Waits()
    for which, idx in READ_ORDER:
        text = text_read(0, which, idx)
        w.read((which, 0, idx), len(text))
        e += text
    e += a_dest() + bases("a", 2) + bases("b", 2) + ["s_mov_b32 m0, s70"]
    w2 = Waits()
    w2.issued, w2.src = w.issued, dict(w.src)
    first, body = emit_step(w, True), emit_step(w, False)
    again = emit_step(w, False)
    assert again == body                                   # the waits of every later step
    strip = lambda t: [x.rsplit(",", 1)[0] if x.startswith("v_mfma") else x for x in t]  # noqa: E731
    assert strip(first) == strip(body)
    step = ["s_add_i32 s48, s48, 1", "s_cmp_ge_i32 s48, %s" % op(NT)]
    e += first + step + ["s_cbranch_scc1 L_%s_end_%%=" % name, "L_%s_loop_%%=:" % name]
    e += body + step + ["s_cbranch_scc0 L_%s_loop_%%=" % name, "L_%s_end_%%=:" % name]
    # fragments read for a step that does not come; the last products must have written; loads of the next tile stay under way
    e += ["s_waitcnt lgkmcnt(0)", "s_mov_b32 m0, s72", "s_nop 15", "s_nop 15"]

    out = out_path or os.path.join(os.path.dirname(os.path.abspath(__file__)), "gemm_%s_loop.inc" % name)
    with open(out, "w") as f:
        f.write("// Generated by gen_gemm_rd_loop.py -- do not edit.  Main loop of gemm_mfma_rd_kernel.\n")
        f.write("#define GEMM_%s_LOOP_ASM \\\n" % name.upper())
        for ln in e:
            f.write('  "%s\\n" \\\n' % ln)
        f.write('  ""\n')
        regs = ['"v%d"' % i for i in range(140)] + ['"s%d"' % i for i in list(range(40, 49)) + list(range(60, 68)) + [70, 71, 72]]
        f.write("#define GEMM_%s_LOOP_CLOBBERS %s, \"vcc\", \"scc\", \"memory\"\n" % (name.upper(), ", ".join(regs)))
    print("wrote", out, len(e), "instructions")


def main(out_path=None, layout="nt"):
    """one loop to a file, or all of them to their places"""
    for one in [layout] if out_path else ["nt", "nn", "tn"]:
        generate(one, out_path)


if __name__ == "__main__":
    import sys
    main(*sys.argv[1:])
