"""CPU checks of the generated instruction sequences: the attention backward (csrc/gen_attn_dkv_tile.py,
csrc/gen_attn_dq_tile.py -> attn_dkv_tile.inc, attn_dq_tile.inc), the adapter-gradient loop (lora_grad_loop.inc) and
the projection GEMM's loops (gemm_rs_loop.inc, gemm_rs_nn_loop.inc, gemm_rs_tn_loop.inc), these at the end of the file.

The blocks are hand-placed instruction streams for one wave, so what a compiler would guarantee is checked here by
replaying them:
  * the committed .inc files are what the generators write;
  * every LDS read has been waited for (lgkmcnt, LDS operations complete in order) before its registers are used, is
    not overwritten before the MFMA(s) it was made for, and does not land in the operand of the MFMA issued last;
  * a vector instruction reads a matrix result only four or more MFMAs (or, where the sequence has gaps, forty
    instructions) after the end of its chain (nothing interlocks that read), and reads a v_exp result two or more
    instructions later;
  * every fixed register of a block is on its clobber list;
  * the fragments the MFMAs receive are the ones the mathematics asks for: the LDS image of a tile is built as the
    kernels' loads leave it (16-byte chunk c of row r at position c ^ f(r)), the addresses are the kernels' per-lane
    formulas, ds_read_b64_tr_b16 is replayed with the lane layout found on the device (the 16 lanes of a block each
    supply 4 consecutive elements; lane 4 r + k of the block receives element k of the lanes r, r + 4, r + 8, r + 12),
    and the registers of every MFMA's A operand are compared with the definition of that operand;
  * row reads and patch reads are free of LDS bank conflicts (64 banks of 4 bytes; 16 lanes per pass for 16-byte
    reads, 32 for 8-byte reads)."""
import importlib.util
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_22673_amd", "csrc")


def _load(name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _macro(path, name):
    text = open(path).read()
    body = text[text.index("#define " + name):]
    lines = []
    for ln in body.splitlines()[1:]:
        m = re.match(r'\s*"(.*)\\n" \\$', ln)
        if not m:
            break
        lines.append(m.group(1))
    return lines


def _clobbers(path, name):
    text = open(path).read()
    line = [l for l in text.splitlines() if l.startswith("#define " + name)][0]
    return set(re.findall(r'"([a-z]+\d*)"', line))


def _bodies(lines, prefix):
    """mode -> instruction list, cut at the dispatch labels"""
    out, cur, mode = {}, None, None
    for ln in lines:
        m = re.match(r"s_cmp_eq_u32 %\d+, (\d+)", ln)
        if m:
            mode, cur = int(m.group(1)), None
            continue
        if ln.startswith("s_cbranch_scc0 L_%s_not" % prefix):
            cur = []
            continue
        if ln.startswith("s_branch L_%s_end" % prefix):
            out[mode] = cur
            cur = None
            continue
        if cur is not None:
            cur.append(ln)
    return out


def _regs(tok):
    """register token -> list of names: v7 -> ['v7'], v[4:7] -> ['v4'..'v7'], %12 -> ['%12'], else []"""
    tok = tok.strip()
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", tok)
    if m:
        return ["v%d" % i for i in range(int(m.group(1)), int(m.group(2)) + 1)]
    if re.fullmatch(r"v\d+", tok) or re.fullmatch(r"%\d+", tok):
        return [tok]
    return []


def _parse(ln):
    """-> (opcode, written registers, read registers, offset)"""
    op, _, rest = ln.partition(" ")
    off = 0
    m = re.search(r"offset:(\d+)", rest)
    if m:
        off = int(m.group(1))
        rest = rest[:m.start()]
    toks = [t for t in re.split(r",\s*(?![^\[]*\])", rest.strip()) if t]
    if op.startswith("v_mfma"):
        return op, _regs(toks[0]), _regs(toks[1]) + _regs(toks[2]) + _regs(toks[3]), off
    if op.startswith("ds_read"):
        return op, _regs(toks[0]), _regs(toks[1]), off
    if op.startswith("global_load_lds"):
        return op, [], _regs(toks[0]), off
    if op.startswith("v_cmp"):
        return op, [], _regs(toks[1]) + _regs(toks[2]), off
    if op.startswith("v_"):
        reads = []
        for t in toks[1:]:
            reads += _regs(t)
        return op, _regs(toks[0]), reads, off
    return op, [], [], off


def _replay_hazards(ins):
    lds_queue = []                # outstanding LDS reads, oldest first: sets of written registers
    pending = {}                  # register -> True while its LDS read is outstanding
    mfma_count = 0
    mfma_write = {}               # register -> (mfma_count, instruction index) at its last write by an MFMA
    exp_write = {}                # register -> instruction index of the v_exp that wrote it
    frag_owner = {}               # register -> [index of the ds_read that filled it, MFMAs that consumed it]
    frag_regs = set()             # registers that serve as A operands
    mfma_read = {}                # register -> number of MFMAs issued before the last one that read it
    for ln in ins:
        if ln.startswith("v_mfma"):
            frag_regs |= set(_regs([t.strip() for t in re.split(r",\s*(?![^\[]*\])", ln.partition(" ")[2])][1]))
    for idx, ln in enumerate(ins):
        op, wr, rd, _ = _parse(ln)
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", ln)
            if m:
                while len(lds_queue) > int(m.group(1)):
                    for r in lds_queue.pop(0):
                        pending.pop(r, None)
            continue
        for r in rd:
            assert r not in pending, ("register read before its LDS read was waited for", idx, ln, r)
        if op.startswith("v_mfma"):
            for r in rd:
                if r in frag_owner:
                    frag_owner[r][1] += 1
                mfma_read[r] = mfma_count
            mfma_count += 1
            for r in wr:
                mfma_write[r] = (mfma_count, idx)
                exp_write.pop(r, None)
            continue
        if op.startswith("ds_read"):
            for r in wr:
                assert r not in pending, ("LDS read into a register with a read outstanding", idx, ln)
                # the MFMA that read the register last has another one behind it: it has taken its operands
                assert r not in mfma_read or mfma_count - mfma_read[r] >= 2, ("LDS read into the operand of the MFMA just issued", idx, ln)
                if r in frag_owner and r in frag_regs:
                    assert frag_owner[r][1] > 0, ("fragment overwritten before any MFMA used it", idx, ln, r)
                frag_owner[r] = [idx, 0]
                pending[r] = True
                mfma_write.pop(r, None)
            lds_queue.append(list(wr))
            while len(lds_queue) > 15:        # the counter has four bits: the wave does not issue another LDS operation before the oldest is back
                for r in lds_queue.pop(0):
                    pending.pop(r, None)
            continue
        if op.startswith("v_") or op.startswith("global_load_lds"):
            for r in rd:
                if r in mfma_write:
                    assert mfma_count - mfma_write[r][0] >= 4 or idx - mfma_write[r][1] >= 40, ("matrix result read too early", idx, ln, r)
                if r in exp_write and not op.startswith("v_exp"):
                    assert idx - exp_write[r] >= 2, ("v_exp result read by the next instruction", idx, ln, r)
            for r in wr:
                mfma_write.pop(r, None)
                exp_write.pop(r, None)
                if op.startswith("v_exp"):
                    exp_write[r] = idx
    assert not lds_queue, "LDS reads still outstanding at the end of the block"
    assert all(v[1] > 0 for r, v in frag_owner.items() if r in frag_regs), "a fragment was read from LDS and never used"
    return mfma_count


def _fixed_registers(ins):
    out = set()
    for ln in ins:
        _, wr, rd, _ = _parse(ln)
        out |= {r for r in wr + rd if r.startswith("v")}
        out |= {"s" + x for x in re.findall(r"\bs(\d+)\b", ln)}
        for a, b in re.findall(r"s\[(\d+):(\d+)\]", ln):
            out |= {"s%d" % i for i in range(int(a), int(b) + 1)}
    return out


CASES = [("gen_attn_dkv_tile", "attn_dkv_tile.inc", "ATTN_DKV_TILE", "dkv", 64), ("gen_attn_dq_tile", "attn_dq_tile.inc", "ATTN_DQ_TILE", "dq", 96)]


@pytest.mark.parametrize("gen,inc,macro,prefix,n_mfma", CASES)
def test_committed_file_is_what_the_generator_writes(gen, inc, macro, prefix, n_mfma, tmp_path):
    mod = _load(gen)
    out = tmp_path / inc
    mod.main(str(out))
    assert open(out).read() == open(os.path.join(CSRC, inc)).read()


@pytest.mark.parametrize("gen,inc,macro,prefix,n_mfma", CASES)
def test_waits_hazards_and_clobbers(gen, inc, macro, prefix, n_mfma):
    path = os.path.join(CSRC, inc)
    bodies = _bodies(_macro(path, macro + "_ASM"), prefix)
    clob = _clobbers(path, macro + "_CLOBBERS")
    assert {m & 3 for m in bodies} >= {1, 2}
    for mode, ins in bodies.items():
        n = _replay_hazards(ins)
        assert n == (n_mfma if mode & 3 else 0), (mode, n)
        assert _fixed_registers(ins) <= clob, (mode, sorted(_fixed_registers(ins) - clob)[:8])
        loads = sum(1 for ln in ins if ln.startswith("global_load_lds"))
        assert loads == ((9 if prefix == "dkv" else 8) if mode & 4 else 0), (mode, loads)


# ---------------------------------------------------------------- what the MFMAs receive

def _f(row):
    return ((row & 3) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1)


def _lds_image(n_tiles):
    """tiles of [64][128] elements, element id = tile * 8192 + row * 128 + column, stored as the kernels' loads store them"""
    img = np.zeros(n_tiles * 8192, dtype=np.int64)
    for t in range(n_tiles):
        for row in range(64):
            for c in range(16):
                g = c ^ _f(row & 15)
                img[t * 8192 + row * 128 + c * 8: t * 8192 + row * 128 + c * 8 + 8] = t * 8192 + row * 128 + g * 8 + np.arange(8)
    return img


def _lane_addresses():
    aR, aT = np.zeros(64, dtype=np.int64), np.zeros(64, dtype=np.int64)
    for lane in range(64):
        l31, h, sl, mh = lane & 31, lane >> 5, lane & 15, (lane >> 4) & 1
        row0 = 4 * h + (sl >> 2)
        aR[lane] = l31 * 256 + ((h ^ _f(l31 & 15)) * 16)
        aT[lane] = row0 * 256 + (((2 * mh + ((sl & 3) >> 1)) ^ _f(row0)) * 16) + (sl & 1) * 8
    return aR, aT


def _bank_conflicts(addr, nbytes, group):
    worst = 1
    for g0 in range(0, 64, group):
        banks = {}
        for lane in range(g0, g0 + group):
            for w in range(int(addr[lane]) // 4, (int(addr[lane]) + nbytes) // 4):
                banks.setdefault(w % 64, set()).add(w)
        worst = max(worst, max(len(v) for v in banks.values()))
    return worst


def _replay_fragments(ins, op_ar, op_at, n_tiles):
    """-> per MFMA: (destination token, B token, A fragment as [64 lanes][8] element ids); checks the banks on the way"""
    img = _lds_image(n_tiles)
    aR, aT = _lane_addresses()
    vreg = {"%%%d" % op_ar: aR, "%%%d" % op_at: aT}
    out = []
    for ln in ins:
        op, wr, rd, off = _parse(ln)
        if op == "v_xor_b32":
            toks = [t.strip() for t in ln.partition(" ")[2].split(",")]
            if toks[2] in vreg:
                vreg[toks[0]] = vreg[toks[2]] ^ int(toks[1])
        elif op == "ds_read_b128" and rd[0] in vreg and int(wr[0][1:]) >= 64:
            a = vreg[rd[0]] + off
            assert _bank_conflicts(a, 16, 16) == 1, ln
            val = np.stack([img[a // 2 + j] for j in range(8)], axis=1)
            for k in range(4):
                vreg[wr[k]] = val[:, 2 * k:2 * k + 2]
        elif op == "ds_read_b64_tr_b16":
            a = vreg[rd[0]] + off
            assert _bank_conflicts(a, 8, 32) == 1, ln
            val = np.zeros((64, 4), dtype=np.int64)
            for blk in range(4):
                for L in range(16):
                    k, r = L % 4, L // 4
                    for j in range(4):
                        val[blk * 16 + L, j] = img[a[blk * 16 + 4 * j + r] // 2 + k]
            vreg[wr[0]], vreg[wr[1]] = val[:, 0:2], val[:, 2:4]
        elif op.startswith("v_mfma"):
            toks = [t.strip() for t in re.split(r",\s*(?![^\[]*\])", ln.partition(" ")[2])]
            a_regs = _regs(toks[1])
            out.append((toks[0], toks[2], np.concatenate([vreg[r] for r in a_regs], axis=1)))
    return out


def _expect_rows(tile, rb):
    """A operand [32 rows of the tile block rb] x [16 of head_dim]: lane (l31, h) holds row l31, columns 8 h .. 8 h + 7 of the slice"""
    def want(lane, j, ks):
        return tile * 8192 + (rb * 32 + (lane & 31)) * 128 + ks * 16 + (lane >> 5) * 8 + j
    return want


def _expect_cols(tile, cb, x):
    """A operand [32 columns of block cb] x [16 rows of chunk x], rows in the order the B operand holds them"""
    def want(lane, j):
        row = 16 * x + 8 * (j >> 2) + 4 * (lane >> 5) + (j & 3)
        return tile * 8192 + row * 128 + cb * 32 + (lane & 31)
    return want


def test_dkv_fragments():
    g = _load("gen_attn_dkv_tile")
    ins = _bodies(_macro(os.path.join(CSRC, "attn_dkv_tile.inc"), "ATTN_DKV_TILE_ASM"), "dkv")[1]
    frs = _replay_fragments(ins, g.OP_AR, g.OP_AT, 2)                  # tile 0 = Q, tile 1 = dO
    assert len(frs) == 64
    seen = set()
    for dst, b, a in frs:
        lanes, js = np.arange(64)[:, None], np.arange(8)[None, :]
        if dst.startswith("v["):                                        # S or dP of query block qb, slice from the B operand
            base = int(re.match(r"v\[(\d+):", dst).group(1))
            kind, qb = ("S", (base - 128) // 16) if base < 160 else ("dP", (base - 160) // 16)
            ks = int(b[1:]) - (g.OP_KF if kind == "S" else g.OP_VF)
            want = _expect_rows(0 if kind == "S" else 1, qb)(lanes, js, ks)
            seen.add((kind, qb, ks))
        else:                                                           # dV / dK column block, query chunk from the B operand
            o = int(dst[1:])
            kind, cb = ("dK", o - g.OP_DK) if o < g.OP_DV else ("dV", o - g.OP_DV)
            bbase = int(re.match(r"v\[(\d+):", b).group(1))
            x = (bbase - (192 if kind == "dV" else 208)) // 4
            assert (kind == "dV") == (bbase < 208)
            want = _expect_cols(1 if kind == "dV" else 0, cb, x)(lanes, js)
            seen.add((kind, cb, x))
        assert np.array_equal(a, want), (dst, b)
    assert len(seen) == 64


def test_dq_fragments():
    g = _load("gen_attn_dq_tile")
    ins = _bodies(_macro(os.path.join(CSRC, "attn_dq_tile.inc"), "ATTN_DQ_TILE_ASM"), "dq")[1]
    frs = _replay_fragments(ins, g.OP_AR, g.OP_AT, 2)                  # tile 0 = K, tile 1 = V
    assert len(frs) == 96
    seen = set()
    lanes, js = np.arange(64)[:, None], np.arange(8)[None, :]
    for dst, b, a in frs:
        if dst.startswith("v["):
            base = int(re.match(r"v\[(\d+):", dst).group(1))
            kind, t = ("S", (base - 128) // 16) if base < 192 else ("dP", (base - 192) // 16)
            qb, kb = t >> 1, t & 1
            o = int(b[1:]) - (g.OP_QF if kind == "S" else g.OP_DOF)
            assert o // 8 == qb
            want = _expect_rows(0 if kind == "S" else 1, kb)(lanes, js, o % 8)
            seen.add((kind, qb, kb, o % 8))
        else:
            o = int(dst[1:]) - g.OP_DQ
            qb, cb = o // 4, o % 4
            bbase = int(re.match(r"v\[(\d+):", b).group(1))
            assert (bbase - 96) // 16 == qb
            x = ((bbase - 96) % 16) // 4
            want = _expect_cols(0, cb, x)(lanes, js)
            seen.add(("dQ", qb, cb, x))
        assert np.array_equal(a, want), (dst, b)
    assert len(seen) == 96


def test_the_load_swizzle_of_a_row_group_is_the_xor_the_blocks_use():
    """A load instruction of a wave fills four rows; lane -> row lane / 16 of the group, position lane % 16.  The blocks
    take the lane's offset of row group 0 and XOR a constant per group: that must be the chunk c ^ f(row)."""
    for gen in ("gen_attn_dkv_tile", "gen_attn_dq_tile"):
        g = _load(gen)
        for i in range(4):
            text = [t for t in g.load_ops(i) if t.startswith("v_xor_b32")][0]
            const = int(text.split(",")[1])
            for wave in range(4):
                for lane in range(64):
                    l4, c = lane >> 4, lane & 15
                    row = wave * 16 + 4 * i + l4
                    assert ((c ^ _f(l4)) * 16) ^ const == (c ^ _f(row & 15)) * 16


def _min_valu_to_mfma_distance(ins):
    last, best = {}, 10 ** 6
    for idx, ln in enumerate(ins):
        op, wr, rd, _ = _parse(ln)
        if op.startswith("v_mfma"):
            for r in rd:
                if r in last:
                    best = min(best, idx - last[r])
        elif op.startswith("v_"):
            for r in wr:
                last[r] = idx
    return best


@pytest.mark.parametrize("gen,inc,macro,prefix,n_mfma", CASES)
def test_an_mfma_never_reads_a_register_a_vector_instruction_just_wrote(gen, inc, macro, prefix, n_mfma):
    """Operands built by vector instructions directly in front of the MFMA that reads them gave wrong results in the
    adapter-gradient loop (with two temporaries in turn); every block keeps a distance."""
    bodies = _bodies(_macro(os.path.join(CSRC, inc), macro + "_ASM"), prefix)
    for mode, ins in bodies.items():
        assert _min_valu_to_mfma_distance(ins) >= 8, mode


# ---------------------------------------------------------------- the adapter-gradient loop

def test_lora_grad_loop():
    """lora_grad_loop.inc: current; loads are waited for before use (vmcnt, loads return in order) and never land in
    registers that instructions issued less than a step ago still read; operands are built a column ahead."""
    mod = _load("gen_lora_grad_loop")
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "lora_grad_loop.inc")
        mod.main(out)
        assert open(out).read() == open(os.path.join(CSRC, "lora_grad_loop.inc")).read()
    lines = _macro(os.path.join(CSRC, "lora_grad_loop.inc"), "LORA_GRAD_LOOP_ASM")
    clob = _clobbers(os.path.join(CSRC, "lora_grad_loop.inc"), "LORA_GRAD_LOOP_CLOBBERS")
    assert _fixed_registers(lines) <= clob
    start = lines.index("L_tn_loop_%=:")
    end = lines.index("L_tn_end_%=:")
    body = [ln for ln in lines[start + 1:end] if not ln.startswith("s_cbranch")]
    seq = lines[:start] + body + body + body                   # three trips: the steady state
    queue, pending, last_read = [], {}, {}
    n_mfma = 0
    for idx, ln in enumerate(seq):
        op, wr, rd, _ = _parse(ln)
        if op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", ln)
            if m:
                while len(queue) > int(m.group(1)):
                    for r in queue.pop(0):
                        pending.pop(r, None)
            continue
        if op.startswith("global_load_dwordx4"):
            toks = [t.strip() for t in re.split(r",\s*(?![^\[]*\])", ln.partition(" ")[2])]
            dst = _regs(toks[0])
            for r in dst:
                assert r not in pending
                assert idx - last_read.get(r, -10 ** 6) > 16, ("load issued right behind a read of its register", idx, ln)
                pending[r] = True
            queue.append(dst)
            assert len(queue) < 64
            continue
        for r in rd:
            assert r not in pending, ("register used before its load was waited for", idx, ln, r)
            last_read[r] = idx
        n_mfma += op.startswith("v_mfma")
    assert n_mfma == 3 * 4 * 32
    assert _min_valu_to_mfma_distance(seq) >= 4


# ---------------------------------------------------------------- the projection GEMM's loop

def _replay_gemm_loop(lines):
    """the loop replayed over the prologue and three trips of the two-step loop body, with counters kept
    independently of the generator's own: a register is not used while a global load or an LDS read into it is
    outstanding (vmcnt / lgkmcnt, both complete in order); a global load does not land in registers whose LDS store
    may still be reading them; a step's fragment reads never touch an LDS stage that stores issued since the last barrier
    are writing.  Which elements the MFMAs receive is checked by the workgroup run below, for all three loops."""
    start, end = lines.index("L_rs_loop_%=:"), lines.index("L_rs_end_%=:")
    body = [ln for ln in lines[start + 1:end] if not ln.startswith("s_cbranch")]
    seq = lines[:start] + body * 3
    vm_q, lds_q = [], []                      # outstanding global loads / LDS operations, oldest first
    vm_pending, lds_pending = {}, {}          # register -> True while a load / an LDS read into it is outstanding
    store_reads = {}                          # register -> True while an LDS store that reads it is outstanding
    written_since_barrier, read_since_barrier = set(), set()     # LDS stages (0/1 for A, 2/3 for B)
    n_mfma = 0

    def stage_of(addr_reg, off):
        # A stages at LDS offsets 0 / 32768, B stages at 65536 / 98304 (the B part sits in the address registers)
        a = int(addr_reg[1:])
        is_b = a in (196, 197, 198, 199, 202, 203)
        return (2 if is_b else 0) + (off // 32768)

    for idx, ln in enumerate(seq):
        op = ln.split()[0]
        toks = [t.strip() for t in re.split(r",\s*(?![^\[]*\])", ln.partition(" ")[2])]
        if op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", ln)
            if m:
                while len(vm_q) > int(m.group(1)):
                    for r in vm_q.pop(0):
                        vm_pending.pop(r, None)
            m = re.search(r"lgkmcnt\((\d+)\)", ln)
            if m:
                while len(lds_q) > int(m.group(1)):
                    kind, regs = lds_q.pop(0)
                    for r in regs:
                        (lds_pending if kind == "read" else store_reads).pop(r, None)
            continue
        if op == "s_barrier":
            assert not lds_q, ("LDS operations outstanding at the barrier", idx)
            written_since_barrier, read_since_barrier = set(), set()
            continue
        if op == "global_load_dwordx4":
            dst = _regs(toks[0])
            for r in dst:
                assert r not in vm_pending and r not in store_reads, ("load into registers still in use", idx, ln)
                vm_pending[r] = True
            vm_q.append(dst)
            assert len(vm_q) <= 63
            continue
        if op == "ds_write_b128":
            off = int(re.search(r"offset:(\d+)", ln).group(1)) if "offset:" in ln else 0
            src = _regs(toks[1].split(" offset")[0])
            for r in src:
                assert r not in vm_pending, ("LDS store of a register whose load was not waited for", idx, ln)
                store_reads[r] = True
            st = stage_of(toks[0], off)
            assert st not in read_since_barrier, ("store into an LDS stage that is being read", idx, ln)
            written_since_barrier.add(st)
            lds_q.append(("write", src))
            while len(lds_q) > 15:
                kind, regs = lds_q.pop(0)
                for r in regs:
                    (lds_pending if kind == "read" else store_reads).pop(r, None)
            continue
        if op == "ds_read_b128":
            off = int(re.search(r"offset:(\d+)", ln).group(1)) if "offset:" in ln else 0
            dst = _regs(toks[0])
            addr = toks[1].split(" offset")[0].strip()
            if addr.startswith("v"):
                st = stage_of(addr, off)
                assert st not in written_since_barrier, ("fragment read from an LDS stage written since the barrier", idx, ln)
                read_since_barrier.add(st)
            for r in dst:
                assert r not in lds_pending
                lds_pending[r] = True
            lds_q.append(("read", dst))
            while len(lds_q) > 15:
                kind, regs = lds_q.pop(0)
                for r in regs:
                    (lds_pending if kind == "read" else store_reads).pop(r, None)
            continue
        if op.startswith("v_mfma"):
            for r in _regs(toks[1]) + _regs(toks[2]):
                assert r not in lds_pending and r not in vm_pending, ("MFMA on a fragment that was not waited for", idx, ln)
            n_mfma += 1
            continue
        if op.startswith("v_"):
            for t in toks[1:]:
                for r in _regs(t):
                    assert r not in lds_pending and r not in vm_pending, (idx, ln)
    return n_mfma


def test_gemm_rs_loop_replay():
    lines = _macro(os.path.join(CSRC, "gemm_rs_loop.inc"), "GEMM_RS_LOOP_ASM")
    assert _replay_gemm_loop(lines) == 3 * 2 * 64
    # the replay has teeth: planted mistakes inside the loop body are caught
    loop_at = lines.index("L_rs_loop_%=:")

    def without(pred, count=1):
        out, left = [], count
        for i, ln in enumerate(lines):
            if left and i > loop_at and pred(ln):
                left -= 1
                continue
            out.append(ln)
        assert left == 0
        return out

    for planted in (without(lambda ln: ln.startswith("s_waitcnt vmcnt")),             # a store of data that has not arrived
                    without(lambda ln: ln.startswith("s_waitcnt lgkmcnt("), 3),      # an MFMA on fragments still on their way
                    without(lambda ln: ln == "s_barrier")):                          # a stage rewritten while it is read
        with pytest.raises(AssertionError):
            _replay_gemm_loop(planted)


class _GemmWorkgroup:
    """A workgroup of four waves running one of the projection GEMM's loops in lockstep, on element numbers instead of values:
    a 32-bit register of a lane is the pair of elements it holds, an element is its byte address / 2, so every MFMA's operands can be
    compared with the elements the product needs.  What is still under way is unknown (-1): the destination of a load or an
    LDS read until a counter wait that covers it.  LDS is kept per 2 bytes, with the barrier interval and the wave of the last
    write and read: a wave may not read what another wrote, or write what another read, in the same interval."""

    BS, A2, B2 = [2 << 40, 3 << 40, 4 << 40], 5 << 40, 6 << 40         # operand bases, far apart

    def __init__(self, lines, layout, nt, nt0, rows=(), lo=0):
        """nt steps, nt0 of them in segment 0, the first one being step lo of the whole contraction (a split tile);
        rows: first steps, in the whole contraction, of the matrices below the first one (nn)"""
        self.layout, self.nt, self.nt0, self.lines, self.lo, self.rows = layout, nt, nt0, lines, lo, list(rows)
        self.A = (1 << 40) - (300_000 if layout == "tn" else 1_200_000)         # a multiple of 2^32 lies inside what is read
        self.lda, self.ldb, self.lda2, self.ldb2 = 1032, 776, 328, 264
        if layout == "nn":
            self.ldb2 = self.ldb
        self.row0, self.col0 = 512, 256
        self.lds = np.full(65536 + 256 * 32, -1, np.int64)            # 2-byte cells; the scratch lines of the lanes behind the tiles
        self.w_at, self.w_by = np.full(65536, -1), np.full(65536, -1)
        self.r_at, self.r_by = np.full(65536, -1), np.full(65536, -1)
        self.interval = 0
        lane, wave = np.arange(64)[None, :], np.arange(4)[:, None]
        self.v = np.full((4, 256, 64, 2), -1, np.int64)               # elements
        self.addr = np.full((4, 256, 64), -1, np.int64)               # registers that hold byte offsets
        self.s, self.scc, self.vcc = np.zeros((4, 106), np.int64), np.zeros(4, bool), np.zeros(4, bool)
        self.vm, self.lg = [], []                                     # outstanding operations, oldest first: what to do when they are done
        self.mfma = 0
        l31, hh, lrow, lch = lane & 31, lane >> 5, lane >> 3, lane & 7
        wm, wn = wave >> 1, wave & 1
        nn, tn = layout != "nt", layout == "tn"
        x7 = (l31 >> 1) & 7
        line = np.zeros((4, 4, 4, 64), np.int64)                      # [wave, line, entry, lane], the kernel's formulas
        for ks in range(4):
            c = ((2 * ks + hh) ^ x7) * 16
            line[:, 0, ks] = (wm * 128 + l31) * 128 + c
            line[:, 1, ks] = 65536 + (wn * 128 + l31) * 128 + c
            r = (lane >> 2) & 3
            tr = (8 * hh + r) * 512 + (ks ^ r) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8
            if nn:
                line[:, 1, ks] = 65536 + tr + wn * 256
            if tn:
                line[:, 0, ks] = tr + wm * 256
        wrow = (wave * 64 + lrow) * 128
        line[:, 2, 0], line[:, 2, 1] = wrow + (lch ^ (lrow >> 1)) * 16, wrow + (lch ^ ((lrow >> 1) | 4)) * 16
        line[:, 2, 2], line[:, 2, 3] = line[:, 2, 0] + 65536, line[:, 2, 1] + 65536
        if nn:
            r, u = (wave * 16 + hh) * 512 + 65536 + (l31 & 3) * 16, l31 >> 2
            line[:, 2, 2], line[:, 2, 3] = r + (u ^ hh) * 64, r + (u ^ (hh + 2)) * 64
        if tn:
            line[:, 2, 0], line[:, 2, 1] = line[:, 2, 2] - 65536, line[:, 2, 3] - 65536
        for i, ld in enumerate((self.lda, self.ldb, self.lda2, self.ldb2)):
            line[:, 3, i] = (lrow * ld + lch * 8) * 2
        if tn:
            line[:, 3, 0] = line[:, 3, 2] = (hh * self.lda + l31 * 8) * 2
        if nn:
            line[:, 3, 1] = line[:, 3, 3] = (hh * self.ldb + l31 * 8) * 2
        self.line = line
        w, k_skip = np.arange(4), lo * 64
        op = {}
        A0 = self.A + 2 * ((self.row0 + w * 64) * self.lda + k_skip)
        A1 = self.A2 + 2 * (self.row0 + w * 64) * self.lda2
        if layout == "nt":
            op = {17: A0, 18: self.BS[0] + 2 * ((self.col0 + w * 64) * self.ldb + k_skip), 19: A1,
                  20: self.B2 + 2 * (self.col0 + w * 64) * self.ldb2,
                  21: 16 * self.lda, 22: 16 * self.ldb, 23: 16 * self.lda2, 24: 16 * self.ldb2, 25: nt0, 26: nt}
        elif layout == "nn":
            row_w = w * 16 * self.ldb + self.col0
            first = [0] + [64 * x for x in self.rows] + [0] * (2 - len(self.rows))
            base = [self.BS[i] + 2 * (row_w + (k_skip - first[i]) * self.ldb) for i in range(3)]
            n = [self.rows[i] - lo if i < len(self.rows) else nt0 for i in range(2)]
            op = {17: A0, 18: base[0], 19: A1, 20: self.B2 + 2 * (row_w - nt0 * 64 * self.ldb),
                  21: 16 * self.lda, 22: 4 * self.ldb, 23: 16 * self.lda2, 24: 4 * self.ldb, 25: nt0, 26: nt,
                  27: base[1], 28: base[2], 29: n[0], 30: n[1], 31: 128 * self.ldb}
        else:
            At, Bt = self.A + 2 * ((k_skip + w * 16) * self.lda + self.row0), self.BS[0] + 2 * ((k_skip + w * 16) * self.ldb + self.col0)
            op = {17: At, 18: Bt, 19: At, 20: Bt, 21: 4 * self.lda, 22: 4 * self.ldb, 23: 4 * self.lda, 24: 4 * self.ldb, 25: nt, 26: nt,
                  27: 128 * self.lda, 28: 128 * self.ldb}
        self.op = {k: np.broadcast_to(np.asarray(x, np.int64), 4) for k, x in op.items()}

    # ---- scalars: 32-bit registers per wave, pairs for addresses
    def sget(self, t, wide=False):
        t = t.strip()
        if t.startswith("%"):
            return self.op[int(t[1:])]
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", t)
        if m:
            i = int(m.group(1))
            return (self.s[:, i] & 0xffffffff) | (self.s[:, i + 1] << 32)
        if t.startswith("s"):
            return self.s[:, int(t[1:])]
        return np.full(4, int(t))

    def sset(self, t, x):
        t = t.strip()
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", t)
        if t == "vcc":
            self.vcc = x != 0
        elif m:
            i = int(m.group(1))
            self.s[:, i], self.s[:, i + 1] = x & 0xffffffff, (x >> 32) & 0xffffffff
        else:
            self.s[:, int(t[1:])] = (x + (1 << 31)) % (1 << 32) - (1 << 31)          # signed 32 bits

    def scalar(self, op, t):
        u = lambda x: np.asarray(x) & 0xffffffff                                      # noqa: E731
        if op in ("s_mov_b32", "s_mov_b64"):
            self.sset(t[0], self.sget(t[1]))
        elif op == "s_min_i32":
            a, b = self.sget(t[1]), self.sget(t[2])
            self.scc = a < b
            self.sset(t[0], np.minimum(a, b))
        elif op == "s_mul_i32":
            self.sset(t[0], self.sget(t[1]) * self.sget(t[2]))
        elif op == "s_mul_hi_u32":
            self.sset(t[0], (u(self.sget(t[1])) * u(self.sget(t[2]))) >> 32)
        elif op in ("s_add_u32", "s_addc_u32"):
            x = u(self.sget(t[1])) + u(self.sget(t[2])) + (self.scc if op == "s_addc_u32" else 0)
            self.scc = x >> 32 != 0
            self.sset(t[0], x)
        elif op in ("s_add_i32", "s_sub_i32"):
            x = self.sget(t[1]) + (1 if op == "s_add_i32" else -1) * self.sget(t[2])
            self.scc = abs(x) >= 1 << 31
            self.sset(t[0], x)
        elif op == "s_lshl_b32":
            x = u(self.sget(t[1])) << self.sget(t[2])
            self.scc = u(x) != 0
            self.sset(t[0], x)
        elif op == "s_cmp_lt_i32":
            self.scc = self.sget(t[0]) < self.sget(t[1])
        elif op == "s_cmp_ge_i32":
            self.scc = self.sget(t[0]) >= self.sget(t[1])
        elif op in ("s_cselect_b32", "s_cselect_b64"):
            self.sset(t[0], np.where(self.scc, self.sget(t[1]), self.sget(t[2])))
        else:
            raise AssertionError("unknown instruction %s" % op)

    def wait(self, queue, n):
        while len(queue) > n:
            queue.pop(0)()

    def run(self):
        at, label = 0, {ln[:-1]: i for i, ln in enumerate(self.lines) if ln.endswith(":")}
        steps = 0
        while at < len(self.lines):
            ln = self.lines[at]
            at += 1
            if ln.endswith(":"):
                continue
            op, _, rest = ln.partition(" ")
            m = re.search(r"offset:(\d+)", rest)
            off = int(m.group(1)) if m else 0
            t = [x.strip() for x in re.split(r",\s*(?![^\[]*\])", rest.split(" offset")[0])]
            if op == "s_waitcnt":
                for name, queue in (("vmcnt", self.vm), ("lgkmcnt", self.lg)):
                    m = re.search(name + r"\((\d+)\)", rest)
                    if m:
                        self.wait(queue, int(m.group(1)))
            elif op == "s_barrier":
                assert not self.lg, "LDS operations outstanding at the barrier"
                self.interval += 1
            elif op == "s_nop":
                pass
            elif op in ("s_cbranch_scc1", "s_cbranch_scc0"):
                assert (self.scc == self.scc[0]).all()
                if self.scc[0] == (op == "s_cbranch_scc1"):
                    at = label[t[0]]
                steps += 1
                assert steps < 2 * self.nt + 4, "the loop does not end"
            elif op.startswith("s_"):
                self.scalar(op, t)
            elif op == "v_cndmask_b32":
                d, f, g = (int(x[1:]) for x in t[:3])
                self.addr[:, d] = np.where(self.vcc[:, None], self.addr[:, g], self.addr[:, f])
            elif op == "global_load_dwordx4":
                self.load(t)
            elif op == "ds_write_b128":
                self.store(t, off)
            elif op in ("ds_read_b128", "ds_read_b64_tr_b16"):
                self.read(t, off, op != "ds_read_b128")
            elif op.startswith("v_mfma"):
                self.check(t)
            else:
                raise AssertionError("unknown instruction %s" % ln)
        assert not self.vm and not self.lg, "operations left behind the loop"
        return self.mfma

    def free(self, regs, queue):
        """the registers may be written now: no operation under way reads or writes them"""
        for fn in queue:
            assert not set(fn.regs) & set(regs), "a register is taken again while an operation on it is under way"

    def push(self, queue, regs, done=lambda: None):
        def fn():
            done()
        fn.regs = regs
        queue.append(fn)

    def load(self, t):
        d = [int(r[1:]) for r in _regs(t[0])]
        self.free(d, self.vm + self.lg)
        off = self.addr[:, int(t[1][1:])]
        assert (off >= 0).all()
        first = (self.sget(t[2])[:, None] + off) // 2
        self.v[:, d] = -1

        def done():
            for i, r in enumerate(d):
                self.v[:, r, :, 0], self.v[:, r, :, 1] = first + 2 * i, first + 2 * i + 1
        self.push(self.vm, d, done)
        assert len(self.vm) <= 63

    def cells(self, at, n):
        assert (at >= 0).all() and (at % (2 * n) == 0).all() and (at + 2 * n <= 131072).all()
        return at[..., None] // 2 + np.arange(n)

    def store(self, t, off):
        d = [int(r[1:]) for r in _regs(t[1])]
        self.free(d, self.vm)
        c = self.cells(self.addr[:, int(t[0][1:])] + off, 8)
        for w in range(4):
            cw = c[w]
            other = (self.r_by[cw] != w) & (self.r_at[cw] == self.interval)
            assert not other.any(), "a stage is written while another wave reads it"
            assert not ((self.w_by[cw] != w) & (self.w_at[cw] == self.interval)).any()
            self.lds[cw] = self.v[w, d].transpose(1, 0, 2).reshape(64, 8)
            self.w_at[cw], self.w_by[cw] = self.interval, w
        self.push(self.lg, d)

    def read(self, t, off, transposing):
        d = [int(r[1:]) for r in _regs(t[0])]
        self.free(d, self.vm + self.lg)
        if t[1].startswith("%"):                                       # this lane's scratch line: addresses
            self.v[:, d] = -1

            def set_addr(i=off // 16):
                for k, r in enumerate(d):
                    self.addr[:, r] = self.line[:, i, k]
            self.push(self.lg, d, set_addr)
            return
        n = 4 if transposing else 8
        assert len(d) * 2 == n
        c = self.cells(self.addr[:, int(t[1][1:])] + off, n)           # [wave, lane, cell]
        got = np.zeros(c.shape, np.int64)
        for w in range(4):
            cw = c[w]
            assert not ((self.w_by[cw] != w) & (self.w_at[cw] == self.interval)).any(), "a stage is read while another wave writes it"
            mixed = (self.r_at[cw] == self.interval) & (self.r_by[cw] != w)
            self.r_at[cw], self.r_by[cw] = self.interval, np.where(mixed, 4, w)
            got[w] = self.lds[cw]
        if transposing:                                                # lane 4 r + k of sixteen receives element k of the lanes r, r + 4, r + 8, r + 12
            g = got.reshape(4, 4, 4, 4, 4)                             # [wave, block, lane / 4, lane % 4, element]
            got = g.transpose(0, 1, 3, 4, 2).reshape(got.shape)
        self.v[:, d] = -1

        def done():
            for i, r in enumerate(d):
                self.v[:, r] = got[:, :, 2 * i:2 * i + 2]
        self.push(self.lg, d, done)

    def check(self, t):
        step, slot = divmod(self.mfma, 64)
        ks, m = divmod(slot, 16)
        i, j = divmod(m, 4)
        self.mfma += 1
        assert step < self.nt
        assert t[0] == t[3] == "%%%d" % m
        lane, wave = np.arange(64)[None, :, None], np.arange(4)[:, None, None]
        k = (step * 64 if step < self.nt0 else (step - self.nt0) * 64) + ks * 16 + 8 * (lane >> 5) + np.arange(8)      # within its segment
        row, col = self.row0 + (wave >> 1) * 128 + i * 32 + (lane & 31), self.col0 + (wave & 1) * 128 + j * 32 + (lane & 31)
        if step >= self.nt0:
            a = self.A2 // 2 + row * self.lda2 + k
            b = self.B2 // 2 + (k * self.ldb2 + col if self.layout == "nn" else col * self.ldb2 + k)
        else:
            k = k + self.lo * 64
            a = self.A // 2 + (k * self.lda + row if self.layout == "tn" else row * self.lda + k)
            piece = sum(step + self.lo >= r for r in self.rows)
            kb = k - (64 * self.rows[piece - 1] if piece else 0)
            b = self.BS[piece] // 2 + (kb * self.ldb + col if self.layout != "nt" else col * self.ldb + kb)
        for want, tok, what in ((b, t[1], "B"), (a, t[2], "A")):
            d = [int(r[1:]) for r in _regs(tok)]
            assert len(d) == 4
            got = self.v[:, d].transpose(0, 2, 1, 3).reshape(4, 64, 8)
            assert (got == want).all(), "step %d, slice %d, block (%d, %d): not the fragment of %s" % (step, ks, i, j, what)


_GEMM_LOOPS = {"nt": ("gemm_rs_loop.inc", "GEMM_RS_LOOP_ASM"), "nn": ("gemm_rs_nn_loop.inc", "GEMM_RS_NN_LOOP_ASM"),
               "tn": ("gemm_rs_tn_loop.inc", "GEMM_RS_TN_LOOP_ASM")}


def _gemm_loop(layout):
    return _macro(os.path.join(CSRC, _GEMM_LOOPS[layout][0]), _GEMM_LOOPS[layout][1])


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_gemm_loops_multiply_the_right_elements(layout):
    """The loop of a whole workgroup on element numbers: every MFMA of every step receives the rows, columns and contraction indices
    of its block, from the right matrix, for one step and more, odd and even counts, with and without a second segment, for a part of
    a split contraction, and (nn) for two and three matrices below one another, also where a part starts behind the first."""
    lines = _gemm_loop(layout)
    shapes = [dict(nt=n, nt0=n) for n in (1, 2, 3, 6)]
    if layout != "tn":
        shapes += [dict(nt=5, nt0=3), dict(nt=4, nt0=0), dict(nt=4, nt0=2, lo=3)]
    else:
        shapes += [dict(nt=3, nt0=3, lo=2)]
    if layout == "nn":
        shapes += [dict(nt=6, nt0=5, rows=[2]), dict(nt=6, nt0=6, rows=[1, 4]), dict(nt=5, nt0=4, rows=[2, 4], lo=3), dict(nt=3, nt0=3, rows=[1, 2], lo=4)]
    for sh in shapes:
        assert _GemmWorkgroup(lines, layout, **sh).run() == 64 * sh["nt"], sh


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_gemm_loop_mistakes_are_caught(layout):
    """Mistakes planted in the loop's text: each one fails the run above."""
    lines = _gemm_loop(layout)
    loop_at = [i for i, ln in enumerate(lines) if ln.endswith(":")][0]

    def edit(pred, change, skip=0):
        out, done = list(lines), False
        for i, ln in enumerate(lines):
            if not done and i > loop_at and pred(ln):
                skip -= 1
                if skip < 0:
                    out[i:i + 1] = change(ln)
                    done = True
        assert done
        return out

    drop = lambda ln: []                                                                   # noqa: E731
    shift = lambda d: lambda ln: [re.sub(r"offset:(\d+)", lambda m: "offset:%d" % (int(m.group(1)) ^ d), ln)]      # noqa: E731
    is_read = lambda ln: ln.startswith("ds_read")                                          # noqa: E731
    planted = [edit(lambda ln: ln.startswith("s_waitcnt vmcnt"), drop), edit(lambda ln: ln == "s_barrier", drop),
               edit(is_read, drop), edit(is_read, shift(32768)), edit(lambda ln: ln.startswith("ds_write"), drop),
               edit(lambda ln: ln.startswith("ds_write"), shift(1024)), edit(lambda ln: ln.startswith("global_load"), drop),
               [ln for i, ln in enumerate(lines) if i < loop_at or not ln.startswith("s_addc_u32")]]
    # every wait of the loop by itself, but where a stricter one follows at once
    planted += [lines[:i] + lines[i + 1:] for i, ln in enumerate(lines)
                if i > loop_at and ln.startswith("s_waitcnt lgkmcnt") and not lines[i + 1].startswith("s_waitcnt")]
    if layout != "nt":                                                                     # halves of a fragment
        is_tr = lambda ln: ln.startswith("ds_read_b64_tr_b16")                             # noqa: E731
        planted += [edit(is_tr, drop), edit(is_tr, drop, skip=1), edit(is_tr, shift(2048)), edit(is_tr, shift(8192), skip=1)]
    for n, text in enumerate(planted):
        with pytest.raises(AssertionError):
            _GemmWorkgroup(text, layout, nt=6, nt0=6).run()
            print("planted mistake %d was not noticed" % n)


@pytest.mark.parametrize("layout", ["nn", "tn"])
def test_gemm_loops_over_rows_of_the_contraction_are_current(layout, tmp_path):
    """the committed loops that read B, or A and B, by rows of the contraction are the generator's output"""
    import subprocess
    import sys
    committed = os.path.join(CSRC, _GEMM_LOOPS[layout][0])
    out = tmp_path / "loop.inc"
    subprocess.run([sys.executable, os.path.join(CSRC, "gen_gemm_rs_loop.py"), str(out), layout], check=True, capture_output=True)
    assert out.read_text() == open(committed).read()
    clob = _clobbers(committed, "GEMM_RS_%s_LOOP_CLOBBERS" % layout.upper())
    assert _fixed_registers(_gemm_loop(layout)) <= clob
