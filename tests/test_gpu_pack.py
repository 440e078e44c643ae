"""as_pack on the GPU against the reference packer, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import random_trajs

pytestmark = pytest.mark.gpu


def _ctx(vocab=1024):
    from paper_2503_22673_amd import binding as B
    return B, B.Context(B.make_config(synth.CONFIGS[1].replace(vocab=vocab)))


def _same(B, ctx, trajs, T, rows, pad_id=0, truncate=True):
    ref = oracle.pack(trajs, T, rows, pad_id=pad_id, truncate=truncate)
    got = ctx.pack(*synth.flatten_trajectories(trajs), T, rows, pad_id=pad_id, truncate=truncate)
    torch.cuda.synchronize()
    assert (got["n_rows"], got["n_segments"], got["n_traj_consumed"]) == (ref["n_rows"], ref["n_segments"], ref["n_traj_consumed"])
    assert np.array_equal(got["tokens"].cpu().numpy(), ref["tokens"])
    assert np.array_equal(got["loss_mask"].cpu().numpy(), ref["loss_mask"])
    assert np.array_equal(got["cu_seqlens"].cpu().numpy(), ref["cu_seqlens"])
    return ref


@pytest.mark.parametrize("seed", range(4))
def test_random_batches(seed):
    B, ctx = _ctx(50)
    _same(B, ctx, random_trajs(seed, 60, 50, turn_lo=0, turn_hi=9), 37, 100, pad_id=49)


def test_edge_cases():
    B, ctx = _ctx(100)
    U, A = 1, 2
    _same(B, ctx, [], 16, 4)                                                   # nothing in
    _same(B, ctx, [[(U, [])], [(A, [5])]], 4, 4, pad_id=9)                     # empty trajectory, ragged tail
    _same(B, ctx, [[(U, list(range(1, 8))), (A, list(range(8, 15)))]], 10, 2)  # truncation cuts a turn
    _same(B, ctx, [[(U, [1] * 3), (A, [2] * 3)] for _ in range(10)], 8, 4)     # max_rows stops early
    _same(B, ctx, [[(U, [1] * 4), (A, [2] * 4)] for _ in range(3)], 8, 8)      # rows exactly full: no pad segment


@pytest.mark.parametrize("cfg_id,rows", [(1, 1), (2, 8), (3, 4), (5, 2)])
def test_benchmark_workloads_full_size(cfg_id, rows):
    sh = synth.CONFIGS[cfg_id]
    B, ctx = _ctx(sh.vocab)
    trajs = synth.workload(cfg_id, seed=0)
    ref = _same(B, ctx, trajs, sh.row_len, rows)
    assert ref["n_rows"] == rows


@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("T,rows", [(1, 5), (37, 9), (64, 8)])
def test_outputs_at_any_address(T, rows, shift):
    """The stream is stored in 16-byte pieces where both buffers allow it, else value by value; nothing outside it is touched"""
    B, ctx = _ctx(50)
    trajs = random_trajs(11, 60, 50, turn_lo=0, turn_hi=9)
    ref = oracle.pack(trajs, T, rows, pad_id=49)
    n = rows * T
    tok = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda"); msk = torch.full((n + 8,), 9, dtype=torch.uint8, device="cuda")
    cu = torch.empty(len(trajs) + rows + 1, dtype=torch.int32, device="cuda")
    got = ctx.pack(*synth.flatten_trajectories(trajs), T, rows, pad_id=49, outputs=(tok[shift:shift + n], cu, msk[shift:shift + n]))
    torch.cuda.synchronize()
    live = ref["n_rows"] * T
    assert got["n_rows"] == ref["n_rows"]
    assert np.array_equal(tok[shift:shift + live].cpu().numpy(), ref["tokens"]) and np.array_equal(msk[shift:shift + live].cpu().numpy(), ref["loss_mask"])
    assert (tok[:shift] == -7).all() and (tok[shift + live:] == -7).all() and (msk[:shift] == 9).all() and (msk[shift + live:] == 9).all()


@pytest.mark.parametrize("T,rows", [(64, 8), (4096, 16)])
def test_every_batch_of_a_context_is_its_own(T, rows):
    """The pinned buffer is written by the host and read by the device call after call, at the same addresses: nothing of an earlier batch"""
    B, ctx = _ctx(1000)
    lens = [T // 2, T // 2 - 1, 1, T, T // 3, T // 3, T // 4] * rows
    for step in range(6):
        g = synth.rng(step, 31)
        trajs = [[(1, g.integers(0, 1000, size=n // 2).astype(np.int32)), (2, g.integers(0, 1000, size=n - n // 2).astype(np.int32))] for n in lens]
        _same(B, ctx, trajs, T, rows, pad_id=step)


# ------------------------------------------------- best fit decreasing (as_pack_policy)

def _same_policy(B, ctx, trajs, T, rows, policy, pad_id=0, truncate=True):
    name = {B.AS_PACK_NEXT_FIT: "next_fit", B.AS_PACK_BEST_FIT_DECREASING: "best_fit_decreasing"}[policy]
    ref = oracle.pack(trajs, T, rows, pad_id=pad_id, truncate=truncate, policy=name)
    got = ctx.pack(*synth.flatten_trajectories(trajs), T, rows, pad_id=pad_id, truncate=truncate, policy=policy)
    torch.cuda.synchronize()
    assert (got["n_rows"], got["n_segments"], got["n_traj_consumed"]) == (ref["n_rows"], ref["n_segments"], ref["n_traj_consumed"])
    assert np.array_equal(got["tokens"].cpu().numpy(), ref["tokens"])
    assert np.array_equal(got["loss_mask"].cpu().numpy(), ref["loss_mask"])
    assert np.array_equal(got["cu_seqlens"].cpu().numpy(), ref["cu_seqlens"])
    if "traj_row" in ref:
        assert np.array_equal(got["traj_row"], ref["traj_row"])
    # the skip flags are those of segments without a target inside
    cu, m = ref["cu_seqlens"], ref["loss_mask"]
    assert got["seg_skip"].tolist() == [int(not m[cu[s]:cu[s + 1]].any()) for s in range(len(cu) - 1)]
    return ref, got


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("max_rows", [100, 7])
def test_best_fit_decreasing_random_batches(seed, max_rows):
    B, ctx = _ctx(50)
    _same_policy(B, ctx, random_trajs(seed, 60, 50, turn_lo=0, turn_hi=9), 37, max_rows, B.AS_PACK_BEST_FIT_DECREASING, pad_id=49)


def test_policy_entry_point_edge_cases():
    B, ctx = _ctx(100)
    U, A = 1, 2
    bfd = B.AS_PACK_BEST_FIT_DECREASING
    _same_policy(B, ctx, [], 16, 4, bfd)
    _same_policy(B, ctx, [[(U, [])], [(A, [5])]], 4, 4, bfd, pad_id=9)
    _same_policy(B, ctx, [[(U, list(range(1, 8))), (A, list(range(8, 15)))], [(U, [3])]], 10, 2, bfd)      # truncation to a full row
    _same_policy(B, ctx, [[(U, [1] * 3), (A, [2] * 3)] for _ in range(10)], 8, 4, bfd)                      # more than fits: left out
    _same_policy(B, ctx, [[(U, [1] * 6)], [(A, [2] * 6)], [(U, [3] * 4)], [(A, [4] * 4)]], 10, 9, bfd)      # 6 6 4 4 -> two full rows
    # the next-fit policy through the same entry point equals as_pack, and reports the rows
    trajs = random_trajs(2, 30, 100, turn_lo=0, turn_hi=9)
    ref, got = _same_policy(B, ctx, trajs, 37, 5, B.AS_PACK_NEXT_FIT)
    assert (got["traj_row"][:ref["n_traj_consumed"]] != -1).all() and (got["traj_row"][ref["n_traj_consumed"]:] == -1).all()
    with pytest.raises(B.ASError) as e:
        ctx.pack(*synth.flatten_trajectories(trajs), 37, 5, policy=7)
    assert e.value.code == B.ERR["SHAPE"]
    with pytest.raises(B.ASError) as e:
        ctx.pack(*synth.flatten_trajectories([[(U, [1] * 20)]]), 10, 5, truncate=False, policy=bfd)
    assert e.value.code == B.ERR["TOO_LONG"]


def test_best_fit_decreasing_cuts_the_pad_share_of_the_benchmark_pool():
    """A pool three times the batch of config 3 (lengths of the benchmark's recipe): best fit decreasing fills
    the 4 x 16384 rows almost completely, next fit leaves about a tenth empty."""
    sh = synth.CONFIGS[3]
    B, ctx = _ctx(sh.vocab)
    pool = synth.workload(3, seed=0, rows=3 * sh.rows)
    ref, got = _same_policy(B, ctx, pool, sh.row_len, sh.rows, B.AS_PACK_BEST_FIT_DECREASING)
    nf = ctx.pack(*synth.flatten_trajectories(pool), sh.row_len, sh.rows)
    fill = lambda r: 1.0 - sum(int(b - a) for a, b, s in zip(r["cu_seqlens"].cpu().numpy()[:-1], r["cu_seqlens"].cpu().numpy()[1:], r["seg_skip"])
                               if s and (int(b) % sh.row_len == 0)) / (sh.rows * sh.row_len)
    print("fill: next fit %.4f, best fit decreasing %.4f" % (fill(nf), fill(got)))
    assert got["n_rows"] == sh.rows and fill(got) > 0.99 and fill(got) > fill(nf)
