"""The head with one pass over the vocabulary (exponentials written before their sum is known), and with two where the gradient's product is too small for
one, against float64.

A gradient row is f * (sum_v e_v W_v), e_v rounded to bf16 (half a unit in the last place: 2^-9 relative), the result rounded once more; f and the sum of
the e_v are float.  So |error| <= 2^-9 sum_v |dz_v W_v| + 2^-9 |row|, of which the test allows twice, and 1e-5 of the sum for float arithmetic
(logits up to 300: an exponent is right to 300 * 2^-24 * 1.5)."""
import numpy as np
import pytest
import torch

import synth
from helpers import random_trajs

pytestmark = pytest.mark.gpu


# One pass is taken where the gradient's product has 128 tiles of 256 x 256 or more: 8192 rows of 1024 columns, 1024 of 8192.
@pytest.mark.parametrize("rows, live, d, V, scale, labels", [
    (8192, 8192, 1024, 512, 1.0, "random"),    # whole tiles
    (8192, 257, 1024, 256, 1.0, "random"),     # a ragged tile of one row; a single column tile
    (7937, 7936, 1024, 1280, 8.0, "random"),   # rows past the last whole tile
    (8192, 300, 1024, 1024, 60.0, "random"),
    (8192, 300, 1024, 1024, 60.0, "lowest"),   # labels hundreds below the maximum: blocks of different exponents in a row
    (8192, 511, 1024, 1024, 60.0, "highest"),  # every probability next to 0 or 1
    (8192, 1, 1024, 512, 1.0, "random"),
    (8192, 0, 1024, 512, 1.0, "random"),       # no target
    (9216, 8200, 8192, 256, 8.0, "random"),    # a second chunk of eight rows
    (256, 256, 256, 512, 1.0, "random"),       # from here on two passes: one whole tile
    (512, 257, 256, 256, 1.0, "random"),       # a ragged tile of one row; a single column tile
    (300, 299, 512, 1280, 8.0, "random"),      # rows past the last whole tile
    (512, 300, 256, 1024, 60.0, "lowest"),     # labels hundreds below the maximum
    (512, 511, 256, 1024, 60.0, "highest"),    # every probability next to 0 or 1
    (512, 0, 256, 512, 1.0, "random"),         # no target
])
@pytest.mark.parametrize("weighted", [False, True])
def test_rows_against_float64(rows, live, d, V, scale, labels, weighted):
    from paper_2503_22673_amd import binding as B
    sh = synth.CONFIGS[1].replace(d_model=d, vocab=V)
    ctx = B.Context(B.make_config(sh, mode=B.AS_BF16))
    g = torch.Generator(device="cuda"); g.manual_seed(rows + V)
    cap = (rows + 255) // 256 * 256
    hf = torch.empty(cap, d, dtype=torch.bfloat16, device="cuda").normal_(0, scale / d ** 0.5, generator=g)
    head = torch.empty(V, d, dtype=torch.bfloat16, device="cuda").normal_(0, 1.0, generator=g)
    z = hf[:rows].double() @ head.double().T
    lab = {"lowest": z.argmin(1), "highest": z.argmax(1), "random": torch.randint(0, V, (rows,), device="cuda", generator=g)}[labels].int()
    count = torch.tensor([live], dtype=torch.int32, device="cuda")
    row_w = torch.empty(rows, dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=g) if weighted else None
    ctx.profile(True)
    loss, dhf = ctx.op_head_loss(hf, head, lab, count, row_w=row_w, mode=B.AS_BF16)
    torch.cuda.synchronize()
    prof, chunks = ctx.profile_read(), (cap + 8191) // 8192
    ctx.profile(False)
    # exponentials and dH of every chunk, with two passes a third product; label logits, the end of every chunk's rows
    assert (prof["gemm_devrows"][0], prof["ce"][0]) == ((2 if min(cap, 8192) // 256 * (d // 256) >= 128 else 3) * chunks, 1 + chunks)
    assert not dhf[live:].any().item() and not loss[live:].any().item()
    if not live:
        return
    z, lab, w = z[:live], lab[:live].long(), (row_w[:live].double() if weighted else torch.full((live,), 1.0 / live, dtype=torch.float64, device="cuda"))
    lse = torch.logsumexp(z, 1)
    want = lse - z.gather(1, lab[:, None])[:, 0]
    assert ((loss[:live].double() - want).abs() <= 1e-5 * (1 + z.abs().amax(1))).all()
    dz = (z - lse[:, None]).exp()
    dz[torch.arange(live, device="cuda"), lab] -= 1.0
    dz *= w[:, None]
    ref, mass = dz @ head.double(), dz.abs() @ head.double().abs()
    # where a label's probability is near 1 its element is the difference of the sum and itself: float rounding of either
    mass_f = mass + w.abs()[:, None] * 2 * head[lab].double().abs()
    err = (dhf[:live].double() - ref).abs()
    bound = 2 * 2.0 ** -9 * (mass + ref.abs()) + 1e-5 * (1 + scale) * mass_f
    assert (err <= bound).all(), (err / bound).max().item()


@pytest.mark.parametrize("vocab", [8192, 512])
@pytest.mark.parametrize("assistant_only", [False, True])
def test_pair_step_over_more_rows_than_a_chunk_holds(assistant_only, vocab):
    """10,240 tokens are two chunks of target rows.  Up to 8192 targets the first chunk's exponentials are still there after the losses; beyond
    that the second pass makes them again.  A vocabulary of 8192 is the shortest that the gradient's product is split over, and one pass taken
    for; with one of 512 there are two passes."""
    import test_gpu_dpo as D
    sh = synth.CONFIGS[1].replace(n_layers=1, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=256, vocab=vocab)
    trajs = random_trajs(5, 26, sh.vocab, turn_lo=120, turn_hi=180, turns=(2, 4))
    if assistant_only:
        trajs = [[(2, t) for _, t in tr] for tr in trajs]
    pairs, beta = [(0, 1), (3, 2), (4, 0)], 0.02
    r = D._run(sh, 3, trajs, 4, 2560, pairs, beta, True)
    D._check(r, pairs, beta, True)
    n = int(r["pk"]["loss_mask"].sum().item())
    assert (n > 8300) if assistant_only else (500 < n < 8000)
    r["ctx"].profile(True)
    again = r["ctx"].dpo_step(r["model"], *r["args"], pairs, torch.from_numpy(r["ref"].astype(np.float32)).cuda(), beta, seg_skip=r["pk"]["seg_skip"])
    torch.cuda.synchronize()
    prof = r["ctx"].profile_read()
    r["ctx"].profile(False)
    assert np.array_equal(again["logp"].cpu().numpy().astype(np.float64), r["logp"])
    kept = int(sum(e - b for b, e, skip in zip(r["pk"]["cu_seqlens"][:-1], r["pk"]["cu_seqlens"][1:], r["pk"]["seg_skip"]) if not skip))
    # label logits; over every chunk of the kept tokens: exponentials and the end of the rows, both once more if there are several, and dH
    # (two passes: statistics and the end of the rows, gradient rows, dH)
    chunks = (kept + 8191) // 8192
    one = (3 * chunks, 1 + 2 * chunks) if chunks > 1 else (2, 2)
    assert (prof["gemm_devrows"][0], prof["ce"][0]) == (one if vocab == 8192 else (3 * chunks, 1 + chunks))
