"""The matrix-core path where its shares of the work can go wrong, against the oracle.

Row counts that leave the last 128-row chunk with at most 64 rows (its own second sweep) or with more; token counts around
the 32-token blocks, the 128-token groups and the splits; ragged batches, whose grid holds live workgroups only; heads long
enough for every form of the combine step; pairs that are scored separately in many blocks.
"""
import pytest
import torch

import oracle
from paper_2510_07651_amd import binding as obc
from paper_2510_07651_amd import synth

from parity_util import TOL, run_case, score_error

pytestmark = pytest.mark.gpu

# (G, W, Hkv, N, lens)
SHAPES = [(1, 9, 2, 127, None), (1, 33, 2, 129, [129, 33]), (1, 64, 1, 4097, None), (5, 13, 2, 1000, [1000, 999, 65]),
          (3, 43, 1, 2111, [65, 2111]), (4, 40, 2, 3000, None), (3, 64, 1, 8200, None), (7, 64, 1, 1500, [700, 1500]),
          (1, 48, 1, 12345, None), (1, 20, 1, 25001, [25001, 64]), (2, 64, 1, 40000, None)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%dx%d_%d" % s[:4])
@pytest.mark.parametrize("range_len", [0, 64])
def test_rows_and_shares_match_oracle(shape, range_len, score_path):
    G, W, Hkv, N, lens = shape
    score_path("mfma")
    obc.obc_set_score_tuning(0, range_len)
    gen = torch.Generator().manual_seed(17)
    B = len(lens or [N])
    q, k, v = (torch.randn(B, H, n, 128, generator=gen).to(torch.bfloat16) for H, n in ((G * Hkv, W), (Hkv, N), (Hkv, N)))
    rows = q.view(B, Hkv, G * W, 128)
    short = min(lens or [N])
    k[:, :, 0] = (3 * rows.float().mean(dim=2)).to(torch.bfloat16)
    for i in range(min(6, short - W)):                     # keys that single rows give nearly all their attention to
        k[:, :, 1 + i * (short - W) // 7] = 2 * rows[:, :, (11 * i) % (G * W)]
    ref = oracle.score(q, k, v, seq_lens=lens)
    for b, n in enumerate(lens or [N]):
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    got = obc.obc_score(q, k, v, "all", seq_lens=lens)
    for i, name in enumerate(("value", "key", "joint")):
        one = obc.obc_score(q, k, v, name, seq_lens=lens)
        for s in (got[i], one):
            err, where = score_error(s.cpu().numpy(), ref[i], max(1, short // 8), lens, TOL["bf16"])
            assert err <= TOL["bf16"], (name, err, where)
    run = torch.full_like(got[2], 2.0)
    obc.obc_score(q, k, v, "joint", seq_lens=lens, scores=run, accumulate=True)
    joint = obc.obc_score(q, k, v, "joint", seq_lens=lens)
    for b, n in enumerate(lens or [N]):
        assert torch.allclose(run[b, :, :n], joint[b, :, :n] + 2.0, rtol=1e-6) and bool((run[b, :, n:] == 2.0).all())


@pytest.mark.parametrize("G,W", [(1, 64), (5, 13), (3, 43)])
@pytest.mark.parametrize("N", [385, 451, 512, 1600])
def test_first_sweep_past_its_splits(G, W, N, score_path):
    """Splits of four blocks (129 rows: two; 1600 tokens: fourteen) whose ring fetches past their end, 64, 65 and 129 rows: a last
    split of one token, of two blocks and three tokens, and full ones; behind the shorter sequence's end stands what is not a number."""
    lens = [N, N - 130]
    score_path("mfma")
    if N > 1536:
        obc.obc_set_score_tuning(4, 0)
    gen = torch.Generator().manual_seed(23)
    q, k, v = (torch.randn(2, H, n, 128, generator=gen).to(torch.bfloat16) for H, n in ((2 * G, W), (2, N), (2, N)))
    ref = oracle.score(q, k, v, seq_lens=lens)
    k[1, :, lens[1]:] = float("nan")
    v[1, :, lens[1]:] = float("nan")
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), "all", seq_lens=lens).cpu().numpy()
    for i, name in enumerate(("value", "key", "joint")):
        err, where = score_error(got[i], ref[i], lens[1] // 8, lens, TOL["bf16"])
        assert err <= TOL["bf16"], (name, err, where)


@pytest.mark.parametrize("G,W,N", [(3, 32, 300), (2, 50, 129), (3, 42, 64), (7, 10, 4097), (1, 1, 40), (1, 63, 63)])
def test_rows_past_the_last_one_weigh_nothing(G, W, N, score_path):
    """96, 100, 126 and 70 rows of a 128-row chunk, 1 and 63 of a 64-row one: on either side of the padded row count."""
    obc.obc_set_sweep2_form(2)
    score_path("mfma")
    run_case(synth.Workload("pad", B=2, Hq=2 * G, Hkv=2, d=128, N=N, W=W, dtype="bf16", budget=max(1, N // 8), seed=79, sinks=1,
                            outlier_channels=4))


@pytest.mark.parametrize("W", [16, 32])
def test_sinks_and_needles_all_over_a_ragged_batch(W, score_path):
    run_case(synth.Workload("needles", B=3, Hq=6, Hkv=2, d=128, N=9000, W=W, dtype="bf16", budget=256, seed=77, sinks=4,
                            outlier_channels=4, needles=64, ragged=(3000, 9000), pad_nan=True))


@pytest.mark.parametrize("form", [0, 1, 2])
def test_few_rows_on_every_form_of_the_second_sweep(form, score_path):
    """Eight rows or fewer keep their logits for a kernel of their own, unless a form is asked for."""
    B, G, Hkv, N = 1, 4, 2, 12001
    score_path("mfma")
    size = []
    for f in (1, form):
        obc.obc_set_sweep2_form(f)
        size.append(obc.obc_score_workspace_bytes(B, N, 1, G * Hkv, Hkv, 128, obc.OBC_BF16, obc.OBC_JOINT))
    assert (size[1] - size[0] >= 4 * G * Hkv * N) == (form == 0)
    run_case(synth.Workload("few_rows", B=B, Hq=G * Hkv, Hkv=Hkv, d=128, N=N, W=1, dtype="bf16", budget=256, seed=78, sinks=2,
                            outlier_channels=4))
