"""The general scoring path where its tiles and pieces can go wrong, against the oracle and against itself.

Row counts around the 16-row tiles and their chunks, token counts around the 64-token tiles, ranges and splits, both
types and head sizes; then caches whose logits exceed the workspace plan, which are scored in pieces of rows and of tokens.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_07651_amd import binding as obc

from parity_util import TOL, score_error

pytestmark = pytest.mark.gpu

# (dtype, d, G, W, N, lens): rows G*W and tokens at and next to tile edges
EDGES = [("fp32", 64, 1, 1, 1, None), ("fp32", 128, 1, 15, 63, None), ("fp32", 64, 1, 16, 64, [64, 17]),
         ("fp32", 128, 1, 17, 65, [65, 64]), ("bf16", 64, 2, 16, 129, None), ("fp32", 64, 3, 11, 4097, [4097, 4032]),
         ("bf16", 64, 7, 9, 4160, [4160, 4159]), ("fp32", 128, 4, 16, 4161, None), ("bf16", 64, 13, 5, 1000, [1000, 65]),
         ("fp32", 128, 8, 64, 300, [300, 64]), ("bf16", 128, 3, 43, 700, [700, 321])]


def _inputs(dtype, d, G, W, N, B, Hkv, seed):
    gen = torch.Generator().manual_seed(seed)
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    q, k, v = (torch.randn(B, H, n, d, generator=gen).to(dt) for H, n in ((G * Hkv, W), (Hkv, N), (Hkv, N)))
    k[:, :, 0] = (3 * q.float().view(B, Hkv, G * W, d).mean(dim=2)).to(dt)
    return q, k, v


# (dtype, d, Hkv, G, W, N, lens) where a sequence is swept in splits with a reference each: one token more than a split's tiles and
# one short of them, as many splits as there are and a single one, sequences that end splits early, windows as long as a split (whose
# first rows see nothing of the last one), rows that fill a workgroup's row blocks in part, heads in two launches
SPLITS = [("bf16", 64, 1, 1, 17, 17, None), ("bf16", 64, 1, 4, 64, 4097, None), ("bf16", 64, 2, 4, 16, 4095, [4095, 130]),
          ("bf16", 64, 9, 5, 7, 705, None), ("bf16", 128, 1, 4, 33, 8191, None), ("fp32", 128, 1, 3, 44, 8193, [8193, 129]),
          ("fp32", 64, 8, 4, 5, 1089, None), ("fp32", 128, 3, 3, 43, 2999, None), ("fp32", 64, 2, 3, 63, 4161, [65, 4161]),
          ("fp32", 128, 40, 4, 32, 4999, None),
          # over 64 rows in workgroups of 64, the last one with 2, 36, 50 or all of its rows, and 140 rows in workgroups of 128
          ("bf16", 64, 2, 4, 25, 300, None), ("fp32", 64, 2, 4, 35, 3910, None), ("fp32", 128, 2, 5, 26, 3000, [3000, 1999]),
          ("bf16", 64, 1, 2, 64, 5001, None), ("bf16", 64, 2, 2, 50, 9001, [9001, 64])]


@pytest.mark.parametrize("case", SPLITS, ids=lambda c: "%s_d%d_%d_%dx%d_%d" % c[:6])
def test_splits_with_references_of_their_own_match_oracle(case, score_path):
    """The largest logit of a row stands in several splits at once (equal keys, unequal values), for half of the heads with most of
    the row's weight."""
    dtype, d, Hkv, G, W, N, lens = case
    B = 1 if lens is None else len(lens)
    q, k, v = _inputs(dtype, d, G, W, N, B, Hkv, 47)
    k[:, ::2, 0] *= 4
    for at in (N // 3, N // 2, N - W):
        k[:, :, at] = k[:, :, 0]
    ref = oracle.score(q, k, v, seq_lens=lens)
    score_path("plain")
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), "all", seq_lens=lens).cpu().numpy()
    for i, name in enumerate(("value", "key", "joint")):
        err, where = score_error(got[i], ref[i], min(lens or [N]) // 8, lens, TOL["fp32"])
        assert err <= TOL["fp32"], (name, err, where)


# (dtype, d, G, W, N, lens): windows whose last chunk of 128 (64) rows leaves two or three (three) of its row blocks empty, the last
# one in use full or with 8, 2 or 1 rows, and whose rows stop seeing tokens in each of a block's sixteen places.  66, 80 and 96 rows are
# one chunk of 128, 144 and 129 three of 64, 200 two of 128
EMPTY = [("fp32", 128, 2, 33, 1900, None), ("bf16", 64, 2, 40, 2601, [2601, 1999]), ("fp32", 64, 2, 48, 2055, None),
         ("bf16", 64, 3, 48, 1500, None), ("fp32", 128, 3, 43, 1203, [1203, 700]), ("bf16", 64, 4, 50, 1700, None),
         ("fp32", 128, 4, 50, 1105, [1105, 640])]


@pytest.mark.parametrize("variant", ["all", "key", "value"])
@pytest.mark.parametrize("case", EMPTY, ids=lambda c: "%s_d%d_%dx%d_%d" % c[:5])
def test_row_blocks_without_rows(case, variant, score_path):
    """A row's largest logit stands in every place of a block of sixteen tokens in turn (row i's at token 100 + 17 i)."""
    dtype, d, G, W, N, lens = case
    q, k, v = _inputs(dtype, d, G, W, N, 1 if lens is None else len(lens), 2, 51)
    rows = q.view(q.shape[0], 2, G * W, d)
    for i in range(min(G * W, 32)):
        k[:, :, 100 + 17 * i] = (1.5 if i % 2 else 3) * rows[:, :, i]        # (some with most of the row's weight)
    ref = oracle.score(q, k, v, seq_lens=lens)
    score_path("plain")
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), variant, seq_lens=lens).cpu().numpy()
    names = ("value", "key", "joint")
    for i, name in enumerate(names if variant == "all" else (variant,)):
        err, where = score_error(got[i] if variant == "all" else got, ref[names.index(name)], min(lens or [N]) // 8, lens, TOL["fp32"])
        assert err <= TOL["fp32"], (name, err, where)


# (dtype, d, Hkv, G, W, N) on either side of where the route changes: five tiles and sixteen of short bf16 calls; twelve heads of 17 to
# 32 fp32 rows; 128 and 160 tiles of longer windows
ROUTES = [("bf16", 64, 2, 4, 5, 256), ("bf16", 64, 2, 4, 5, 257), ("bf16", 64, 2, 4, 5, 1025), ("fp32", 64, 11, 1, 20, 1100),
          ("fp32", 64, 12, 1, 20, 1100), ("fp32", 128, 2, 2, 40, 5120), ("fp32", 128, 2, 2, 40, 5056), ("fp32", 64, 2, 1, 33, 4032)]


@pytest.mark.parametrize("variant", ["joint", "value", "attn", "vatp"])
@pytest.mark.parametrize("case", ROUTES, ids=lambda c: "%s_d%d_%d_%dx%d_%d" % c)
def test_every_score_on_either_side_of_a_route(case, variant):
    """Which kernels take a call depends on whether its score needs the outputs."""
    dtype, d, Hkv, G, W, N = case
    q, k, v = _inputs(dtype, d, G, W, N, 1, Hkv, 48)
    ref = {"attn": oracle.attn_score, "vatp": oracle.vatp_score}.get(variant, lambda *x: oracle.score(*x)[("value", "key", "joint").index(variant)])(q, k, v)
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), variant).cpu().numpy()
    err, where = score_error(got, ref, N // 8, None, TOL["fp32"])
    assert err <= TOL["fp32"], (err, where)


@pytest.mark.parametrize("case", EDGES, ids=lambda c: "%s_d%d_%dx%d_%d" % c[:5])
def test_tile_edges_match_oracle(case, score_path):
    dtype, d, G, W, N, lens = case
    B, Hkv = (1 if lens is None else len(lens)), 2
    q, k, v = _inputs(dtype, d, G, W, N, B, Hkv, 31)
    ref = oracle.score(q, k, v, seq_lens=lens)
    if lens is not None:
        for b, n in enumerate(lens):
            k[b, :, n:] = float("nan")
            v[b, :, n:] = float("nan")
    score_path("plain")
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    got = obc.obc_score(qd, kd, vd, "all", seq_lens=lens)
    budget = max(1, min(lens or [N]) // 4)
    for i, name in enumerate(("value", "key", "joint")):
        err, where = score_error(got[i].cpu().numpy(), ref[i], budget, lens, TOL["fp32"])
        assert err <= TOL["fp32"], (name, err, where)       # the path's own precision, whatever the storage type
        one = obc.obc_score(qd, kd, vd, name, seq_lens=lens)
        assert torch.equal(one, got[i]), name
    run = torch.full_like(got[2], 2.0)
    obc.obc_score(qd, kd, vd, "joint", seq_lens=lens, scores=run, accumulate=True)
    for b, n in enumerate(lens or [N]):
        assert torch.equal(run[b, :, :n], got[2][b, :, :n] + 2.0) and bool((run[b, :, n:] == 2.0).all())


# (G, W, N, Hkv): static scratch holds the logits of a few heads / of a part of one head's rows / of a part of the tokens
PIECES = [(4, 32, 13001, 12), (8, 64, 40003, 1), (1, 16, 900003, 1)]


@pytest.mark.parametrize("case", PIECES, ids=["heads", "rows", "tokens"])
def test_pieces_agree_with_one_piece(case):
    G, W, N, Hkv = case
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(1, H, n, 64, generator=gen, device="cuda") for H, n in ((G * Hkv, W), (Hkv, N), (Hkv, N)))
    assert obc.obc_score_workspace_bytes(1, N, W, G * Hkv, Hkv, 64, obc.OBC_F32, obc.OBC_ALL) > obc.OBC_STATIC_SCRATCH_BYTES
    want = obc.obc_score(q, k, v, "all")
    got = torch.full_like(want, -1.0)
    obc.obc_score_static(q, k, v, "all", got)
    for i in range(3):
        err, where = score_error(got[i].cpu().numpy(), want[i].cpu().numpy().astype(np.float64), 1000, None, TOL["fp32"])
        assert err <= TOL["fp32"], (i, err, where)
