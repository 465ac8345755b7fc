"""An eviction step moves a head's rows in pieces (2048 16-byte words of K and of V, 2048 scores) whose last row comes from the
next piece: lengths around the pieces' edges, against the same step written with torch.  Bytes have to be equal."""
import pytest
import torch

from paper_2510_07651_amd import binding as obc

pytestmark = pytest.mark.gpu

# (N, true lengths): one piece, an edge with one row behind it, several pieces of scores, ragged ends on and beside an edge
SIZES = [(40, None), (128, None), (129, None), (257, [257, 129]), (1025, [1025, 1024]), (2049, None), (2113, [2113, 2048]),
         (4097, None)]


def _check_step(N, lens, G, d, Hkv, variant, where):
    B, sinks, recent = (len(lens) if lens else 1), 4, 8
    gen = torch.Generator().manual_seed(N * 8 + G)
    q = torch.randn(B, Hkv * G, 1, d, generator=gen).bfloat16().cuda()
    k = torch.randn(B, Hkv, N, d, generator=gen).bfloat16().cuda()
    v = torch.randn(B, Hkv, N, d, generator=gen).bfloat16().cuda()
    run = (torch.rand(B, Hkv, N, generator=gen) + 1).cuda()
    for b in range(B):                                       # the token to go: first, last or any of those that compete
        L = lens[b] if lens else N
        run[b, :, L:] = 0
        if where != "any":
            run[b, :, sinks if where == "low" else L - recent - 1] = -1000.
    acc = run.clone()
    obc.obc_score(q, k, v, variant, seq_lens=lens, scores=acc, accumulate=True)
    k0, v0 = k.clone(), v.clone()
    evicted = obc.obc_decode_step(q, k, v, run, variant, sinks, recent, seq_lens=lens)
    for b in range(B):
        L = lens[b] if lens else N
        for h in range(Hkv):
            e = int(evicted[b, h])
            assert float(acc[b, h, e]) == float(acc[b, h, sinks:L - recent].min())
            stay = torch.cat([torch.arange(e), torch.arange(e + 1, L)]).cuda()
            assert torch.equal(k[b, h, :L - 1], k0[b, h, stay]) and torch.equal(v[b, h, :L - 1], v0[b, h, stay])
            assert torch.equal(k[b, h, L - 1:], k0[b, h, L - 1:]) and torch.equal(v[b, h, L - 1:], v0[b, h, L - 1:])
            assert torch.equal(run[b, h, :L - 1], acc[b, h, stay]) and (run[b, h, L - 1:] == 0).all()


@pytest.mark.parametrize("N,lens", SIZES)
@pytest.mark.parametrize("G,d", [(1, 128), (4, 128), (2, 64), (7, 64)])
@pytest.mark.parametrize("where", ["low", "high", "any"])
def test_gap_is_closed_across_piece_edges(N, lens, G, d, where):
    _check_step(N, lens, G, d, 3, "joint", where)


# (N, lens, d, Hkv): ranges of four tokens per lane (more than 48 of two), ranges that a kernel of its own merges (more than 48 of
# four), and more pieces than run at once, where a workgroup looks for the token first
LONG = [(6273, None, 128, 2), (6273, [6273, 6145], 128, 1), (12417, None, 64, 2), (12673, None, 128, 1), (24833, [24833, 24577], 64, 1),
        (2049, None, 128, 32), (4097, [4097, 2049], 64, 16)]


@pytest.mark.parametrize("N,lens,d,Hkv", LONG)
@pytest.mark.parametrize("G,variant", [(1, "joint"), (2, "value"), (8, "key"), (8, "attn")])
@pytest.mark.parametrize("where", ["low", "any"])
def test_gap_is_closed_behind_long_ranges(N, lens, d, Hkv, G, variant, where):
    _check_step(N, lens, G, d, Hkv, variant, where)


@pytest.mark.parametrize("N,lens", SIZES[1:4] + SIZES[5:7])
@pytest.mark.parametrize("G,d,variant", [(1, 64, "value"), (4, 64, "attn"), (2, 128, "vatp"), (4, 128, "key")])
def test_gap_is_closed_for_every_score(N, lens, G, d, variant):
    """Scores without output sums leave V's rows alone otherwise."""
    _check_step(N, lens, G, d, 3, variant, "any")
