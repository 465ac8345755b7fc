"""The general scoring path on inputs whose elements span many binades, against the oracle.

A logit is a sum of products; nothing may be lost of it that its terms hold, whatever else the rows contain.  The same
goes for the squared distance of a value from a row's output, also where most of both is common to them.
"""
import pytest
import torch

import oracle
from paper_2510_07651_amd import binding as obc

from parity_util import TOL, score_error

pytestmark = pytest.mark.gpu

# (dtype, d, G, W, N): rows G*W on either side of 32, the last one in two chunks of rows
SHAPES = [("fp32", 128, 1, 32, 700), ("fp32", 128, 3, 11, 700), ("fp32", 64, 4, 32, 1500), ("bf16", 64, 4, 32, 1500),
          ("bf16", 64, 5, 40, 333)]
IDS = ["%s_d%d_%dx%d_%d" % s for s in SHAPES]
HKV = 2


def _random(shape, seed):
    dtype, d, G, W, N = shape
    gen = torch.Generator().manual_seed(seed)
    return [torch.randn(1, H, n, d, generator=gen) for H, n in ((G * HKV, W), (HKV, N), (HKV, N))]


def _check(shape, q, k, v, tol=TOL["fp32"]):
    dt = torch.float32 if shape[0] == "fp32" else torch.bfloat16
    q, k, v = (x.to(dt) for x in (q, k, v))
    ref = oracle.score(q, k, v)
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), "all").cpu().numpy()
    errors = []
    for i, name in enumerate(("value", "key", "joint")):
        err, where = score_error(got[i], ref[i], shape[4] // 8, None, tol)
        errors.append((name, err, where))
    print(errors)
    assert all(err <= tol for _, err, _ in errors), errors


@pytest.mark.parametrize("binades", [12, 26])
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_large_key_channel_meets_small_query_channel(shape, binades):
    """Two channels whose keys are 2^binades larger and queries as much smaller: their products are of the others' size, so
    the logits are ordinary, but a row's largest element says nothing about them."""
    q, k, v = _random(shape, 71)
    k[..., 3:5] *= 2.0 ** binades
    q[..., 3:5] *= 2.0 ** -binades
    _check(shape, q, k, v)


# How the values of a head resemble each other, and with them the outputs.  Distances stay above 2^-6 of the norm: an output
# is a sum in fp32 (some 4 roundings of 2^-24), which moves a squared distance by 2 * 4 * 2^-24 / (2^-6 sqrt(d)), 4e-6.
VALUES = {
    # one channel is the same for all: the distance lies in the others
    "common_channel_2^8": lambda v: _set_channel(v, 2.0 ** 8),
    "common_channel_2^14": lambda v: _set_channel(v, 2.0 ** 14),
    "common_channel_2^16": lambda v: _set_channel(v, 2.0 ** 16),
    # nearly the same row everywhere
    "nearly_repeated": lambda v: v[:, :, :1] + v * 2.0 ** -4,
    # the same row exactly, but for every eighth token
    "repeated": lambda v: torch.where((torch.arange(v.shape[2]) % 8 == 5)[:, None], v, v[:, :, :1]),
    # a common part of two and three times the rest
    "common_part_2": lambda v: v + 2 * v[:, :, :1],
    "common_part_3": lambda v: v + 3 * v[:, :, :1],
    # multiples of one row: (1 + Z) v cancels Z o for some pairs
    "parallel": lambda v: v[:, :, :1] * (1 + v[..., :1]) + v * 2.0 ** -4,
}


def _set_channel(v, x):
    v = v.clone()
    v[..., 7] = x
    return v


@pytest.mark.parametrize("values", VALUES)
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_values_close_to_the_outputs(shape, values):
    q, k, v = _random(shape, 72)
    _check(shape, q, k, VALUES[values](v))


# Outputs of about the values' norm, distances between 1/16 and 1/4 of its square.
COMMON = {
    "channel": lambda v: _set_channel(v, 2.75 * v.shape[-1] ** 0.5),
    "part": lambda v: v + 2.75 * v[:, :, :1],
}


@pytest.mark.parametrize("common", COMMON)
@pytest.mark.parametrize("shape", SHAPES + [("bf16", 64, 1, 20, 1500), ("fp32", 64, 4, 8, 5000), ("fp32", 128, 4, 32, 2100)],
                         ids=IDS + ["bf16_d64_1x20_1500", "fp32_d64_4x8_5000", "fp32_d128_4x32_2100"])
def test_squared_distances_element_by_element(shape, common):
    """Every row asks the same, so key over value score of a token is Z^2 ||v_p - o||^2 / ||v_p||^2: the weights, whose errors are
    as large as those looked for, cancel.  Left are, in roundings of 2^-24 at most: Z twice (1), three products (3), the distance
    (1) and the norm (1), their products' sums over a row block and the blocks, key and value (2 * 5), and what the fp32
    outputs move a distance by: 2 (v - o) . do / ||v - o||^2 with do of some 2 roundings of ||o|| <= 2.75 ||v - o|| and a cosine of
    5 / sqrt(d) among thousands of tokens (7).  The cross term itself has to add nothing."""
    dtype, d, G, W, N = shape
    q, k, v = _random(shape, 77)
    q = q[:, ::G, :1].repeat_interleave(G, 1).expand(-1, -1, W, -1).contiguous() * 0.5
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    q, k, v = (x.to(dt) for x in (q, k, COMMON[common](v)))
    sv, sk, _ = (torch.from_numpy(x) for x in oracle.score(q, k, v))
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), "all").cpu().double()
    z = (q[:, ::G, :1].double() @ k.double().transpose(2, 3))[:, :, 0] / d ** 0.5
    seen = (torch.arange(N) <= N - W) & (z.abs() > 2.0 ** -10) & (z < z.amax(2, keepdim=True))     # (the top token is scored apart)
    err = ((got[1] / got[0]) / (sk / sv) - 1).abs()[seen]
    print(float(err.max()), float(err.square().mean().sqrt()))
    assert float(err.max()) <= 23 * 2.0 ** -24


@pytest.mark.parametrize("shape", SHAPES + [("fp32", 64, 1, 4, 3000)], ids=IDS + ["fp32_d64_1x4_3000"])
def test_logits_at_the_end_of_fp32_have_weight_zero(shape):
    """One key's logit is -3.1e38, another's overflows to -infinity: both have weight 0, and nothing else changes."""
    q, k, v = _random(shape, 73)
    dt = torch.float32 if shape[0] == "fp32" else torch.bfloat16
    q[..., 0], k[..., 0] = 2.0 ** 63, 0.0
    k[:, :, 5, 0] = -3.1e38 * shape[1] ** 0.5 / 2.0 ** 63
    k[:, :, 11, 0] = -1e39 * shape[1] ** 0.5 / 2.0 ** 63
    q, k, v = (x.to(dt) for x in (q, k, v))
    want = {"value": oracle.score(q, k, v)[0], "attn": oracle.attn_score(q, k, v), "vatp": oracle.vatp_score(q, k, v)}
    for variant, ref in want.items():
        got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), variant).cpu().numpy()
        assert (got[:, :, [5, 11]] == 0).all(), variant
        err, where = score_error(got, ref, shape[4] // 8, None, TOL["fp32"])
        assert err <= TOL["fp32"], (variant, err, where)


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_a_value_that_is_not_a_number_shows(shape):
    """It is part of every row's output, and with that of every key and joint score of its head; other heads are left alone."""
    q, k, v = _random(shape, 74)
    dt = torch.float32 if shape[0] == "fp32" else torch.bfloat16
    v[:, 1, 17, 3] = float("nan")
    for variant in ("key", "joint"):
        got = obc.obc_score(*(x.to(dt).cuda() for x in (q, k, v)), variant)
        assert bool(got[:, 1].isnan().all()) and bool(got[:, 0].isfinite().all()), variant


# What the digits of a logit cannot hold, or hold only in part.
LOGITS = {
    # the query's large element meets the keys' small one, and the other way round: the digits' error next to the logit's size
    "apart_2^7": lambda q, k: _apart(q, k, 7),
    "apart_2^12": lambda q, k: _apart(q, k, 12),
    "apart_2^20": lambda q, k: _apart(q, k, 20),
    "channels_2^12": lambda q, k: (_scaled(q, slice(3, 5), -12), _scaled(k, slice(3, 5), 12)),
    "channels_2^26": lambda q, k: (_scaled(q, slice(3, 5), -26), _scaled(k, slice(3, 5), 26)),
    # elements far below their rows' largest, in every 16th key and one query row
    "small_elements": lambda q, k: (_put(q, slice(3, 4), 2.0 ** -29), _put(k, slice(5, None, 16), 2.0 ** -27)),
    # keys that are zero, here and there and in every block; queries that are; keys at a right angle to every query
    "zero_keys": lambda q, k: (q, _put(k, slice(9, None, 50), 0.0, slice(None))),
    "zero_key_per_block": lambda q, k: (q, _put(k, slice(5, None, 16), -0.0, slice(None))),
    "zero_queries": lambda q, k: (_put(q, slice(2, None, 5), 0.0, slice(None)), k),
    "right_angles": lambda q, k: (_put(q, slice(None), 0.0, slice(0, 32)), _put(k, slice(2, None, 7), 0.0, slice(32, None))),
}


def _put(x, rows, value, channels=slice(1, 4)):
    x = x.clone()
    x[:, :, rows, channels] = value
    return x


def _scaled(x, channels, binades):
    x = x.clone()
    x[..., channels] *= 2.0 ** binades
    return x


def _apart(q, k, binades):
    return _scaled(q, slice(0, 1), binades), _scaled(k, slice(0, 1), -binades)


# Sequences of many splits and of few, with rows in one chunk and in several; the last one is too short for digits.
DIGIT_SHAPES = [("fp32", 128, 3, 43, 12301), ("fp32", 64, 1, 64, 40991), ("fp32", 128, 3, 43, 8131), ("fp32", 64, 1, 64, 16332),
                ("bf16", 64, 5, 40, 12303), ("bf16", 64, 1, 33, 24595), ("bf16", 64, 5, 40, 8145), ("bf16", 64, 1, 33, 16321),
                ("bf16", 128, 1, 40, 24597), ("bf16", 128, 1, 40, 16323), ("fp32", 128, 3, 43, 129)]


@pytest.mark.parametrize("logits", LOGITS)
@pytest.mark.parametrize("shape", DIGIT_SHAPES, ids=lambda s: "%s_d%d_%dx%d_%d" % s)
def test_logits_beyond_their_digits(shape, logits, score_path):
    score_path("plain")
    q, k, v = _random(shape, 75)
    q, k = LOGITS[logits](q, k)
    _check(shape, q, k, v)


@pytest.mark.parametrize("big", ["query", "key", "half"])
@pytest.mark.parametrize("shape", DIGIT_SHAPES[:4], ids=lambda s: "%s_d%d_%dx%d_%d" % s)
def test_rows_that_the_digits_cut(shape, big):
    """Rows with elements half a unit of their digits above a whole one, all of them where the other side has its large ones:
    the dot products stand out above 2^-17 2^E and what is cut off is 2^-23.3 of them, three roundings to fp32.  Logits of
    some 2^12 make that 2^-11 in a weight, next to those of 16 keys whose rows are held.  Against weights of exact dot
    products rounded once, which is what the logits are defined as."""
    _, d, G, W, N = shape
    below_one, tiny = 1 - 2.0 ** -24, 2.0 ** -24 * (1.25 + 2.0 ** -23)
    n = {"query": 1, "half": d // 2, "key": d - 1}[big]      # elements of the key that are large
    key, query = torch.full((d,), tiny), torch.full((d,), tiny)
    key[:n], query[n:] = below_one, below_one
    held = torch.zeros(d)
    held[n:] = float(key.double() @ query.double()) / (d - n)
    query *= 2.0 ** 32
    k = key.repeat(1, HKV, N, 1)
    k[:, :, :16] = held
    q, v = query.repeat(1, G * HKV, W, 1), _random(shape, 76)[2]
    z64 = (torch.stack((held, key)).double() @ query.double()) / d ** 0.5
    z = z64.float()
    ulp = 2.0 ** (torch.frexp(z)[1] - 24).double()
    assert bool((((z64 - z.double()).abs() / ulp) < 0.49).all()) and 2.0 ** 11 < float(z.min())     # no matter of rounding
    row = torch.full((N,), float(z[1]), dtype=torch.float64)
    row[:16] = float(z[0])
    want = sum(G * torch.nn.functional.pad(torch.softmax(row[:N - W + 1 + r], 0), (0, W - 1 - r)) for r in range(W))
    got = obc.obc_score(q.cuda(), k.cuda(), v.cuda(), "attn").cpu().double()
    err = float(((got - want) / want).abs().max())
    print(err)
    assert err <= TOL["fp32"], err


@pytest.mark.parametrize("shape", DIGIT_SHAPES[:8], ids=lambda s: "%s_d%d_%dx%d_%d" % s)
def test_digit_logits_at_the_end_of_fp32(shape):
    test_logits_at_the_end_of_fp32_have_weight_zero(shape)
