"""The general scoring path on inputs whose elements span many binades, against the oracle.

A logit is a sum of products; nothing may be lost of it that its terms hold, whatever else the rows contain.
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
