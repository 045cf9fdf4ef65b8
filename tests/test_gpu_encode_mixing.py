"""GPU test of fp32 encode where S passes little of a coordinate on to a pair: just above and just below the 2^-16 from which on
two binary16 terms per number are taken, with vectors of one large coordinate and 127 so small that their second terms are cut."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_02617_amd import Context, PQ_KEY, PQ_VALUE
from tests.test_gpu_parity import check_encode, say

pytestmark = pytest.mark.gpu
ROW, PAIR = 37, 20


def weak_pair(entry):
    """An orthogonal matrix whose row ROW has `entry` and its half in pair PAIR: two columns are turned against others."""
    S = np.linalg.qr(np.random.default_rng(11).standard_normal((128, 128)))[0]
    for column, other, want in ((2 * PAIR, 3, entry), (2 * PAIR + 1, 5, 0.5 * entry)):
        a, b = S[ROW, column], S[ROW, other]
        t = np.arctan2(b, a) + np.arccos(want / np.hypot(a, b))
        c, s = np.cos(t), np.sin(t)
        S[:, [column, other]] = S[:, [column, other]] @ np.array([[c, -s], [s, c]])
    assert np.abs(S.T @ S - np.eye(128)).max() < 1e-14 and abs(S[ROW, 2 * PAIR] / entry - 1.0) < 1e-9
    return S


@pytest.mark.parametrize("entry", [2.0 ** -15.9, 2.0 ** -16.1])
@pytest.mark.parametrize("small", [-17, -22])
def test_a_pair_that_sees_little_of_the_largest_coordinate(entry, small):
    say(f"fp32 encode, smallest pair {entry:.2e}, other coordinates 2^{small}")
    S = weak_pair(entry)
    g = torch.Generator().manual_seed(13)
    x = torch.randn((3000, 1, 128), generator=g) * 2.0 ** small
    x[:, :, ROW] = 1.0 + torch.rand((3000, 1), generator=g)
    x *= torch.exp2(torch.randint(0, 13, (3000, 1, 1), generator=g).float())
    cb = oracle.default_codebooks()
    for kind in (PQ_KEY, PQ_VALUE):
        check_encode(Context(S=S), S, cb, x, kind, "one large coordinate")
