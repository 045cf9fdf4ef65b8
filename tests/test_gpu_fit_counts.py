"""GPU test of the angle counts of vectors so small that the squares of their coordinates are subnormal numbers."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2502_02617_amd import Context, _build
from tests.test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu


def counts(ctx, x):
    ws = torch.empty(Context.fit_workspace_bytes(), dtype=torch.uint8, device=DEV)
    ctx.fit_count_angles(x.to(DEV), ws)
    torch.cuda.synchronize()
    return ws.view(torch.int32).cpu().long()


@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_counts_do_not_depend_on_the_scale_of_the_vectors(dtype, depth):
    say(f"angle counts of small vectors, {dtype}, depth {depth}")
    ctx = Context(S=np.eye(128))
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    x = torch.randn((3001, 2, 128), generator=torch.Generator().manual_seed(3)).to(dtype)
    ref = counts(ctx, x)
    assert torch.equal(counts(ctx, x * 2.0 ** -40), ref)       # all squares are normal numbers: the same operations
    small = counts(ctx, x * 2.0 ** -63)
    assert small.sum() == ref.sum()
    # A square of z 2^-63 keeps z^2 2^23 units: an angle is off by about 1e-7 / z^2, a bin 5e-4 to 1e-3 wide, so fewer than
    # one node in a hundred changes its bin (it leaves one and enters another).
    assert (small - ref).abs().sum() <= 0.02 * ref.sum()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_counts_of_pieces_add_up(dtype):
    say(f"angle counts of a long input and of its pieces, {dtype}")
    ctx, n = Context(seed=4), 12800                # 8 heads: 1600 tiles; the pieces take 8 to 1056 of them
    x = torch.randn((n, 8, 128), generator=torch.Generator().manual_seed(6)).to(dtype)
    x[5], x[6], x[7, 0, :16], x[8] = 0.0, 1e30, 0.0, 1e-25     # zeros and squares outside the range of the short roots
    whole, at = counts(ctx, x), 0
    assert whole.sum() == 8 * n * 120              # four levels of 64 + 32 + 16 + 8 angles
    total = torch.zeros_like(whole)
    for piece in (1, 63, 4000, 300, n - 4364):
        total += counts(ctx, x[at:at + piece])
        at += piece
    assert at == n and torch.equal(total, whole)


def test_short_roots_are_the_rounded_ones():
    say("the short square root against sqrtf, all numbers of its range")
    path = _build.ROOTCHECK_PATH if os.path.exists(_build.ROOTCHECK_PATH) else _build.build_rootcheck()
    res = subprocess.run([path], capture_output=True, text=True, timeout=60)
    print(res.stdout, res.stderr)
    assert res.returncode == 0
    assert f"compared {201 * 2 ** 23 + 1} numbers, 0 different" in res.stdout


@pytest.mark.parametrize("scale", [2.0 ** -52, 2.0 ** 50])
@pytest.mark.parametrize("depth", [4, 7])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_both_kinds_of_roots_count_the_same(dtype, depth, scale):
    """Squares around 1 take the short root, those around 2^-104 and 2^100 sqrtf; every operation scales exactly."""
    say(f"angle counts with either root, {dtype}, depth {depth}, vectors times {scale:.1e}")
    ctx = Context(seed=4)
    if depth == 7:
        ctx.set_recursion_depth(7, (2, 2, 2))
    x = torch.randn((6001, 8, 128), generator=torch.Generator().manual_seed(7)).to(dtype)
    assert torch.equal(counts(ctx, x), counts(ctx, x * scale))
