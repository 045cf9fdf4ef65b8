"""pq_fit_cluster (host code) where a k-means cell holds a sliver of one bin, or nothing, next to large counts."""
import math

import numpy as np
import pytest

from paper_2502_02617_amd import Context

BINS1, BINSU = 8192, 2048


def edges(bins, quarter_turns):
    per = bins // quarter_turns
    return [(k // per) * (math.pi / 2) + math.atan2(k % per, per - k % per) for k in range(bins + 1)]


EDGES = {BINS1: edges(BINS1, 4), BINSU: edges(BINSU, 1)}


def one_round(hist, c):
    """Bin by bin: the part of every bin that falls into a cell, centred on that part; sums exactly rounded."""
    e = EDGES[len(hist)]
    cut = [-math.inf] + [0.5 * (a + b) for a, b in zip(c, c[1:])] + [math.inf]
    mass, moment, q = [[] for _ in c], [[] for _ in c], 0
    for b in np.nonzero(hist)[0]:
        while cut[q + 1] <= e[b]:
            q += 1
        k = q
        while k < len(c) and cut[k] < e[b + 1]:
            lo, hi = max(e[b], cut[k]), min(e[b + 1], cut[k + 1])
            m = int(hist[b]) * ((hi - lo) / (e[b + 1] - e[b]))
            mass[k].append(m)
            moment[k].append(m * (0.5 * (lo + hi)))
            k += 1
    return [math.fsum(s) / math.fsum(m) if m else old for m, s, old in zip(mass, moment, c)]


def built_in():
    return np.concatenate([Context(seed=0).codebook(l)[0] for l in (1, 2, 3, 4)])


def check(hists, start=None):
    full = np.concatenate(list(hists) + [np.zeros(3 * BINSU, dtype=np.int64)]).astype(np.uint32)
    got = np.asarray(Context(seed=0).fit_cluster(full, 1, cb_init=start)[0]).ravel()
    start = built_in() if start is None else start
    for l, at in enumerate((slice(0, 16), slice(16, 20), slice(20, 24), slice(24, 28))):
        # a dozen roundings of numbers up to 2 pi, 4.4e-16 each at most
        assert np.max(np.abs(got[at] - one_round(hists[l], list(start[at])))) <= 1e-14, l + 1
        assert np.all(np.diff(got[at]) > 0), l + 1


@pytest.mark.parametrize("count", [1, 50, 3000])
@pytest.mark.parametrize("half", ["lower", "upper"])
def test_half_empty_levels_from_the_built_in_start(half, count):
    """The middle boundary of the built-in codebooks is a bin edge to within an ulp."""
    at1, at = np.arange(BINS1) < BINS1 // 2, np.arange(BINSU) < BINSU // 2
    if half == "upper":
        at1, at = ~at1, ~at
    check([at1 * count] + [at * count] * 3)


@pytest.mark.parametrize("empty", [0, 3, 9, 15])
@pytest.mark.parametrize("shift", [sign * 10.0 ** -k for k in range(10, 17) for sign in (1, -1)])
def test_an_empty_cell_whose_boundary_is_next_to_a_bin_edge(shift, empty):
    start = built_in()
    start[:16] += shift
    h1 = np.full(BINS1, 1234567)
    h1[empty * 512:(empty + 1) * 512] = 0
    check([h1] + [np.full(BINSU, 7)] * 3, start)


@pytest.mark.parametrize("part", [1e-9, 1e-7, 1e-4, 0.3])
@pytest.mark.parametrize("at", [1000, 4095, 5000, 8000])
def test_a_sliver_of_one_count_next_to_large_counts(at, part):
    """1.2e9 counts in 400 bins below, and a bin of one count whose last `part` alone falls into the cell above."""
    e = EDGES[BINS1]
    h1 = np.zeros(BINS1, dtype=np.int64)
    rng = np.random.default_rng(6)
    h1[rng.choice(at - 500, 400, replace=False)] = rng.integers(1000000, 5000000, size=400)
    h1[at] = 1
    cut = e[at + 1] - part * (e[at + 1] - e[at])
    start = np.concatenate([np.linspace(0.05, cut - 0.1, 14), [cut - 0.03125, cut + 0.03125], built_in()[16:]])
    check([h1] + [np.full(BINSU, 7)] * 3, start)


def test_cells_inside_one_bin_and_counts_of_32_bits():
    e = EDGES[BINS1]
    h1 = np.full(BINS1, 0xFFFFFFFF)
    step = (e[3001] - e[3000]) / 40
    start = np.concatenate([e[3000] + step * (2 + 2 * np.arange(16)), built_in()[16:]])
    check([h1] + [np.full(BINSU, 0xFFFFFFFF)] * 3, start)
