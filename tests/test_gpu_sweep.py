"""GPU parity of the sweep (dimensions 0 and 1 over Z/2, one workgroup per
cloud) against the oracle, bit for bit, at the sizes where its splits change:
the lanes that scan one edge's cofacets (32), the words of the nonzero-edge
bits (64), the LDS part of those bits, the survivors' sort, the threads of a
workgroup; and where its tables are full and the column reduction takes over."""

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def rips():
    import paper_1908_02518_amd as r
    return r


def two_simplices(m):
    """2m points of R^2m: two regular simplices, every point of one a little
    closer to every point of the other than to its own side: m * m edges
    without a triangle, (m - 1)^2 loops open at once."""
    a = np.eye(m) - 1.0 / m
    z = np.zeros((m, m))
    return np.vstack([np.hstack([a, z]), np.hstack([z, a])]).astype(np.float32)


def clouds(kind):
    s = workloads.SEED_BASE
    if kind == "sizes":
        return [workloads.sphere(n, s + n) for n in (1, 2, 3, 31, 32, 33, 34, 63, 64, 65, 66, 127, 128, 129, 201)]
    if kind == "ties":
        return [workloads.integer_lattice(n, 3, s + n, side=2 + n % 4) for n in (2, 5, 33, 64, 97, 130, 260)] + \
            [np.ones((7, 3), np.float32), np.zeros((1, 3), np.float32)]
    if kind == "loops":  # 23^2 loops at once: eighteen words a vector
        return [two_simplices(24), workloads.uniform_cube(90, 48, s)]
    assert kind == "full"  # 40 * 40 survivors: more than the sort of 80 points holds
    return [two_simplices(40), workloads.uniform_cube(50, 80, s)]


@pytest.mark.parametrize("max_dim", [0, 1])
@pytest.mark.parametrize("threshold", [float("inf"), 0.8])
@pytest.mark.parametrize("kind", ["sizes", "ties", "loops", "full"])
def test_batched_sweep_vs_oracle(kind, threshold, max_dim):
    import torch
    r = rips()
    cs = clouds(kind)
    print(f"[case] sweep {kind} t={threshold} max_dim={max_dim}", flush=True)
    x, off, nmax = r.pack_clouds(cs)
    bb = r.barcode_batched(x, off, nmax, max_dim=max_dim, threshold=threshold)
    torch.cuda.synchronize()
    for b, c in enumerate(cs):
        ref = oracle.barcode(c, max_dim=max_dim, threshold=threshold, p=2)
        for d in range(max_dim + 1):
            got = [t.cpu().numpy() for t in bb.segment(b, d)]
            want = (ref.bars[d].birth, ref.bars[d].death, ref.bars[d].birth_simplex, ref.bars[d].death_simplex)
            for g, w in zip(got, want):
                assert np.array_equal(g, w), (kind, b, d)
        assert float(bb.thresholds[b]) == ref.threshold


@pytest.mark.parametrize("n", [608, 700])
def test_batched_sweep_vs_column_reduction(n):
    """Sizes on both sides of the LDS part of the nonzero-edge bits, against
    the column reduction with the general working column."""
    import torch
    r = rips()
    cs = [workloads.noisy_circle_with_outliers(workloads.SEED_BASE + n, n - 40, 40), workloads.uniform_cube(60, 2, n)]
    x, off, nmax = r.pack_clouds(cs)
    print(f"[case] sweep vs column reduction n={n}", flush=True)
    one = r.barcode_batched(x, off, nmax, max_dim=1, threshold=0.7)
    r.set_working_column(r.WORKING_COLUMN_GENERAL)
    try:
        two = r.barcode_batched(x, off, nmax, max_dim=1, threshold=0.7)
    finally:
        r.set_working_column()
    torch.cuda.synchronize()
    k = int(one.offsets[-1])
    assert torch.equal(one.offsets, two.offsets)
    for a, b in ((one.birth, two.birth), (one.death, two.death), (one.birth_simplex, two.birth_simplex),
                 (one.death_simplex, two.death_simplex)):
        assert torch.equal(a[:k], b[:k])
    for f in ("candidates", "cleared", "apparent_col", "apparent_pivot", "columns", "bars_nonzero", "essential"):
        q = r.STAT_FIELDS.index(f)
        assert torch.equal(one.stats[:, :, q], two.stats[:, :, q]), f
