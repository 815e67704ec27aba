"""Distances of -0.0 are zeros: the bars are those of the same matrix with 0.0
in their place, by every path a matrix can take."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
INF = float("inf")


@pytest.mark.parametrize("columns", [False, True])
@pytest.mark.parametrize("n,side,t,max_dim,p", [(40, 3, INF, 1, 2), (60, 4, INF, 2, 2), (300, 7, 2.3, 1, 2),
                                                (300, 7, 2.3, 2, 3), (700, 12, 2.1, 2, 2), (300, 16, 3.1, 1, 3)])
def test_negative_zeros(n, side, t, max_dim, p, columns):
    import torch
    import paper_1908_02518_amd as r
    x = workloads.integer_lattice(n, 3, n, side=side)
    x[: n // 6] = x[n // 6: 2 * (n // 6)]  # duplicate points
    x[n // 2:] += (0.0003 * workloads.rng(n).standard_normal((n - n // 2, 3))).astype(np.float32)
    d = np.sqrt(((x[:, None].astype(np.float64) - x[None]) ** 2).sum(2)).astype(np.float32)
    z = np.where(d == 0.0, np.float32(-0.0), d)
    assert np.signbit(z).sum() > n
    print(f"[case] negative zeros n={n} side={side} max_dim={max_dim} p={p} columns={columns}", flush=True)
    if columns:
        r.set_sweep(0)
    a, ia = r.barcode_device(torch.from_numpy(d).cuda(), max_dim=max_dim, threshold=t, is_distance=True, p=p, cap=4 * n)
    b, ib = r.barcode_device(torch.from_numpy(z).cuda(), max_dim=max_dim, threshold=t, is_distance=True, p=p, cap=4 * n)
    same = [all(torch.equal(s, w) for s, w in zip(u, v)) for u, v in zip(a, b)]
    assert all(same), same
    for f in ("candidates", "cleared", "apparent_col", "columns", "bars_nonzero", "essential"):
        assert [s[f] for s in ia["stats"]] == [s[f] for s in ib["stats"]], f
