"""GPU parity of the sweep of one cloud with the column reduction, bit for bit:
the whole cloud by one workgroup (small clouds, and any without a threshold),
dimension 1 in chunks (larger ones of 32 to 200 edges a point) and dimension 2
by blocks of one longest edge, on both sides of each rule, from points and from
a distance matrix; and where a table is full, a distance overflows or edges of
equal length meet and the other path takes over."""

import itertools

import numpy as np
import pytest

import oracle
import workloads
from tests.test_gpu_sweep import two_simplices

pytestmark = pytest.mark.gpu
INF = float("inf")


def rips():
    import paper_1908_02518_amd as r
    return r


def bars(x, **kw):
    import torch
    r = rips()
    out, info = r.barcode_device(x, **kw)
    torch.cuda.synchronize()
    return [[t.cpu().numpy() for t in b] for b in out], info


def both(x, **kw):
    """Bars by the default method and by the reduction of columns."""
    r = rips()
    r.set_working_column()
    one, i1 = bars(x, **kw)
    r.set_reduce_workgroups(0)
    try:
        two, i2 = bars(x, **kw)
    finally:
        r.set_working_column()
    for d, (a, b) in enumerate(zip(one, two)):
        for u, v in zip(a, b):
            assert np.array_equal(u, v), d
    for f in ("threshold", "sparse", "simplex_count"):
        assert i1[f] == i2[f], f
    for f in ("candidates", "cleared", "apparent_col", "apparent_pivot", "columns", "bars_nonzero", "essential"):
        assert [s[f] for s in i1["stats"]] == [s[f] for s in i2["stats"]], f
    return one


def degree_threshold(x, degree):
    d = np.sqrt(((x[::7, None, :].astype(np.float64) - x[None, :, :]) ** 2).sum(2)).ravel()
    return float(np.float32(np.partition(d, int(degree / len(x) * d.size))[int(degree / len(x) * d.size)]))


@pytest.mark.parametrize("max_dim", [0, 1])
@pytest.mark.parametrize("matrix", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 31, 33, 64, 65, 129, 255, 256, 257, 300])
def test_whole_cloud_vs_column_reduction(n, matrix, max_dim):
    import torch
    x = workloads.sphere(n, workloads.SEED_BASE + n)
    if matrix:
        x = np.sqrt(((x[:, None] - x[None]) ** 2).sum(2, dtype=np.float32))
        x = np.ascontiguousarray(np.tril(x) + np.triu(np.full_like(x, 7.0)))  # the part above is not read
    for t in (INF, 0.9, 0.0):
        print(f"[case] whole cloud n={n} matrix={matrix} t={t} max_dim={max_dim}", flush=True)
        both(torch.from_numpy(x).cuda(), max_dim=max_dim, threshold=t, is_distance=matrix)


@pytest.mark.parametrize("p", [3, 5, 65521])
@pytest.mark.parametrize("n", [2, 33, 65, 127, 128, 129, 200, 201])
def test_whole_cloud_over_another_field(n, p):
    import torch
    s = workloads.SEED_BASE + n
    for x in (workloads.sphere(n, s), workloads.integer_lattice(n, 3, s, side=5),
              workloads.noisy_circle_with_outliers(s, n - n // 8, n // 8), workloads.uniform_cube(n, 6, s)):
        for t in (INF, 0.7):
            print(f"[case] whole cloud n={n} p={p} m={x.shape[1]} t={t}", flush=True)
            both(torch.from_numpy(x).cuda(), max_dim=1, threshold=t, p=p)


def test_whole_cloud_torsion():
    """A projective plane: one bar more over Z/2 than over Z/3."""
    import torch
    r = rips()
    x = np.float32(projective_plane())
    d = torch.from_numpy(x).cuda()
    n1 = {}
    for p in (2, 3):
        n1[p] = len(both(d, max_dim=1, threshold=1.5, p=p, is_distance=True)[1][0])
    assert n1[2] == n1[3] + 1


def projective_plane():
    """Distances whose complex at 1 is the barycentric subdivision of the
    6-vertex projective plane (31 points)."""
    tris = [(0, 1, 4), (0, 1, 5), (0, 2, 3), (0, 2, 5), (0, 3, 4), (1, 2, 3), (1, 2, 4), (1, 3, 5), (2, 4, 5), (3, 4, 5)]
    faces = sorted({f for t in tris for k in (1, 2, 3) for f in itertools.combinations(t, k)})
    x = np.full((len(faces), len(faces)), 2.0)
    for i, f in enumerate(faces):
        for j, g in enumerate(faces):
            if set(f) <= set(g) or set(g) <= set(f):
                x[i, j] = 0.0 if i == j else 1.0
    return x


@pytest.mark.parametrize("kind", ["ties", "loops", "full", "overflow"])
def test_whole_cloud_special_inputs(kind):
    import torch
    r = rips()
    r.set_working_column()
    s = workloads.SEED_BASE
    x = {"ties": lambda: workloads.integer_lattice(130, 3, s, side=3), "loops": lambda: two_simplices(24),
         "full": lambda: two_simplices(40),
         "overflow": lambda: workloads.sphere(40, s) * np.float32(3e38)}[kind]()
    print(f"[case] whole cloud {kind}", flush=True)
    if kind == "overflow":  # finite points, some distances are not
        both(torch.from_numpy(x).cuda(), max_dim=1, threshold=2e38)
        return
    ref = oracle.barcode(x, max_dim=1, threshold=INF, p=2)
    got, info = bars(torch.from_numpy(x).cuda(), max_dim=1)
    for d in range(2):
        want = (ref.bars[d].birth, ref.bars[d].death, ref.bars[d].birth_simplex, ref.bars[d].death_simplex)
        for g, w in zip(got[d], want):
            assert np.array_equal(g, w)
    host = r.barcode(x, max_dim=1)  # through host memory
    for d in range(2):
        assert np.array_equal(host.bars[d].birth, ref.bars[d].birth)
        assert np.array_equal(host.bars[d].death_simplex, ref.bars[d].death_simplex)


def test_not_finite_is_refused():
    import torch
    r = rips()
    r.set_working_column()
    for bad in (float("nan"), INF):
        for n in (1, 2, 40):
            x = torch.from_numpy(workloads.sphere(n, 5)).cuda()
            x[n - 1, 1] = bad
            with pytest.raises(r.RipsError):
                r.barcode_device(x, max_dim=1)


@pytest.mark.parametrize("n,degree", [(260, 31), (260, 33), (700, 64), (700, 199), (700, 201), (3000, 40), (24000, 36)])
@pytest.mark.parametrize("data", ["torus", "lattice"])
def test_chunked_sweep_vs_column_reduction(data, n, degree):
    """24,000 points: places by hashing (more than 2^28 possible edges)."""
    import torch
    if n == 24000 and data == "lattice":
        pytest.skip("one large cloud is enough")
    s = workloads.SEED_BASE + n
    x = workloads.clifford_torus(n, 0.02, s) if data == "torus" else workloads.integer_lattice(n, 4, s, side=9)
    t = degree_threshold(x, degree) if n < 24000 else 0.138
    print(f"[case] chunked sweep {data} n={n} degree={degree} t={t}", flush=True)
    both(torch.from_numpy(x).cuda(), max_dim=1, threshold=t)


@pytest.mark.parametrize("p", [3, 65521])
@pytest.mark.parametrize("data,n,t,max_dim", [("torus", 1200, 0.5, 2), ("so3", 900, 1.4, 1), ("sphere", 500, 0.8, 1),
                                              ("circle", 600, 0.25, 2), ("lattice", 700, 2.3, 1)])
def test_chunked_sweep_over_another_field(data, n, t, max_dim, p):
    import torch
    s = workloads.SEED_BASE + n
    x = {"torus": lambda: workloads.clifford_torus(n, 0.02, s), "so3": lambda: workloads.so3(n, s),
         "sphere": lambda: workloads.sphere(n, s),
         "circle": lambda: workloads.noisy_circle_with_outliers(s, n - 60, 60),
         "lattice": lambda: workloads.integer_lattice(n, 4, s, side=9)}[data]()
    print(f"[case] chunked sweep {data} n={n} t={t} p={p}", flush=True)
    both(torch.from_numpy(x).cuda(), max_dim=max_dim, threshold=t, p=p)


def octahedra(k, seed):
    """k crosses of R^3 side by side, points slightly moved: k voids."""
    g = workloads.rng(seed)
    a = np.concatenate([np.eye(3), -np.eye(3)])
    x = np.concatenate([a + [5.0 * i, 0.0, 0.0] for i in range(k)]) + 0.02 * g.standard_normal((6 * k, 3))
    return x.astype(np.float32)


@pytest.mark.parametrize("p", [2, 3, 65521])
@pytest.mark.parametrize("kind", ["sphere-5", "sphere-46", "sphere-64", "sphere-65", "sphere-129", "cube-70", "so3-300",
                                  "so3-700", "o3-300", "o3-600", "mixture-90", "voids-1500", "lattice-60", "line-60",
                                  "torus-1500"])
def test_dimension_2_by_blocks_vs_column_reduction(kind, p):
    import torch
    name, n = kind.split("-")
    n = int(n)
    s = workloads.SEED_BASE + n
    x, t, max_dim = {
        "sphere": lambda: (workloads.sphere(n, s), INF, 2),
        "cube": lambda: (workloads.uniform_cube(n, 5, s), INF, 2),      # trees joined late, many classes
        "so3": lambda: (workloads.so3(n, s), 1.4, 2),
        "o3": lambda: (workloads.orthogonal(n, s), 1.8, 3),             # a dimension follows: pivots handed on
        "mixture": lambda: (workloads.mixture_cloud(s, n, n), INF, 2),
        "voids": lambda: (octahedra(n, s), 2.1, 3),
        "lattice": lambda: (workloads.integer_lattice(n, 3, s), INF, 2),  # ties everywhere: columns
        "line": lambda: (workloads.uniform_cube(n, 1, s), INF, 2),      # no class at all
        "torus": lambda: (workloads.clifford_torus(n, 0.02, s), 0.55, 2),
    }[name]()
    print(f"[case] dimension 2 {kind} p={p}", flush=True)
    both(torch.from_numpy(x).cuda(), max_dim=max_dim, threshold=t, p=p)


@pytest.mark.parametrize("digits", [2, 3, 4, 5])
@pytest.mark.parametrize("data", ["o3", "sphere"])
def test_dimension_2_some_ties(data, digits):
    """Distances rounded so that a few, or many, edges of equal length share
    simplices, with a dimension that follows and without."""
    import torch
    s = workloads.SEED_BASE + digits
    for seed in (s, s + 100, s + 200):
        x = workloads.orthogonal(520, seed) if data == "o3" else workloads.sphere(52, seed)
        d = np.sqrt(((x[:, None].astype(np.float64) - x[None]) ** 2).sum(2)).round(digits).astype(np.float32)
        d = torch.from_numpy(np.ascontiguousarray(d)).cuda()
        for max_dim, p in ((2, 2), (3, 2), (2, 3)):
            print(f"[case] dimension 2 some ties {data} digits={digits} max_dim={max_dim} p={p}", flush=True)
            both(d, max_dim=max_dim, threshold=1.8 if data == "o3" else INF, is_distance=True, p=p)


def test_dimension_2_large_lune():
    """A lune of more points than one block's forest holds: columns."""
    import torch
    g = workloads.rng(workloads.SEED_BASE)
    x = (0.01 * g.standard_normal((1100, 3))).astype(np.float32)
    x[:2] = [[-1, 0, 0], [1, 0, 0]]
    d = np.sqrt(((x[:, None] - x[None]) ** 2).sum(2, dtype=np.float32))
    far = (d > 0.004) & (d < 0.9)  # the middle's own edges are too long but for a few
    d[far] = 3.0
    print("[case] dimension 2 large lune", flush=True)
    both(torch.from_numpy(np.ascontiguousarray(d)).cuda(), max_dim=2, threshold=2.5, is_distance=True)


@pytest.mark.parametrize("n", [2048, 2049, 3001])
@pytest.mark.parametrize("data", ["torus", "lattice"])
def test_dimension_0_on_both_sides_of_the_wide_boruvka(data, n):
    """Many components at the threshold; the lattice: equal lengths and duplicate points."""
    import torch
    s = workloads.SEED_BASE + n
    x = workloads.clifford_torus(n, 0.02, s) if data == "torus" else workloads.integer_lattice(n, 3, s, side=17)
    t = 0.08 if data == "torus" else 1.0
    print(f"[case] dimension 0 {data} n={n}", flush=True)
    ref = oracle.barcode(x, max_dim=0, threshold=t, p=2)
    got, _ = bars(torch.from_numpy(x).cuda(), max_dim=0, threshold=t)
    want = (ref.bars[0].birth, ref.bars[0].death, ref.bars[0].birth_simplex, ref.bars[0].death_simplex)
    for g, w in zip(got[0], want):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("kind", ["sphere-70", "sphere-150", "sphere-65", "lattice-150"])
def test_columns_sorted_by_the_whole_chip(kind):
    """Without the apparent pairs every edge off the forest is a column: 2016
    (below the rule), 2346 and 11,026, and thousands of one length, which are
    left to one workgroup."""
    r = rips()
    name, n = kind.split("-")
    s = workloads.SEED_BASE + int(n)
    x = workloads.sphere(int(n), s) if name == "sphere" else workloads.integer_lattice(int(n), 2, s, side=2)
    print(f"[case] wide sort {kind}", flush=True)
    ref = oracle.barcode(x, max_dim=1, threshold=INF, p=2)
    r.set_working_column()
    r.set_shortcuts(r.SHORTCUT_EMERGENT | r.SHORTCUT_CLEARING)
    try:
        got = r.barcode(x, max_dim=1)
    finally:
        r.set_shortcuts()
    for d in range(2):
        want = (ref.bars[d].birth, ref.bars[d].death, ref.bars[d].birth_simplex, ref.bars[d].death_simplex)
        b = got.bars[d]
        for g, w in zip((b.birth, b.death, b.birth_simplex, b.death_simplex), want):
            assert np.array_equal(g, w), d
