"""The switch between the sweep and the column reduction, and that each of them
runs where it is meant to: what a comparison of the two compares."""

import numpy as np
import pytest

import cpu_baseline
import oracle
import workloads
from tests.method_of import method_of
from tests.test_gpu_batched import small_batch
from tests.test_gpu_sweep import two_simplices

pytestmark = pytest.mark.gpu
INF = float("inf")


def rips():
    import paper_1908_02518_amd as r
    return r


def ring(n, noise=0.002):
    g = workloads.rng(n)
    a, r = g.uniform(0.0, 2.0 * np.pi, n), 1.0 + noise * g.standard_normal(n)
    return np.stack([r * np.cos(a), r * np.sin(a)], axis=1).astype(np.float32)


def rounded(x, digits):
    d = np.sqrt(((x[:, None].astype(np.float64) - x[None]) ** 2).sum(2)).round(digits).astype(np.float32)
    return np.ascontiguousarray(d)


SINGLE = [
    ("whole", lambda: workloads.sphere(100, 1), dict(max_dim=1, threshold=INF), {"sweep"}, {"reduce_d1"}),
    ("whole-p5", lambda: workloads.sphere(90, 2), dict(max_dim=1, threshold=INF, p=5), {"sweep"}, {"reduce_d1"}),
    ("chunks", lambda: workloads.clifford_torus(2000, 0.02, 3), dict(max_dim=1, threshold=0.5), {"sweep_d1"},
     {"reduce_d1"}),
    ("chunks-p3", lambda: workloads.clifford_torus(2000, 0.02, 3), dict(max_dim=1, threshold=0.5, p=3), {"sweep_d1"},
     {"reduce_d1"}),
    ("blocks", lambda: workloads.sphere(64, 4), dict(max_dim=2, threshold=INF), {"sweep_d1", "sweep_d2"},
     {"reduce_d1", "reduce_d2"}),
    # more than 2^28 possible edges: places by hashing (few classes are open at once on a ring)
    ("chunks-hashed-places", lambda: ring(23400), dict(max_dim=1, threshold=0.006), {"sweep_d1"}, {"reduce_d1"}),
    ("chunks-hashed-places-p3", lambda: ring(23400, 0.0001), dict(max_dim=1, threshold=0.006, p=3), {"sweep_d1"},
     {"reduce_d1"}),
    ("blocks-few-ties", lambda: rounded(workloads.sphere(52, workloads.SEED_BASE + 5), 5),
     dict(max_dim=2, threshold=INF, is_distance=True), {"sweep_d2"}, {"reduce_d1", "reduce_d2"}),
    ("blocks-few-ties-d3", lambda: rounded(workloads.orthogonal(520, workloads.SEED_BASE + 105), 5),
     dict(max_dim=3, threshold=1.8, is_distance=True), {"sweep_d2"}, {"reduce_d1", "reduce_d2", "reduce_d3"}),
    ("blocks-so3", lambda: workloads.so3(700, 5), dict(max_dim=2, threshold=1.4), {"sweep_d2"},
     {"reduce_d1", "reduce_d2"}),
]


@pytest.mark.parametrize("name,make,kw,sweeps,columns", SINGLE, ids=[c[0] for c in SINGLE])
def test_single_cloud_switch(name, make, kw, sweeps, columns):
    import torch
    r = rips()
    x = torch.from_numpy(make()).cuda()
    print(f"[case] method {name}", flush=True)
    (one, _), s, c = method_of(lambda: r.barcode_device(x, **kw))
    assert s >= sweeps and not any(f"reduce_{q[6:]}" in c for q in s if q != "sweep"), (s, c)
    for off in ("sweep", "workgroups"):
        if off == "sweep":
            r.set_sweep(r.SWEEP_BATCHED)
        else:
            r.set_sweep()
            r.set_reduce_workgroups(0)
        assert r.get_sweep() == r.SWEEP_BATCHED
        (two, _), s, c = method_of(lambda: r.barcode_device(x, **kw))
        assert not s and c == columns, (off, s, c)
        for a, b in zip(one, two):
            assert all(torch.equal(u, v) for u, v in zip(a, b))
    r.set_working_column()
    assert r.get_sweep() == r.SWEEP_SINGLE | r.SWEEP_BATCHED
    _, s, c = method_of(lambda: r.barcode_device(x, **kw))
    assert s >= sweeps


def assert_reference(bars, x, threshold, p=2):
    """Equal to the single-threaded CPU implementation, which the CPU tests
    hold to the oracle (the columns of large dense clouds take GPU memory that
    the process then keeps)."""
    ref = cpu_baseline.barcode(oracle.distances(x), len(x), max_dim=len(bars) - 1, threshold=threshold, p=p).bars
    for got, want in zip(bars, ref):
        for u, v in zip(got, (want.birth, want.death, want.birth_simplex, want.death_simplex)):
            assert np.array_equal(u.cpu().numpy(), v)


@pytest.mark.parametrize("n,max_dim,t,p", [(128, 0, INF, 2), (128, 0, 0.5, 3), (256, 1, 0.5, 2), (128, 1, 0.5, 3),
                                           (1024, 1, INF, 2), (200, 1, INF, 5)])
def test_largest_clouds_swept_whole(n, max_dim, t, p):
    """Swept up to n points, by the staged path from the next on."""
    import torch
    r = rips()
    for k, whole in ((n, True), (n + 1, False)):
        if k > 1024:
            continue
        x = workloads.sphere(k, k)
        print(f"[case] whole n={k} max_dim={max_dim} t={t} p={p}", flush=True)
        d = torch.from_numpy(x).cuda()
        (bars, _), s, _ = method_of(lambda: r.barcode_device(d, max_dim=max_dim, threshold=t, p=p))
        assert ("sweep" in s) == whole
        assert_reference(bars, x, t, p)


@pytest.mark.parametrize("m", [1, 4, 5, 64, 700])
@pytest.mark.parametrize("p", [2, 3])
def test_whole_clouds_of_many_coordinates(m, p):
    """The distances by the sweep's workgroup, and by the whole chip before it;
    from device and from host memory, and refused where one is not finite."""
    import torch
    r = rips()
    for n in (2, 33, 90):
        x = workloads.uniform_cube(n, m, n + m)
        d = torch.from_numpy(x).cuda()
        print(f"[case] coordinates m={m} n={n} p={p}", flush=True)
        (one, i1), s, c = method_of(lambda: r.barcode_device(d, max_dim=1, p=p))
        host = r.barcode(x, max_dim=1, p=p)
        r.set_sweep(0)
        two, i2 = r.barcode_device(d, max_dim=1, p=p)
        r.set_sweep()
        assert s == {"sweep"} and not c and i1["threshold"] == i2["threshold"]
        for a, b, h in zip(one, two, host.bars):
            assert all(torch.equal(u, v) for u, v in zip(a, b))
            assert np.array_equal(a[1].cpu(), h.death) and np.array_equal(a[3].cpu(), h.death_simplex)
        for bad in (float("nan"), INF):
            y = d.clone()
            y[n - 1, m - 1] = bad
            with pytest.raises(r.RipsError) as e:
                r.barcode_device(y, max_dim=1, p=p)
            assert e.value.status == -4


@pytest.mark.parametrize("n,m,p,whole", [(200, 16, 2, True), (220, 64, 2, False), (160, 5, 3, True),
                                           (200, 16, 3, False)])
def test_whole_clouds_of_many_classes(n, m, p, whole):
    """Up to two classes a point, or 220 over another field, by the sweep;
    with more the staged path follows it."""
    import torch
    r = rips()
    x = torch.from_numpy(workloads.uniform_cube(n, m, n)).cuda()
    print(f"[case] classes n={n} m={m} p={p}", flush=True)
    (one, info), s, c = method_of(lambda: r.barcode_device(x, max_dim=1, p=p, cap=4 * n))
    most = 2 * n if p == 2 else 220
    assert (info["stats"][1]["columns"] <= most) == whole
    assert "sweep" in s and (not c) == whole
    r.set_sweep(0)
    two, _ = r.barcode_device(x, max_dim=1, p=p, cap=4 * n)
    for a, b in zip(one, two):
        assert all(torch.equal(u, v) for u, v in zip(a, b))


@pytest.mark.parametrize("data,sweeps", [("even", True), ("crowded", False)])
def test_chunks_where_the_points_lie_evenly(data, sweeps):
    """A cloud with a crowd in it goes by columns, at the same mean degree."""
    import torch
    r = rips()
    g = workloads.rng(7)
    x = g.uniform(0.0, 1.0, (1500, 3))
    t = 0.19
    if data == "crowded":
        x[:250] = 0.5 + 0.03 * g.standard_normal((250, 3))
        t = 0.13
    x = torch.from_numpy(x.astype(np.float32)).cuda()
    print(f"[case] chunks {data}", flush=True)
    (one, info), s, c = method_of(lambda: r.barcode_device(x, max_dim=1, threshold=t))
    degree = 2 * info["simplex_count"][1] / 1500
    assert 32 < degree < 200, degree
    assert (s == {"sweep_d1"} and not c) if sweeps else (not s and c == {"reduce_d1"})
    r.set_sweep(0 if sweeps else 3)
    two, _ = r.barcode_device(x, max_dim=1, threshold=t)
    for a, b in zip(one, two):
        assert all(torch.equal(u, v) for u, v in zip(a, b))


@pytest.mark.parametrize("data,t,sweeps", [("so3", 1.3, True), ("so3", 1.1, False), ("crowded", 0.15, False)])
@pytest.mark.parametrize("p", [2, 3])
def test_blocks_where_edges_have_triangles(data, t, sweeps, p):
    """Dimension 2 of a sparse or of a crowded cloud goes by columns."""
    import torch
    r = rips()
    x = workloads.so3(1000, 11)
    if data == "crowded":
        g = workloads.rng(8)
        x = g.uniform(0.0, 1.0, (900, 3))
        x[:150] = 0.5 + 0.05 * g.standard_normal((150, 3))
        x = x.astype(np.float32)
    d = torch.from_numpy(x).cuda()
    print(f"[case] blocks {data} t={t} p={p}", flush=True)
    (one, info), s, c = method_of(lambda: r.barcode_device(d, max_dim=2, threshold=t, p=p))
    edges, triangles = info["simplex_count"][1:3]
    assert triangles > 12288 and (triangles >= 5 * edges) == (sweeps or data == "crowded"), (edges, triangles)
    assert ("sweep_d2" in s) == sweeps and ("reduce_d2" in c) != sweeps, (s, c)
    assert_reference(one, x, t, p)


def test_blocks_of_a_lune_of_many_points():
    """An even cloud in which two points are near 1100 others: their edge has
    more points in its lune than one block's forest holds."""
    import torch
    r = rips()
    x = workloads.sphere(6000, 12)
    d = np.empty((6000, 6000), np.float32)
    for i in range(0, 6000, 500):
        d[i:i + 500] = np.sqrt(np.maximum(((x[i:i + 500, None] - x[None]) ** 2).sum(2), 0.0))
    t = 0.2
    d[d > t] = 9.0
    w = t * (1.0 + 0.1 * workloads.rng(13).uniform(0.0, 1.0, (2, 1100))).astype(np.float32)
    d[:2, 2:1102], d[2:1102, :2] = w, w.T
    d[0, 1] = d[1, 0] = np.float32(1.2 * t)
    x = torch.from_numpy(d).cuda()
    out = {}
    for flags in (3, 0):
        print(f"[case] blocks, large lune, flags={flags}", flush=True)
        r.set_sweep(flags)
        r.profile_enable(True)
        try:
            out[flags], info = r.barcode_device(x, max_dim=2, threshold=1.2 * t, is_distance=True)
            torch.cuda.synchronize()
            ran = r.profile_read()
        finally:
            r.profile_enable(False)
        assert ("sweep_build_d2" in ran) == (flags == 3) and "reduce_d2" in ran, sorted(ran)
    for a, b in zip(out[3], out[0]):
        assert all(torch.equal(u, v) for u, v in zip(a, b))


def _bars(bb):
    n = int(bb.offsets[-1])
    return [t[:n].clone() for t in (bb.birth, bb.death, bb.birth_simplex, bb.death_simplex)] + [bb.offsets.clone()]


@pytest.mark.parametrize("m", [7, 8, 9, 16, 17, 130])
def test_batches_of_many_coordinates(m):
    """Distances pair by pair and coordinate by coordinate, with remainders;
    clouds of 129 points and more than 128 coordinates go by columns."""
    import torch
    r = rips()
    for n in (65, 129):
        x, off, nmax = r.pack_clouds([workloads.uniform_cube(k, m, k) for k in (1, 2, 33, 64, n)])
        print(f"[case] batch coordinates m={m} n={n}", flush=True)
        call = lambda: _bars(r.barcode_batched(x, off, nmax, max_dim=1, cap=1 << 13))
        one, s, c = method_of(call)
        assert (s, c) == ((set(), {"batched_graph"}) if n > 128 and m > 128 else ({"batched_sweep"}, set()))
        r.set_sweep(0)
        two = call()
        r.set_sweep()
        assert all(torch.equal(a, b) for a, b in zip(one, two))
        y = x.clone()
        y[-1, m - 1] = INF
        with pytest.raises(r.RipsError) as e:
            r.barcode_batched(y, off, nmax, max_dim=1)
        assert e.value.status == -4


def test_batched_columns_over_z2():
    """The direct-mapped columns of a batch, spread out and by one workgroup a
    cloud, the replays of their graph, and the sweep: the same bars."""
    import torch
    r = rips()
    x, off, nmax = r.pack_clouds(small_batch() + [workloads.integer_lattice(n, 3, n, side=4) for n in (20, 64, 90)]
                                 + [np.pad(workloads.noisy_circle_with_outliers(1, 270, 30), ((0, 0), (0, 1)))])
    print("[case] batched columns over Z/2", flush=True)
    call = lambda: _bars(r.barcode_batched(x, off, nmax, max_dim=1, p=2, cap=1 << 15))
    want, s, c = method_of(call)
    assert s == {"batched_sweep"} and not c
    r.set_sweep(r.SWEEP_SINGLE)
    for spread in (0, 1):
        r.batched_set_spread(spread)
        for _ in range(3):
            got, s, c = method_of(call)
            assert not s and c == {"batched_graph"}
            assert all(torch.equal(a, b) for a, b in zip(want, got))


def test_batch_with_a_full_cloud_goes_by_columns():
    r = rips()
    x, off, nmax = r.pack_clouds([two_simplices(40), workloads.uniform_cube(40, 80, 1)])
    print("[case] batch with a full cloud", flush=True)
    _, s, c = method_of(lambda: r.barcode_batched(x, off, nmax, max_dim=1))
    assert s == {"batched_sweep"} and c == {"batched_graph"}


def test_autotune_times_the_columns():
    r = rips()
    x, off, nmax = r.pack_clouds(small_batch())
    print("[case] autotune", flush=True)
    want = _bars(r.barcode_batched(x, off, nmax, max_dim=1, cap=1 << 14))
    tuned, s, c = method_of(lambda: r.batched_autotune(x, off, nmax, max_dim=1, cap=1 << 14, reps=1))
    assert s == {"batched_sweep"} and c == {"batched_graph"}  # its first call is an ordinary one
    assert r.batched_get_config() == tuned[:2]
    assert r.get_sweep() == r.SWEEP_SINGLE | r.SWEEP_BATCHED
    got, s, c = method_of(lambda: _bars(r.barcode_batched(x, off, nmax, max_dim=1, cap=1 << 14)))
    assert s == {"batched_sweep"} and not c
    assert all(np.array_equal(a.cpu(), b.cpu()) for a, b in zip(want, got))


DENSE = [("circle", 614), ("circle", 615), ("circle", 1023), ("circle", 1024), ("lattice", 614), ("lattice", 615),
         ("lattice", 1024)]


@pytest.mark.parametrize("data,n", DENSE, ids=[f"{d}-{n}" for d, n in DENSE])
def test_large_dense_clouds(data, n):
    """Every edge in: the nonzero-edge bits in LDS up to 614 points, longer
    sorts, chunks and lists."""
    import torch
    r = rips()
    x = workloads.noisy_circle_with_outliers(n, n - n // 10, n // 10) if data == "circle" else \
        workloads.integer_lattice(n, 2, n, side=40)
    print(f"[case] dense {data} n={n}", flush=True)
    (bars, _), s, c = method_of(lambda: r.barcode_device(torch.from_numpy(x).cuda(), max_dim=1))
    assert s == {"sweep"} and not c
    assert_reference(bars, x, INF)


def test_batch_of_tiny_and_largest_clouds():
    r = rips()
    clouds = [workloads.uniform_cube(k, 2, k) for k in (1, 2, 3, 40)] + \
        [workloads.noisy_circle_with_outliers(3, 1900, 148), workloads.integer_lattice(900, 2, 5, side=60)]
    x, off, nmax = r.pack_clouds(clouds)
    assert nmax == 2048
    print("[case] batch of tiny and largest clouds", flush=True)
    bb, s, c = method_of(lambda: r.barcode_batched(x, off, nmax, max_dim=1, threshold=0.3))
    assert s == {"batched_sweep"} and not c
    for b, cloud in enumerate(clouds):
        assert_reference([bb.segment(b, d) for d in range(2)], cloud, 0.3)
