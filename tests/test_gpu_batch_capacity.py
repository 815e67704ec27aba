"""A batch with more bars than the caller's arrays hold: RIPS_E_CAPACITY with
the number needed, the arrays as they were, and every bar once they are large
enough. The bars of a cloud lie anywhere in the unordered buffer, so that a
cloud whose output fits may have none there; over Z/2 some clouds exceed the
sweep's tables and the whole batch goes by columns."""

import ctypes

import pytest

import workloads
from tests.test_gpu_sweep import two_simplices

pytestmark = pytest.mark.gpu
INF = float("inf")


def rips():
    import paper_1908_02518_amd as r
    return r


def call(x, off, nmax, cap, p, max_dim):
    """Status, number needed and the arrays, filled with -7 before the call."""
    import torch
    r = rips()
    B, d1 = off.shape[0] - 1, max_dim + 1
    f = [torch.full((max(cap, 1),), -7.0, device="cuda") for _ in range(2)]
    i = [torch.full((max(cap, 1),), -7, dtype=torch.int64, device="cuda") for _ in range(2)]
    offsets = torch.empty(B * d1 + 1, dtype=torch.int64, device="cuda")
    o = r.rips_batch_out()
    o.cap = cap
    o.birth, o.death, o.birth_simplex, o.death_simplex = (t.data_ptr() for t in f + i)
    o.bar_offsets, o.stats, o.threshold_used = offsets.data_ptr(), None, None
    st = r.lib().rips_barcode_batched_device(
        ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(off.data_ptr()), B, x.shape[1], nmax, max_dim,
        ctypes.c_float(INF), p, ctypes.byref(o), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return st, int(o.needed), f + i, offsets


CLOUDS = {
    "uneven": lambda: [workloads.sphere(3 + 11 * (b % 5), b + 1) for b in range(24)],
    "loops": lambda: [two_simplices(40)] * 12,
    "one-full": lambda: [two_simplices(40)] + [workloads.uniform_cube(40, 80, b) for b in range(30)],
}


@pytest.mark.parametrize("max_dim", [0, 1])
@pytest.mark.parametrize("method", ["default", "columns", "another-field"])
@pytest.mark.parametrize("kind", sorted(CLOUDS))
def test_arrays_untouched_below_the_need(kind, method, max_dim):
    import torch
    r = rips()
    p = 3 if method == "another-field" else 2
    x, off, nmax = r.pack_clouds(CLOUDS[kind]())
    r.set_working_column(r.WORKING_COLUMN_GENERAL if method == "columns" else r.WORKING_COLUMN_AUTO)
    try:
        want = r.barcode_batched(x, off, nmax, max_dim=max_dim, p=p, cap=1 << 16)
        total = int(want.offsets[-1])
        for cap in (0, 1, total // 7, total - 1, total):
            print(f"[case] capacity {kind} {method} max_dim={max_dim} cap={cap} of {total}", flush=True)
            st, need, arrays, offsets = call(x, off, nmax, cap, p, max_dim)
            assert need == total
            assert torch.equal(offsets, want.offsets)
            if cap < total:
                assert st == -6
                for t in arrays:
                    assert bool((t == -7).all())
            else:
                assert st == 0
                for t, w in zip(arrays, (want.birth, want.death, want.birth_simplex, want.death_simplex)):
                    assert torch.equal(t, w[:total])
    finally:
        r.set_working_column()
