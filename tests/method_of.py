"""Which method ran a call, by the kernel classes that the library times."""

SWEEPS = ("sweep", "sweep_d1", "sweep_d2", "batched_sweep")
COLUMNS = ("reduce_d1", "reduce_d2", "reduce_d3", "batched_graph")


def method_of(call):
    """The call's result and the sets of its sweeps and column reductions."""
    import torch
    import paper_1908_02518_amd as r
    r.profile_enable(True)
    try:
        out = call()
        torch.cuda.synchronize()
        ran = r.profile_read()
    finally:
        r.profile_enable(False)
    return out, {c for c in SWEEPS if c in ran}, {c for c in COLUMNS if c in ran}
