"""Routed and shared experts in one launch per projection (loader_gemm.hip) against the tiled kernels in launches of
their own, which the oracle tests pin: the same bits whatever the two sides' tile counts, K and columns are."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(monkeypatch, wl, inp, merge, prepared, calls, pinned=False):
    import gpu_util as g
    monkeypatch.setenv("MOE_EP_NARROW_ROWS", "0")
    monkeypatch.setenv("MOE_EP_MERGE", str(merge))
    ctx = g.make_ctx(wl, pinned=pinned)
    d = g.DeviceInputs(wl, inp, pinned=pinned)
    if prepared:
        ctx.prepare_weights(d.routed, d.shared)
    outs = []
    for r, order in calls:
        outs.append(g.run_forward(ctx, wl, d, r=r, order=order))
        assert ctx.last_shared_beside() == bool(merge), "the launches under test"
        assert ctx.last_tile_shape("routed_gate_up_gemm")["rows"] >= 128   # not the narrow kernels
    ctx.destroy()
    return outs


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("n_tokens,hidden,inter,n_shared,shared_inter", [
    (1, 192, 192, 1, 192),        # one tile of each, the shortest K
    (161, 320, 192, 3, 256),      # a shared down tile worth four routed ones (K 768 against 192), K segments
    (777, 192, 576, 1, 192),      # and one of a third of a routed tile's K
    (600, 448, 320, 2, 320),      # columns that end inside a tile on both sides
    (3000, 256, 192, 2, 1024),    # more shared gate/up tiles than workgroups
    (20500, 256, 192, 1, 192),    # more shared down tiles than workgroups, few routed ones
])
def test_same_bits_as_launches_of_their_own(monkeypatch, n_tokens, hidden, inter, n_shared, shared_inter, prepared):
    wl = tiny_workload(name="merged", n_tokens=n_tokens, hidden=hidden, inter=inter, n_experts=24, local_begin=3,
                       n_local=7, top_k=3, n_shared=n_shared, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=91)
    inp["gate_logits"][:, 5] -= 30.0    # an expert of the share without rows
    calls = ((1, 0), (1, 1), (3, 0), (3, 1)) if n_tokens < 4000 else ((1, 0),)
    want = _run(monkeypatch, wl, inp, 0, prepared, calls)
    assert want[0].any()
    for pinned in (False, True):
        got = _run(monkeypatch, wl, inp, 1, prepared, calls, pinned)
        for w, o, c in zip(want, got, calls):
            assert np.array_equal(o, w), f"r, order = {c}, pinned = {pinned}"


def test_share_without_any_row(monkeypatch):
    """No token keeps a local expert: the launch is the shared experts alone."""
    wl = tiny_workload(name="merged_none", n_tokens=500, hidden=256, inter=192, n_experts=8, local_begin=6, n_local=2,
                       top_k=2, n_shared=1, shared_inter=256)
    inp = make_inputs(wl, seed=92)
    inp["gate_logits"][:, 6:] = -40.0
    want = _run(monkeypatch, wl, inp, 0, True, ((1, 0),))
    got = _run(monkeypatch, wl, inp, 1, True, ((1, 0),))
    assert want[0].any() and np.array_equal(got[0], want[0])


@pytest.mark.parametrize("narrow_rows", ["0", "1e9"])   # the tiled launches, the narrow ones
def test_timing_a_forward(monkeypatch, narrow_rows):
    """What bench.py times inside its timed region is the launches an untimed forward makes; timing the shared experts'
    stages takes them apart, timing the routed ones alone does not.  The bits are the same."""
    import bench
    import gpu_util as g
    monkeypatch.setenv("MOE_EP_NARROW_ROWS", narrow_rows)
    monkeypatch.setenv("MOE_EP_MERGE", "1")
    wl = tiny_workload(name="timing", n_tokens=300, hidden=256, inter=192, n_experts=8, n_local=8, top_k=2, n_shared=1, shared_inter=256)
    ctx = g.make_ctx(wl)
    d = g.DeviceInputs(wl, make_inputs(wl, seed=93))
    want = g.run_forward(ctx, wl, d)
    assert ctx.last_shared_beside() and want.any()
    for names, beside in ((bench.TIMED_REGION_STAGES, True), (["routed_gate_up_gemm", "routed_down_gemm"], True),
                          (["shared_down_gemm"], False), (None, False)):
        ctx.set_profiling_stages(names)
        ctx.set_profiling(1)
        assert np.array_equal(g.run_forward(ctx, wl, d), want)
        assert ctx.last_shared_beside() == beside, names
        ms = ctx.get_stage_ms()
        assert all(ms[n] > 0.0 for n in names or ("routed_gate_up_gemm", "shared_gate_up_gemm", "shared_down_gemm", "forward"))
        ctx.set_profiling(0)
    assert np.array_equal(g.run_forward(ctx, wl, d), want) and ctx.last_shared_beside()
    ctx.destroy()
