"""Gate, partition and aggregation where their workgroups, masks and passes begin and end: token counts around 16 and
64, experts around the registers of a lane and the threads of a workgroup, top-k up to 64, equal and infinite scores."""
import numpy as np
import pytest

import oracle
from helpers import rel_err_rows
from workloads import bf16_bits_to_f32, make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tokens", [1, 2, 15, 16, 17, 63, 64, 65, 79, 129, 1100])
@pytest.mark.parametrize("n_experts,n_local,top_k", [(1, 1, 1), (17, 5, 4), (128, 128, 8), (161, 100, 9), (512, 512, 64)])
def test_routing_is_exact(n_tokens, n_experts, n_local, top_k):
    """Selected experts, counts, offsets and both maps bit for bit; a third of the scores on a coarse grid (equal
    scores, both zeros), some rows with scores of minus infinity and of the type's lowest value."""
    import gpu_util as g
    begin = min(2, n_experts - n_local)
    wl = tiny_workload(name="routing", n_tokens=n_tokens, hidden=64, inter=64, n_experts=n_experts, local_begin=begin,
                       n_local=n_local, top_k=top_k)
    inp = make_inputs(wl, seed=81)
    lg = inp["gate_logits"]
    lg[::3] = np.round(lg[::3] * 2.0) / 2.0
    lg[1::6] = np.where(lg[1::6] < -0.3, np.float32(-0.0), np.float32(0.0))
    if n_experts > 2 * top_k:
        lg[2::5, : n_experts // 3] = -np.inf
        lg[4::5, n_experts // 3: n_experts // 2] = np.finfo(np.float32).min
    idx = np.argsort(-lg.astype(np.float64), axis=1, kind="stable")[:, :top_k].astype(np.int32)
    sel = np.take_along_axis(lg, idx, 1).astype(np.float64)
    w = np.exp(sel - sel[:, :1])
    w /= w.sum(axis=1, keepdims=True)
    ctx = g.make_ctx(wl)
    d = g.DeviceInputs(wl, inp)
    g.run_forward(ctx, wl, d)
    got = ctx.get_routing(0)
    ctx.destroy()
    part = oracle.dispatch(idx, begin, n_local)
    assert np.array_equal(got["idx"], idx)
    for key in ("count", "offset", "perm", "pos"):
        assert np.array_equal(got[key], part[key]), key
    assert np.max(np.abs(got["w"] - w)) <= 2e-6   # fp32 exp and division against float64


@pytest.mark.parametrize("hidden", [64, 960, 1024, 1088, 2112])
@pytest.mark.parametrize("top_k,n_local,n_shared", [(1, 9, 0), (3, 9, 1), (7, 9, 0), (7, 4, 1)])
def test_aggregation_of_every_slot_count(hidden, top_k, n_local, n_shared):
    """Rows shorter than, equal to and longer than a wavefront's piece of 1024 columns, and every number of kept
    slots from none to seven (fetched in fours, twos and ones)."""
    import gpu_util as g
    wl = tiny_workload(name="aggregation", n_tokens=70, hidden=hidden, inter=64, n_experts=9, n_local=n_local, top_k=top_k,
                       n_shared=n_shared, shared_inter=64)
    inp = make_inputs(wl, seed=82)
    ref = oracle.forward(inp["tokens"], inp["gate_logits"], inp["routed_w"], inp["shared_w"], hidden=hidden, inter=64,
                         n_experts=9, local_begin=0, n_local=n_local, n_shared=n_shared, shared_inter=64, top_k=top_k, r_chunks=1)
    for pinned in (False, True):
        ctx = g.make_ctx(wl, pinned=pinned)
        out = bf16_bits_to_f32(g.run_forward(ctx, wl, g.DeviceInputs(wl, inp, pinned=pinned)))
        ctx.destroy()
        assert rel_err_rows(out, ref["out"]) <= 2e-2   # the bound of every full-path comparison (test_gpu_parity)


@pytest.mark.parametrize("n_tokens", [5, 100])   # one launch with the partition, and one in front of it
@pytest.mark.parametrize("n_experts,top_k", [(128, 8), (20, 7)])
def test_scores_that_are_not_numbers_select_no_expert_twice(n_tokens, n_experts, top_k):
    """Padding rows of 0xff bytes (every score a NaN) and rows in which only a few scores are numbers: a token's experts
    are different ones, so that the partition's rows and maps belong together; the other tokens are not touched."""
    import gpu_util as g
    wl = tiny_workload(name="nan", n_tokens=n_tokens, hidden=64, inter=64, n_experts=n_experts, n_local=n_experts, top_k=top_k)
    inp = make_inputs(wl, seed=83)
    lg = inp["gate_logits"]
    clean = np.argsort(-lg.astype(np.float64), axis=1, kind="stable")[:, :top_k]
    bits = lg.view(np.uint32)
    bits[0::4] = 0xffffffff
    bits[1::4, 3:] = 0xffffffff
    ctx = g.make_ctx(wl)
    g.run_forward(ctx, wl, g.DeviceInputs(wl, inp))
    got = ctx.get_routing(0)
    ctx.destroy()
    idx = got["idx"]
    assert idx.min() >= 0 and idx.max() < n_experts
    assert all(len(set(row)) == top_k for row in idx.tolist())
    part = oracle.dispatch(idx, 0, n_experts)
    for key in ("count", "offset", "perm", "pos"):
        assert np.array_equal(got[key], part[key]), key
    assert np.array_equal(idx[2::4], clean[2::4]) and np.array_equal(idx[3::4], clean[3::4])
