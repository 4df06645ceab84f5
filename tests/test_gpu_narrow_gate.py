"""Gate and partition of at most 4 tokens inside the gate/up projection's launch (narrow_gemm.hip): the routing and the bits of the
gate's own launch, with ties, scores out of order, experts and slots where its lists end, shared experts beside and apart."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("hidden,inter,n_experts,local_begin,n_local,top_k,n_shared,shared_inter", [
    (64, 64, 4, 1, 1, 4, 0, 0),            # fewer experts than lanes, every one chosen, one here
    (1088, 192, 64, 0, 64, 6, 2, 1024),    # 64 scores: the shortest list full; tiles of one wavefront
    (192, 576, 65, 3, 62, 64, 1, 64),      # one more; as many slots as there can be
    (256, 512, 160, 5, 20, 6, 2, 192),     # the next list full, a share
    (1024, 1024, 161, 1, 160, 8, 0, 0),    # one more
    (320, 64, 256, 0, 256, 9, 3, 448),     # the longest list full
    (320, 64, 257, 0, 257, 9, 0, 0),       # one more: a launch of its own
])
def test_same_routing_and_bits(monkeypatch, hidden, inter, n_experts, local_begin, n_local, top_k, n_shared, shared_inter, prepared):
    import gpu_util as g
    wl = tiny_workload(name=f"gate_E{n_experts}", n_tokens=9, hidden=hidden, inter=inter, n_experts=n_experts, local_begin=local_begin,
                       n_local=n_local, top_k=top_k, n_shared=n_shared, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=95)
    inp["gate_logits"][1] = np.round(inp["gate_logits"][1])     # ties: the lower expert
    inp["gate_logits"][2] = -0.0
    inp["gate_logits"][3, ::2] = -np.inf
    d = g.DeviceInputs(wl, inp)

    def run(narrow_rows):
        with monkeypatch.context() as m:
            m.setenv("MOE_EP_NARROW_ROWS", narrow_rows)
            ctx = g.make_ctx(wl)
        if prepared:
            ctx.prepare_weights(d.routed, d.shared if n_shared else None)
        got = {}
        for n, r, order in ((1, 1, 0), (2, 1, 0), (3, 1, 1), (4, 1, 0), (5, 1, 0), (8, 2, 0), (9, 3, 1)):
            out = g.run_forward(ctx, wl, d, n_tokens=n, r=r, order=order)[:n].copy()
            got[n, r] = out, [ctx.get_routing(chunk) for chunk in range(r)]
        ctx.destroy()
        return got

    want, got = run("0"), run("1e9")
    for case, (out, routing) in want.items():
        for a, b in zip(routing, got[case][1]):
            for name in a:
                assert np.array_equal(np.asarray(a[name]), np.asarray(b[name])), (case, name)
        assert np.array_equal(got[case][0], out), case
    assert want[9, 3][0].any()
