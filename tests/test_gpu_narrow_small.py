"""Tiles of one wavefront and of pairs (narrow_gemm.hip, up to 32 tokens): the bits of the tiled kernels, which the oracle
tests pin, at the token counts where the tiles change and with columns and reductions that end inside a tile or a staged chunk."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _forwards(monkeypatch, wl, d, what, rows, token_counts):
    import gpu_util as g
    with monkeypatch.context() as m:
        m.setenv("MOE_EP_NARROW_ROWS", rows)
        ctx = g.make_ctx(wl)
    if what:
        ctx.prepare_weights(d.routed, d.shared if wl.n_shared else None)
    outs = []
    for n in token_counts:
        out = g.run_forward(ctx, wl, d, n_tokens=n)[:n].copy()
        outs.append((out, [(ctx.last_tile_shape(s)["rows"], ctx.last_tile_shape(s)["waves_n"]) for s in ("routed_gate_up_gemm", "routed_down_gemm")]))
    ctx.destroy()
    return outs


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("hidden,inter,n_shared,shared_inter", [
    (1024, 1024, 0, 0),       # 16 K steps: whole staged chunks; whole tiles
    (1088, 1088, 2, 1024),    # 17 and 32; columns that end inside tiles of 64 and 128
    (1216, 1152, 1, 1344),    # 19, 18 and 21
])
def test_same_bits_as_the_tiled_kernels(monkeypatch, hidden, inter, n_shared, shared_inter, prepared):
    import gpu_util as g
    wl = tiny_workload(name=f"small_M{hidden}", n_tokens=33, hidden=hidden, inter=inter, n_experts=24, local_begin=4, n_local=3,
                       top_k=3, n_shared=n_shared, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=81)
    inp["gate_logits"][::3, 5] += 20.0     # an expert of the share that every third token chooses
    d = g.DeviceInputs(wl, inp)
    counts = (1, 2, 15, 16, 17, 31, 32, 33)
    want = _forwards(monkeypatch, wl, d, prepared, "0", counts)
    got = _forwards(monkeypatch, wl, d, prepared, "1e9", counts)
    for n, (w, tiled), (o, tiles) in zip(counts, want, got):
        tile = (16, 1) if n <= 16 else (32, 2) if n <= 32 else (64, 4)
        assert tiles == [tile, (16, 8) if n <= 16 else tile] and tiled[0][0] > 64, f"{n} tokens: the launches under test"
        assert np.array_equal(o, w), f"{n} tokens"
    assert want[-1][0].any()


def test_every_token_on_the_same_experts(monkeypatch):
    """16 and 32 rows in one group, the others empty."""
    import gpu_util as g
    wl = tiny_workload(name="small_hot", n_tokens=32, hidden=1024, inter=1088, n_experts=24, n_local=24, top_k=1)
    inp = make_inputs(wl, seed=82)
    inp["gate_logits"][:, 7] += 30.0
    d = g.DeviceInputs(wl, inp)
    want = _forwards(monkeypatch, wl, d, True, "0", (16, 32))
    got = _forwards(monkeypatch, wl, d, True, "1e9", (16, 32))
    for (w, _), (o, _) in zip(want, got):
        assert w.any() and np.array_equal(o, w)
