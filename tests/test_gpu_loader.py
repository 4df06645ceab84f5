"""The projections with loading wavefronts (loader_gemm.hip): the bits of the tiled kernels that load and multiply in the
same wavefronts, which the oracle tests pin, on every row count, K extent and column remainder where a tile, a ring or the
order of the tiles can go wrong."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# rows of the experts: none, one, around a block of 16, an odd and an even number of blocks, around a row tile of 192,
# tiles of unequal height
LOADS = [0, 1, 15, 16, 17, 0, 33, 95, 96, 97, 191, 192, 193, 210, 385, 600]


def _run(monkeypatch, wl, inp, what, calls, **env):
    import gpu_util as g
    with monkeypatch.context() as m:
        m.setenv("MOE_EP_NARROW_ROWS", "0")
        for name, value in env.items():
            m.setenv(name, value)
        ctx = g.make_ctx(wl)
    d = g.DeviceInputs(wl, inp)
    if what:
        ctx.prepare_weights(d.routed, d.shared)
    outs = [g.run_forward(ctx, wl, d, r=r, order=order) for r, order in calls]
    shape = ctx.last_tile_shape("routed_gate_up_gemm")
    assert (shape["rows"] == 192) == ("MOE_EP_GEMM_VARIANT" not in env), "the launches under test"
    ctx.destroy()
    return outs


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("merge", ["0", "1"])
@pytest.mark.parametrize("hidden,inter,shared_inter", [
    (64, 64, 64),        # one K step everywhere
    (128, 192, 64),      # 2, 3, and a shared down projection of 2: shorter than the rings are deep
    (320, 576, 320),     # 5, 9, 10; columns that end inside a tile on all sides
    (576, 256, 704),     # 9, 4 and 22
])
def test_same_bits_as_the_tiled_kernels(monkeypatch, hidden, inter, shared_inter, merge, prepared):
    wl = tiny_workload(name=f"loader_M{hidden}_H{inter}", n_tokens=sum(LOADS), hidden=hidden, inter=inter, n_experts=16,
                       n_local=16, top_k=1, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=71)
    logits = np.full((wl.n_tokens, wl.n_experts), -30.0, dtype=np.float32)
    logits[np.arange(wl.n_tokens), np.repeat(np.arange(16), LOADS)] = 5.0
    inp["gate_logits"][:] = logits[np.random.default_rng(7).permutation(wl.n_tokens)]
    calls = ((1, 0), (3, 0), (3, 1))
    want = _run(monkeypatch, wl, inp, prepared, calls, MOE_EP_GEMM_VARIANT="21")
    got = _run(monkeypatch, wl, inp, prepared, calls, MOE_EP_MERGE=merge)
    assert want[0].any()
    for w, o, c in zip(want, got, calls):
        assert np.array_equal(o, w), f"r, order = {c}"


@pytest.mark.parametrize("n_tokens,n_local,shared_inter", [
    (40, 7, 64),        # every expert one row tile: every second workgroup goes through its tiles backwards
    (700, 7, 1024),     # and with a shared down tile worth several routed ones
    (700, 1, 64),       # one expert
    (700, 300, 192),    # most experts one short tile, some none
])
def test_shared_experts_beside_single_row_tiles(monkeypatch, n_tokens, n_local, shared_inter):
    wl = tiny_workload(name=f"loader_mix_{n_local}", n_tokens=n_tokens, hidden=320, inter=192, n_experts=n_local + 3, local_begin=2,
                       n_local=n_local, top_k=2 if n_local > 1 else 1, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=72)
    want = _run(monkeypatch, wl, inp, True, ((1, 0), (2, 1)), MOE_EP_GEMM_VARIANT="21")
    got = _run(monkeypatch, wl, inp, True, ((1, 0), (2, 1)), MOE_EP_MERGE="1")
    assert want[0].any() and all(np.array_equal(o, w) for o, w in zip(got, want))


def test_more_tiles_than_are_decoded_ahead(monkeypatch):
    """512 experts of one row tile and 17 column tiles: 34 tiles of a single K step for every workgroup of 256."""
    import paper_2512_21487_amd as pkg
    M, H, E, T, k = 4352, 64, 512, 2048, 8
    gen = torch.Generator(device="cuda").manual_seed(73)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    outs = []
    for env in ({"MOE_EP_GEMM_VARIANT": "21"}, {"MOE_EP_NARROW_ROWS": "0"}):
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=0, shared_inter=0, max_tokens=T, max_top_k=k, max_chunks=1)
        out = torch.zeros(T * M, dtype=torch.bfloat16, device="cuda")
        ctx.forward(tokens, logits, routed, None, k, 1, 0, n_tokens=T, out=out)
        torch.cuda.synchronize()
        outs.append(out)
        ctx.destroy()
    assert outs[0].any() and torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.parametrize("prepared", [False, True])
def test_more_mixed_tiles_than_are_decoded_ahead(monkeypatch, prepared):
    """The same with shared experts in the launch and experts of one row tile, every second workgroup going through its tiles
    backwards: the list of decoded tiles (32 entries) is written over more than once, in either direction."""
    import paper_2512_21487_amd as pkg
    M, H, E, T, k, Ns, Hs = 8704, 64, 512, 2048, 8, 2, 64
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert E * (M // 256) > 2 * 32 * n_cu, "tiles of a workgroup"
    gen = torch.Generator(device="cuda").manual_seed(76)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed, shared = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02), normal(Ns * 3 * Hs * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    outs = []
    for env in ({"MOE_EP_GEMM_VARIANT": "21"}, {"MOE_EP_NARROW_ROWS": "0", "MOE_EP_MERGE": "1"}):
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=Ns, shared_inter=Hs, max_tokens=T, max_top_k=k, max_chunks=1)
        if prepared:
            ctx.prepare_weights(routed, shared)
        out = torch.zeros(T * M, dtype=torch.bfloat16, device="cuda")
        ctx.forward(tokens, logits, routed, shared, k, 1, 0, n_tokens=T, out=out)
        torch.cuda.synchronize()
        own = "MOE_EP_MERGE" in env
        assert (ctx.last_tile_shape("routed_down_gemm")["rows"] == 192) == own and ctx.last_shared_beside() == own, "the launches under test"
        assert ctx.get_routing()["count"].max() <= 192, "one row tile each"
        outs.append(out)
        ctx.destroy()
    assert outs[0].any() and torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


def test_tile_shape_of_a_chunk_without_a_token(monkeypatch):
    """Five tokens in four chunks of two: the last chunk launches nothing and is answered as the others."""
    import gpu_util as g
    wl = tiny_workload(name="loader_empty", n_tokens=5, hidden=128, inter=192, n_experts=4, n_local=4, top_k=2, n_shared=1, shared_inter=64)
    with monkeypatch.context() as m:
        m.setenv("MOE_EP_NARROW_ROWS", "0")
        ctx = g.make_ctx(wl)
    g.run_forward(ctx, wl, g.DeviceInputs(wl, make_inputs(wl, seed=75)), r=4, order=1)
    for stage in ("routed_gate_up_gemm", "routed_down_gemm"):
        shapes = [ctx.last_tile_shape(stage, chunk) for chunk in range(4)]
        assert shapes[0]["rows"] == 192 and all(shape == shapes[0] for shape in shapes)
    assert not ctx.last_shared_beside(3)
    ctx.destroy()


# 192 rows of 11184832 elements and more are 2^32 bytes: past what a lane of these kernels addresses in one tile
@pytest.mark.parametrize("hidden,inter,env", [
    (64, 11184832, {}),                                    # the down projection's rows
    (11184832, 64, {"MOE_EP_FUSED_GATHER": "0"}),          # the grouped copy of the token rows
])
def test_rows_longer_than_a_tile_can_address(monkeypatch, hidden, inter, env):
    import paper_2512_21487_amd as pkg
    T = 32
    gen = torch.Generator(device="cuda").manual_seed(74)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(T * hidden, 1.0), normal(3 * inter * hidden, 0.02 if hidden < 1000 else 5e-4)
    with monkeypatch.context() as m:
        for name, value in env.items():
            m.setenv(name, value)
        ctx = pkg.MoeEp(hidden=hidden, inter=inter, n_experts=1, n_local=1, n_shared=0, shared_inter=0, max_tokens=T, max_top_k=1, max_chunks=1)
    out = torch.zeros(T * hidden, dtype=torch.bfloat16, device="cuda")
    ctx.forward(tokens, torch.zeros(T, device="cuda"), routed, None, 1, 1, 0, n_tokens=T, out=out)
    torch.cuda.synchronize()
    assert ctx.last_tile_shape("routed_down_gemm")["rows"] == 128
    ctx.destroy()
    gate, up, down = routed.view(3, -1)
    x = tokens.view(T, hidden).float()
    z = x @ gate.view(inter, hidden).float().t()
    act = torch.nn.functional.silu(z) * (x @ up.view(inter, hidden).float().t())
    want = act @ down.view(hidden, inter).float().t()
    # bf16 rounding of the activation, of the expert's output and of the result: 2^-9 / sqrt(3) each at most, relative to the norm;
    # sums of 1.1e7 products in 3.5e5 steps of fp32: under 2^-24 sqrt(3.5e5) = 3.5e-5
    assert float((out.float().view(T, hidden) - want).norm() / want.norm()) < 5e-3


@pytest.mark.parametrize("n_shared", [0, 1])
@pytest.mark.parametrize("rounds", [1, 2])
@pytest.mark.parametrize("past", [0, 1])
def test_low_tiles_fill_the_rounds_or_miss_the_last(monkeypatch, n_shared, rounds, past):
    """Two experts that every token chooses: 128-row tiles, those of a shared expert among them, that are one or two per workgroup
    (or one less in all); with one row more in each expert they would be a round more and are 192 rows high."""
    import paper_2512_21487_amd as pkg
    n_cu = (torch.cuda.get_device_properties(0).multi_processor_count + 7) // 8 * 8
    M, H, T = 64, 64, rounds * n_cu // (2 + n_shared) * 128 + past
    gen = torch.Generator(device="cuda").manual_seed(77)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed, shared = normal(T * M, 1.0), normal(2 * 3 * H * M, 0.1), normal(3 * H * M, 0.1) if n_shared else None
    logits = torch.empty((T, 2), dtype=torch.float32, device="cuda").normal_(generator=gen)
    outs = []
    for env in ({"MOE_EP_GEMM_VARIANT": "21"}, {"MOE_EP_MERGE": "1"}):
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=2, n_local=2, n_shared=n_shared, shared_inter=H if n_shared else 0, max_tokens=T,
                            max_top_k=2, max_chunks=1)
        out = torch.zeros(T * M, dtype=torch.bfloat16, device="cuda")
        ctx.forward(tokens, logits, routed, shared, 2, 1, 0, n_tokens=T, out=out)
        torch.cuda.synchronize()
        assert (ctx.last_tile_shape("routed_down_gemm")["rows"] == 192) == ("MOE_EP_MERGE" in env)
        outs.append(out)
        ctx.destroy()
    assert outs[0].any() and torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
