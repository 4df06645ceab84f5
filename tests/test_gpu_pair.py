"""Both projections in one launch (loader_gemm.hip) against a launch of each, which test_gpu_loader.py pins: the same bits on every
row count, K extent and column remainder, however many tiles are drawn at a time and whoever draws them."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# as in test_gpu_loader.py: none, one, around blocks of 16 and row tiles of 128 and 192
LOADS = [0, 1, 15, 16, 17, 0, 33, 95, 96, 97, 191, 192, 193, 210, 385, 600]


def _joint(ctx, chunks=1):
    return [ctx.last_projections_joint(c) for c in range(chunks)]


def _ctx(monkeypatch, make, pair, **env):
    with monkeypatch.context() as m:
        m.setenv("MOE_EP_NARROW_ROWS", "0")
        m.setenv("MOE_EP_PAIR", str(pair))
        for name, value in env.items():
            m.setenv(name, value)
        return make()


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("merge", ["0", "1"])
@pytest.mark.parametrize("hidden,inter,shared_inter", [
    (64, 64, 64),        # one K step everywhere: eight tiles at a time
    (128, 192, 64),      # 2, 3, and a shared down projection of 2
    (576, 256, 704),     # 9, 4 and 22; columns that end inside a tile
    (64, 1088, 64),      # 17 column tiles of gate/up, one of down
])
def test_same_bits_as_a_launch_of_each(monkeypatch, hidden, inter, shared_inter, merge, prepared):
    import gpu_util as g
    wl = tiny_workload(name=f"pair_M{hidden}_H{inter}", n_tokens=sum(LOADS), hidden=hidden, inter=inter, n_experts=16,
                       n_local=16, top_k=1, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=81)
    logits = np.full((wl.n_tokens, wl.n_experts), -30.0, dtype=np.float32)
    logits[np.arange(wl.n_tokens), np.repeat(np.arange(16), LOADS)] = 5.0
    inp["gate_logits"][:] = logits[np.random.default_rng(8).permutation(wl.n_tokens)]
    outs = []
    for pair in (0, 1):
        ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl), pair, MOE_EP_MERGE=merge)
        d = g.DeviceInputs(wl, inp)
        if prepared:
            ctx.prepare_weights(d.routed, d.shared)
        outs.append([])
        for r, order in ((1, 0), (3, 0), (3, 1)):
            outs[-1].append(g.run_forward(ctx, wl, d, r=r, order=order))
            assert _joint(ctx, r) == [bool(pair)] * r, "the launches under test"
        assert ctx.last_tile_shape("routed_gate_up_gemm")["rows"] == 192, "the launches under test"
        ctx.destroy()
    assert outs[0][0].any() and all(np.array_equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("n_tokens,n_local,shared_inter", [
    (40, 7, 64),        # one row tile each: some workgroups begin with the routed tiles
    (700, 1, 64),       # one expert
    (700, 300, 192),    # most experts one short tile, some none
    (1, 3, 64),         # one row
])
def test_few_and_many_experts(monkeypatch, n_tokens, n_local, shared_inter):
    import gpu_util as g
    wl = tiny_workload(name=f"pair_{n_local}", n_tokens=n_tokens, hidden=320, inter=192, n_experts=n_local + 3, local_begin=2,
                       n_local=n_local, top_k=2 if n_local > 1 else 1, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=82)
    outs = []
    for pair in (0, 1):
        ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl), pair, MOE_EP_MERGE="1")
        d = g.DeviceInputs(wl, inp)
        ctx.prepare_weights(d.routed, d.shared)
        outs.append([])
        for r in (1, 2):
            outs[-1].append(g.run_forward(ctx, wl, d, r=r, order=r - 1))
            assert _joint(ctx, r) == [bool(pair) and c < n_tokens for c in range(r)], "the launches under test"   # none for a chunk without a token
        ctx.destroy()
    assert outs[0][0].any() and all(np.array_equal(a, b) for a, b in zip(*outs))


def _layer(monkeypatch, pair, M=4352, H=64, E=512, T=2048, k=8, seed=83):
    """Experts of one row tile and 17 column tiles of a single K step in the down projection."""
    import paper_2512_21487_amd as pkg
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    ctx = _ctx(monkeypatch, lambda: pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=0, shared_inter=0, max_tokens=T,
                                              max_top_k=k, max_chunks=1), pair)
    out = torch.zeros(T * M, dtype=torch.bfloat16, device="cuda")
    return ctx, lambda: ctx.forward(tokens, logits, routed, None, k, 1, 0, n_tokens=T, out=out), out, logits


def test_more_tiles_than_are_kept_and_two_streams(monkeypatch):
    """The list of drawn tiles is written over many times; two contexts on two streams share the compute units."""
    want = []
    for seed in (83, 84):
        ctx, run, out, _ = _layer(monkeypatch, 0, seed=seed)
        run()
        torch.cuda.synchronize()
        assert _joint(ctx) == [False]
        want.append(out.clone())
        ctx.destroy()
    sides = [_layer(monkeypatch, 1, seed=seed) for seed in (83, 84)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(4):
        for (ctx, run, out, _), s in zip(sides, streams):
            with torch.cuda.stream(s):
                out.zero_()
                run()
    torch.cuda.synchronize()
    for (ctx, _, out, _), w in zip(sides, want):
        assert _joint(ctx) == [True] and w.any() and torch.equal(out.view(torch.int16), w.view(torch.int16))
        ctx.destroy()


def test_replayed_graph(monkeypatch):
    """The counters are cleared inside the captured launches: every replay gives the eager bits, also for other scores."""
    ctx, run, out, logits = _layer(monkeypatch, 1, T=512)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run()
    assert _joint(ctx) == [True], "the launches under test"
    for i in range(4):
        logits.copy_(torch.roll(logits, 7, 1))
        run()
        torch.cuda.synchronize()
        want = out.clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert want.any() and torch.equal(out.view(torch.int16), want.view(torch.int16)), f"replay {i}"
    ctx.destroy()


def test_without_a_context(monkeypatch):
    """moe_ep_forward_noalloc, at a size that makes one launch of both projections by rule."""
    import paper_2512_21487_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count > 256:
        pytest.skip("512 tiles are not two rounds here")
    M, H, E, T, k = 1024, 512, 128, 1500, 4
    gen = torch.Generator(device="cuda").manual_seed(85)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    layer = dict(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=0, shared_inter=0, max_tokens=T, max_top_k=k, max_chunks=2)
    ctx = _ctx(monkeypatch, lambda: pkg.MoeEp(**layer), 0)
    by_rule = pkg.MoeEp(**layer)
    cfg = pkg.MoeEpConfig(local_begin=0, io_mode=pkg.IO_DEVICE, device=0, **layer)
    want, got = (torch.zeros(T * M, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    for r in (1, 2):
        ctx.forward(tokens, logits, routed, None, k, r, 0, n_tokens=T, out=want)
        pkg.forward_noalloc(cfg, tokens, logits, routed, None, k, r, 0, n_tokens=T, out=got)
        torch.cuda.synchronize()
        assert _joint(ctx, r) == [False] * r and want.any() and torch.equal(got.view(torch.int16), want.view(torch.int16)), f"r = {r}"
        by_rule.forward(tokens, logits, routed, None, k, r, 0, n_tokens=T, out=got)
        torch.cuda.synchronize()
        assert _joint(by_rule, r) == [True] * r and torch.equal(got.view(torch.int16), want.view(torch.int16)), f"r = {r}"
    ctx.destroy()
    by_rule.destroy()


@pytest.mark.parametrize("n_tokens,prepared,tile_rows", [(224, True, 64), (240, True, 192), (240, False, 64), (384, True, 192), (400, False, 192)])
def test_narrow_or_one_tiled_launch(monkeypatch, n_tokens, prepared, tile_rows):
    """On both sides of the line between the narrow kernels and one tiled launch: 14 and 15 rows per expert, 24 and 25 with weights as the
    caller holds them.  The bits do not depend on it."""
    import paper_2512_21487_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count > 320:
        pytest.skip("640 tiles are not two rounds here")
    M, H, E, k = 512, 576, 128, 8
    gen = torch.Generator(device="cuda").manual_seed(86)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(n_tokens * M, 1.0), normal(E * 3 * H * M, 0.02)
    logits = torch.empty((n_tokens, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    outs = []
    for env in ({}, {"MOE_EP_GEMM_VARIANT": "21"}):
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=0, shared_inter=0, max_tokens=n_tokens, max_top_k=k, max_chunks=1)
        if prepared:
            ctx.prepare_weights(routed, None)
        out = torch.zeros(n_tokens * M, dtype=torch.bfloat16, device="cuda")
        ctx.forward(tokens, logits, routed, None, k, 1, 0, n_tokens=n_tokens, out=out)
        torch.cuda.synchronize()
        if not env:
            assert ctx.last_tile_shape("routed_gate_up_gemm")["rows"] == tile_rows, "the launches under test"
            assert _joint(ctx) == [tile_rows == 192]
        outs.append(out)
        ctx.destroy()
    assert outs[0].any() and torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("r,order", [(1, 0), (1, 1), (2, 0), (2, 1)])
def test_output_that_begins_on_8_bytes(r, order, prepared):
    """The shared experts write into `out` itself, the narrow kernels 8 bytes at a time, the tiled ones 16: between the two lines an `out`
    that begins on 8 bytes stays with the narrow ones, and what neither takes is refused."""
    import paper_2512_21487_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count > 288:
        pytest.skip("576 tiles are not two rounds here")
    M, H, E, k, T = 512, 1088, 64, 6, 200 * r       # 18.75 rows per expert and chunk, nine column tiles
    gen = torch.Generator(device="cuda").manual_seed(87)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed, shared = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02), normal(2 * 3 * 512 * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=2, shared_inter=512, max_tokens=T, max_top_k=k, max_chunks=r)
    if prepared:
        ctx.prepare_weights(routed, shared)
    outs = {}
    for offset, rows in ((0, 192), (4, 64), (8, 192), (12, 64)):
        flat = torch.full((T * M + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
        out = flat[offset:offset + T * M]
        ctx.forward(tokens, logits, routed, shared, k, r, order, n_tokens=T, out=out)
        torch.cuda.synchronize()
        assert ctx.last_tile_shape("routed_gate_up_gemm")["rows"] == rows, f"the launches under test, offset {offset}"
        assert _joint(ctx) == [rows == 192]
        outs[offset] = out.view(torch.int16).cpu()
        assert bool((flat[:offset] == 7.0).all()) and bool((flat[offset + T * M:] == 7.0).all())
    assert outs[0].any() and all(torch.equal(o, outs[0]) for o in outs.values())
    flat = torch.zeros(T * M + 8, dtype=torch.bfloat16, device="cuda")
    for args, out in (((tokens, logits), flat[2:2 + T * M]), ((flat[4:4 + T * M], logits), torch.zeros_like(tokens))):
        with pytest.raises(pkg.MoeEpError):
            ctx.forward(*args, routed, shared, k, r, order, n_tokens=T, out=out)
    torch.cuda.synchronize()
    ctx.destroy()


def test_a_small_call_of_a_context_for_large_ones():
    """A context whose largest call has more row tiles than there are counters for still runs a small one as any other context does."""
    import paper_2512_21487_amd as pkg
    if torch.cuda.get_device_properties(0).multi_processor_count > 320:
        pytest.skip("640 tiles are not two rounds here")
    M, H, E, k, T = 128, 576, 128, 8, 240      # 15 rows per expert: past the line only where both projections are one launch
    gen = torch.Generator(device="cuda").manual_seed(88)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(T * M, 1.0), normal(E * 3 * H * M, 0.02)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    outs = []
    for most in (T, 1 << 18):
        ctx = pkg.MoeEp(hidden=M, inter=H, n_experts=E, n_local=E, n_shared=0, shared_inter=0, max_tokens=most, max_top_k=k, max_chunks=1)
        ctx.prepare_weights(routed, None)
        out = torch.zeros(T * M, dtype=torch.bfloat16, device="cuda")
        ctx.forward(tokens, logits, routed, None, k, 1, 0, n_tokens=T, out=out)
        torch.cuda.synchronize()
        assert ctx.last_tile_shape("routed_gate_up_gemm")["rows"] == 192 and _joint(ctx) == [True], "the launches under test"
        outs.append(out.view(torch.int16))
        ctx.destroy()
    assert outs[0].any() and torch.equal(*outs)


def _wide(n_tokens=900, hidden=320):
    """A few experts and shared ones whose tiles are more than the workgroups of a launch."""
    wl = tiny_workload(name="pair_wide", n_tokens=n_tokens, hidden=hidden, inter=1088, n_experts=70, local_begin=3, n_local=64, top_k=3, n_shared=2,
                       shared_inter=192)
    return wl, make_inputs(wl, seed=89)


@pytest.mark.parametrize("prepared", [False, True])
def test_chunks_from_host_memory(monkeypatch, prepared):
    """Workgroups fewer by those that leave their compute units to the next chunk's transfer."""
    import gpu_util as g
    wl, inp = _wide()
    outs = []
    for pair, pinned in ((0, False), (1, True)):
        ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl, pinned=pinned), pair, MOE_EP_MERGE="1")
        d = g.DeviceInputs(wl, inp, pinned=pinned)
        if prepared:
            ctx.prepare_weights(d.routed, d.shared)
        outs.append([])
        for r, order in ((2, 0), (2, 1), (4, 1)):
            outs[-1].append(g.run_forward(ctx, wl, d, r=r, order=order))
            assert _joint(ctx, r) == [bool(pair)] * r and ctx.last_shared_beside(), "the launches under test"
        ctx.destroy()
    assert outs[0][0].any() and all(np.array_equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("pinned", [False, True])
def test_in_the_disaggregated_schedule(monkeypatch, pinned):
    """moe_ep_forward_dep: the shared experts' launches run on another stream beside the joint ones."""
    import gpu_util as g
    wl, inp = _wide()
    outs = []
    for pair in (0, 1):
        ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl, pinned=pinned), pair)
        d = g.DeviceInputs(wl, inp, pinned=pinned)
        outs.append([])
        for r_1, r_2, order in ((1, 1, 0), (2, 2, 0), (2, 2, 1)):
            outs[-1].append(g.run_forward_dep(ctx, wl, d, r_1, r_2, order, 20.0))
            assert _joint(ctx, r_1 * r_2) == [bool(pair)] * (r_1 * r_2), "the launches under test"
        ctx.destroy()
    assert outs[0][0].any() and all(np.array_equal(a, b) for a, b in zip(*outs))


def test_rows_that_are_not_numbers(monkeypatch):
    """NaN and infinite token rows: the bits of a launch of each, and the other tokens' results untouched."""
    import gpu_util as g
    wl, inp = _wide()
    outs = []
    for bad in (False, True):
        if bad:
            inp["tokens"][5], inp["tokens"][400, 7], inp["tokens"][899, ::2] = 0x7fc0, 0x7f80, 0xff80   # NaN, +inf, -inf
        for pair in (0, 1):
            ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl), pair, MOE_EP_MERGE="1")
            outs.append(g.run_forward(ctx, wl, g.DeviceInputs(wl, inp)))
            assert _joint(ctx) == [bool(pair)], "the launches under test"
            ctx.destroy()
    assert outs[0].any() and np.array_equal(outs[0], outs[1]) and np.array_equal(outs[2], outs[3])
    other = np.setdiff1d(np.arange(wl.n_tokens), [5, 400, 899])
    assert np.array_equal(outs[2][other], outs[0][other])
    assert all(((outs[2][t] & 0x7f80) == 0x7f80).any() for t in (5, 400, 899)), "what is not finite stays so"


def test_timed_and_untimed_forwards_of_one_context(monkeypatch):
    """A projection that is timed is a launch of its own; the forwards before and behind it are not changed by that."""
    import gpu_util as g
    wl, inp = _wide()
    ctx = _ctx(monkeypatch, lambda: g.make_ctx(wl), 1, MOE_EP_MERGE="1")
    d = g.DeviceInputs(wl, inp)
    want = g.run_forward(ctx, wl, d, r=2, order=1)
    for stages, joint in ((["routed_gate_up_gemm"], False), (["aggregation"], True), (["routed_down_gemm"], False), (None, False)):
        ctx.set_profiling_stages(stages)
        ctx.set_profiling(1)
        for now in (joint, True):    # the forward that is timed, and one behind the last that is
            assert np.array_equal(g.run_forward(ctx, wl, d, r=2, order=1), want)
            assert _joint(ctx, 2) == [now] * 2, stages
        ctx.set_profiling(0)
    assert want.any()
    ctx.destroy()
