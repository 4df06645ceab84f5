"""The projections of chunks with few rows per expert (narrow_gemm.hip): the bits of the tiled kernels, which the
oracle tests pin, on every row count and column or K remainder where a tile, a staged chunk or a ring can go wrong."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# rows of the experts: none, one, around a block of 16, around a row tile of 64, several tiles with a remainder
LOADS = [0, 1, 15, 16, 17, 0, 33, 63, 64, 65, 129, 200]


def _env(monkeypatch, rows):
    monkeypatch.setenv("MOE_EP_NARROW_ROWS", str(rows))


def _exact_loads(wl, inp):
    lg = np.full((wl.n_tokens, wl.n_experts), -30.0, dtype=np.float32)
    t = 0
    for e, n in enumerate(LOADS):
        lg[t:t + n, e] = 5.0
        t += n
    inp["gate_logits"][:] = lg[np.random.default_rng(7).permutation(wl.n_tokens)]


def _run(monkeypatch, wl, inp, rows, what=(), calls=((1, 0),), pinned=False):
    """Output bits of the calls (r, order) with the narrow kernels up to `rows` rows per expert (0: never)."""
    import gpu_util as g
    _env(monkeypatch, rows)
    ctx = g.make_ctx(wl, pinned=pinned)
    d = g.DeviceInputs(wl, inp, pinned=pinned)
    if what:
        ctx.prepare_weights(d.routed if "routed" in what else None, d.shared if "shared" in what else None)
    outs = [g.run_forward(ctx, wl, d, r=r, order=order) for r, order in calls]
    narrow = ctx.last_tile_shape("routed_gate_up_gemm")["rows"] == 64
    assert not (narrow and rows == 0), "the tiled kernels are the reference"
    ctx.destroy()
    return outs, narrow


@pytest.mark.parametrize("what", [(), ("routed", "shared"), ("routed",), ("shared",)])
@pytest.mark.parametrize("hidden,inter,shared_inter", [(64, 64, 64), (192, 128, 192), (256, 320, 64), (320, 576, 320), (576, 448, 128)])
def test_same_bits_as_the_tiled_kernels(monkeypatch, hidden, inter, shared_inter, what):
    """K of 1, 2, 3, 4, 5, 7 and 9 steps of 64, columns that end inside a tile, two shared experts whose K
    segments end inside a staged chunk, weights in either layout and in both at once, and chunks."""
    wl = tiny_workload(name=f"narrow_M{hidden}_H{inter}", n_tokens=sum(LOADS), hidden=hidden, inter=inter, n_experts=12,
                       n_local=12, top_k=1, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=61)
    _exact_loads(wl, inp)
    calls = ((1, 0), (3, 0), (3, 1))
    want, _ = _run(monkeypatch, wl, inp, 0, what, calls)
    got, narrow = _run(monkeypatch, wl, inp, 1e9, what, calls)
    assert narrow and want[0].any()
    for w, o, c in zip(want, got, calls):
        assert np.array_equal(o, w), f"r, order = {c}"


@pytest.mark.parametrize("n_tokens", [1, 2, 16, 63, 300])
@pytest.mark.parametrize("n_shared,what", [(0, ()), (0, ("routed",)), (2, ()), (2, ("routed", "shared"))])
@pytest.mark.parametrize("pinned", [False, True])
def test_small_calls_of_a_share(monkeypatch, n_tokens, pinned, n_shared, what):
    """By the library's own rule: a local share that starts at expert 2 of 70, k = 5, without and with shared experts
    (up to 16 tokens the down projection's tiles are half as wide)."""
    wl = tiny_workload(name=f"narrow_share_{n_tokens}", n_tokens=n_tokens, hidden=192, inter=320, n_experts=70,
                       local_begin=2, n_local=66, top_k=5, n_shared=n_shared, shared_inter=192 if n_shared else 0)
    inp = make_inputs(wl, seed=62)
    calls = ((1, 0), (2, 0))
    want, _ = _run(monkeypatch, wl, inp, 0, what, calls, pinned)
    got, narrow = _run(monkeypatch, wl, inp, 24, what, calls, pinned)
    assert narrow
    for w, o in zip(want, got):
        assert np.array_equal(o, w)


@pytest.mark.parametrize("what", [(), ("routed", "shared")])
@pytest.mark.parametrize("n_tokens,hidden,inter,shared_inter", [
    (1, 192, 64, 64),        # K steps of 64 in the down projection, routed and shared: 1 and 2
    (15, 320, 128, 320),     # 2 and 10: segments of 5, two and a half staged chunks of 4
    (16, 192, 512, 704),     # 8 (the first turn of the steady loop) and 22: segments of 11
    (17, 192, 512, 704),     # the same out of 64-row tiles
    (16, 448, 576, 192),     # 9: the loop and one step; columns that end inside a tile
    (2, 2048, 1088, 576),    # 17, and more column tiles
    (16, 192, 1408, 1408),   # 22 and 44
])
def test_down_projection_of_a_few_tokens(monkeypatch, n_tokens, hidden, inter, shared_inter, what):
    """The 16-row tiles with two wavefronts, from fewer K steps than are staged at once to many turns of the loop over
    both row buffers, shared experts' segments that end inside a staged chunk, weights in either layout."""
    import gpu_util as g
    wl = tiny_workload(name="narrow_few", n_tokens=n_tokens, hidden=hidden, inter=inter, n_experts=12, local_begin=1, n_local=11,
                       top_k=3, n_shared=2, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=66)
    want, _ = _run(monkeypatch, wl, inp, 0, what)
    monkeypatch.delenv("MOE_EP_NARROW_ROWS")
    ctx = g.make_ctx(wl)   # by the library's own rule
    d = g.DeviceInputs(wl, inp)
    if what:
        ctx.prepare_weights(d.routed, d.shared)
    got = g.run_forward(ctx, wl, d)
    few = ctx.last_tile_shape("routed_down_gemm")["rows"] == 16
    assert ctx.last_shared_beside() and few == (n_tokens <= 16)
    ctx.destroy()
    assert want[0].any() and np.array_equal(got, want[0])


def test_most_experts_and_nothing_kept(monkeypatch):
    """512 local experts, 64 per token (several groups of lanes in the kernel's prefix sum); then no token at all
    for the local share."""
    wl = tiny_workload(name="narrow_E512", n_tokens=40, hidden=64, inter=64, n_experts=512, n_local=512, top_k=64)
    inp = make_inputs(wl, seed=63)
    want, _ = _run(monkeypatch, wl, inp, 0)
    got, narrow = _run(monkeypatch, wl, inp, 24)
    assert narrow and np.array_equal(got[0], want[0]) and want[0].any()
    wl = tiny_workload(name="narrow_none", n_tokens=40, hidden=64, inter=64, n_experts=8, local_begin=6, n_local=2, top_k=2)
    inp = make_inputs(wl, seed=64)
    inp["gate_logits"][:, 6:] = -40.0
    got, narrow = _run(monkeypatch, wl, inp, 24)
    assert narrow and not got[0].any()


def _skewed_us(monkeypatch, knobs, *, hidden, inter, n_experts, n_local, top_k, n_tokens, hot, n_shared=0):
    """Microseconds of a forward whose tokens all choose among the first `hot` experts, best of five runs of 20, and its
    output, for each set of environment knobs in turn."""
    import paper_2512_21487_amd as pkg
    gen = torch.Generator(device="cuda").manual_seed(5)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens = normal(n_tokens * hidden, 1.0)
    logits = torch.empty((n_tokens, n_experts), dtype=torch.float32, device="cuda").normal_(generator=gen)
    logits[:, :hot] += 50.0
    routed = normal(n_local * 3 * inter * hidden, 0.02)
    shared = normal(n_shared * 3 * inter * hidden, 0.02) if n_shared else None
    sides = []
    for env in knobs:
        with monkeypatch.context() as m:
            for name, value in env.items():
                m.setenv(name, value)
            ctx = pkg.MoeEp(hidden=hidden, inter=inter, n_experts=n_experts, n_local=n_local, n_shared=n_shared,
                            shared_inter=inter if n_shared else 0, max_tokens=n_tokens, max_top_k=top_k, max_chunks=1)
        ctx.prepare_weights(routed, shared)
        out = torch.zeros(n_tokens * hidden, dtype=torch.bfloat16, device="cuda")
        sides.append((ctx, out, lambda c=ctx, o=out: c.forward(tokens, logits, routed, shared, top_k, 1, 0, n_tokens=n_tokens, out=o)))
    best = [float("inf")] * len(sides)
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(5):
        for i, (_, _, call) in enumerate(sides):
            for _ in range(3):
                call()
            begin.record()
            for _ in range(20):
                call()
            end.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], begin.elapsed_time(end) * 50.0)
    outs = [out for _, out, _ in sides]
    for ctx, _, _ in sides:
        ctx.destroy()
    return best, outs


@pytest.mark.parametrize("n_tokens", [200, 400])
def test_row_tiles_of_one_group_share_its_weights(monkeypatch, n_tokens):
    """Every token on the same six experts: 4 or 7 row tiles read each expert's weights.  Against the tiled kernels, read
    past the caches once per row tile they took 1.73 and 1.83 times as long, shared through L2 1.34 and 1.33 times."""
    (tiled, narrow), outs = _skewed_us(monkeypatch, [{"MOE_EP_NARROW_ROWS": "0"}, {"MOE_EP_NARROW_ROWS": "24"}], hidden=5120, inter=1536,
                                       n_experts=160, n_local=20, top_k=6, n_tokens=n_tokens, hot=6, n_shared=2)
    assert torch.equal(outs[0], outs[1])
    assert narrow < 1.5 * tiled, f"{narrow:.0f} us against {tiled:.0f}"


@pytest.mark.parametrize("n_tokens,top_k,hot", [(384, 8, 8), (384, 8, 16), (1536, 1, 1)])
def test_a_load_far_from_balanced_runs_tall_tiles(monkeypatch, n_tokens, top_k, hot):
    """At most 24 rows per expert on average, but all of them on few: 6 to 24 row tiles would stream each expert's
    weights.  By the mean alone the narrow kernels ran, 1.45, 1.8 and 1.55 times as long as the tiled ones."""
    (tiled, rule), outs = _skewed_us(monkeypatch, [{"MOE_EP_NARROW_ROWS": "0"}, {}], hidden=4096, inter=1536, n_experts=128,
                                     n_local=16, top_k=top_k, n_tokens=n_tokens, hot=hot)
    assert torch.equal(outs[0], outs[1])
    assert rule < 1.2 * tiled, f"{rule:.0f} us against {tiled:.0f}"


def test_the_tile_shape_that_ran_is_reported():
    """moe_ep_last_tile_shape: the tiles of a few tokens' down projection, the 64-row tiles, and the shapes of a call
    without tokens and of a chunk without a token."""
    import gpu_util as g
    wl = tiny_workload(name="narrow_shape", n_tokens=17, hidden=192, inter=320, n_experts=70, n_local=70, top_k=5,
                       n_shared=1, shared_inter=192)
    ctx = g.make_ctx(wl)
    d = g.DeviceInputs(wl, make_inputs(wl, seed=65))
    tile = lambda stage, chunk=0: tuple(ctx.last_tile_shape(stage, chunk)[n] for n in ("rows", "cols", "k_step", "ring_slots", "waves_m", "waves_n"))
    g.run_forward(ctx, wl, d, n_tokens=0)
    assert ctx.last_tile_shape("shared_gate_up_gemm") and ctx.last_tile_shape("shared_down_gemm")
    for n_tokens, down in ((1, (16, 64, 64, 4, 1, 2)), (16, (16, 64, 64, 4, 1, 2)), (17, (64, 128, 64, 4, 1, 4))):
        g.run_forward(ctx, wl, d, n_tokens=n_tokens)
        assert tile("routed_gate_up_gemm") == tile("shared_gate_up_gemm") == (64, 128, 64, 4, 1, 4)
        assert tile("routed_down_gemm") == tile("shared_down_gemm") == down
    g.run_forward(ctx, wl, d, r=4, n_tokens=2)   # two of the four chunks are empty
    for chunk in range(4):
        assert ctx.last_tile_shape("routed_gate_up_gemm", chunk) and ctx.last_tile_shape("routed_down_gemm", chunk)
    ctx.destroy()
