"""Down projection and weighted sum of at most 16 tokens in one launch (narrow_gemm.hip): the bits of the tiled kernels and the
aggregation, which the oracle tests pin, where its staged K steps, its list of experts and its columns begin and end."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("hidden,inter,n_experts,local_begin,n_local,top_k,n_shared,shared_inter", [
    (64, 512, 4, 1, 1, 1, 0, 0),           # a tile that ends after 64 columns; most tokens keep nothing
    (320, 768, 24, 4, 3, 3, 0, 0),         # as many K steps as can be in flight; columns past one tile
    (192, 832, 24, 4, 3, 3, 2, 512),       # one more; shared experts in one reduction, more than half of the tokens on them alone
    (256, 704, 130, 0, 130, 8, 1, 768),    # one less; more experts than a wavefront lists at once, more than there are wavefronts
    (64, 1344, 70, 5, 64, 64, 3, 512),     # every slot a lane can hold
    (4096, 512, 8, 2, 4, 3, 1, 576),       # 16 columns per workgroup
    (4160, 640, 8, 2, 4, 3, 0, 0),         # more workgroups than compute units: 4 tokens at most
])
def test_same_bits_as_separate_launches(monkeypatch, hidden, inter, n_experts, local_begin, n_local, top_k, n_shared, shared_inter, prepared,
                                        pinned):
    import gpu_util as g
    import paper_2512_21487_amd as pkg
    wl = tiny_workload(name=f"sum_M{hidden}", n_tokens=33, hidden=hidden, inter=inter, n_experts=n_experts, local_begin=local_begin,
                       n_local=n_local, top_k=top_k, n_shared=n_shared, shared_inter=shared_inter)
    inp = make_inputs(wl, seed=91)
    inp["gate_logits"][::3, local_begin] += 20.0     # an expert that every third token chooses
    d = g.DeviceInputs(wl, inp)
    shared = d.shared if n_shared else None

    def run(narrow_rows):
        with monkeypatch.context() as m:
            m.setenv("MOE_EP_NARROW_ROWS", narrow_rows)
            ctx = pkg.MoeEp(hidden=hidden, inter=inter, n_experts=n_experts, local_begin=local_begin, n_local=n_local, n_shared=n_shared,
                            shared_inter=shared_inter, max_tokens=33, max_top_k=top_k, max_chunks=3,
                            io_mode=pkg.IO_PINNED_HOST if pinned else pkg.IO_DEVICE)
        if prepared:
            ctx.prepare_weights(d.routed, shared)
        outs = {}
        for n, r, order in ((1, 1, 0), (4, 1, 1), (16, 1, 0), (17, 1, 0), (31, 2, 0), (33, 3, 1)):
            tokens, scores = (x.reshape(33, -1)[:n].contiguous() for x in (d.tokens, d.logits))
            out = torch.full((n, hidden), 7.0, dtype=tokens.dtype, device="cpu" if pinned else "cuda", pin_memory=pinned)
            if pinned:
                tokens, scores = tokens.cpu().pin_memory(), scores.cpu().pin_memory()
            ctx.forward(tokens, scores, d.routed, shared, top_k, r, order, out=out)
            torch.cuda.synchronize()
            outs[n, r] = out.cpu().view(torch.int16).numpy().copy(), ctx.last_tile_shape("routed_down_gemm")["waves_n"]
        ctx.destroy()
        return outs

    want, got = run("0"), run("1e9")
    for case, (w, _) in want.items():
        assert np.array_equal(got[case][0], w), case
    assert want[33, 3][0].any()
    most = 16 if hidden <= 4096 else 4
    for (n, r), (_, waves) in got.items():
        # in several chunks with the shared experts of all of them first, the aggregation adds to rows that are already there
        assert (waves == 8) == (-(-n // r) <= most and not (r == 2 and n_shared)), (n, r)


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("offset", [1, 2, 3, 4])
def test_output_that_begins_anywhere(offset, pinned):
    """`out` at `offset` elements behind a 16-byte boundary: the rows of one that begins on it, and nothing beside them."""
    import gpu_util as g
    import paper_2512_21487_amd as pkg
    wl = tiny_workload(name="sum_offset", n_tokens=16, hidden=192, inter=512, n_experts=6, local_begin=1, n_local=4, top_k=2, n_shared=0,
                       shared_inter=0)
    inp = make_inputs(wl, seed=92)
    d = g.DeviceInputs(wl, inp, pinned=pinned)
    ctx = g.make_ctx(wl, pinned=pinned)
    for n in (1, 16):
        want = g.run_forward(ctx, wl, d, n_tokens=n)
        assert ctx.last_tile_shape("routed_down_gemm")["waves_n"] == 8, "the launch under test"
        flat = torch.full((n * wl.hidden + 8,), 7, dtype=torch.int16, device="cpu" if pinned else "cuda", pin_memory=pinned)
        out = flat[offset:offset + n * wl.hidden]
        ctx.forward(d.tokens, d.logits, d.routed, None, wl.top_k, 1, 0, n_tokens=n, out=out)
        torch.cuda.synchronize()
        assert (ctx.last_tile_shape("routed_down_gemm")["waves_n"] == 8) == (offset % 2 == 0)
        assert np.array_equal(out.cpu().numpy().view(np.uint16).reshape(n, -1), want) and want.any()
        rest = flat.cpu().numpy()
        assert (rest[:offset] == 7).all() and (rest[offset + n * wl.hidden:] == 7).all()
    ctx.destroy()


@pytest.mark.parametrize("hidden,inter,n_experts,top_k,n_tokens,one", [
    (64, 1408, 8, 2, 4, True),
    (64, 1408, 128, 33, 2, False),         # eight workgroups would draw the weights of 58 experts
    (512, 1024, 64, 64, 4, False),
    (512, 1024, 8, 2, 9, True),
    (1024, 2880, 64, 64, 9, False),
    (2048, 1024, 64, 6, 16, True),         # a workgroup per compute unit
])
def test_few_columns_of_many_experts_take_launches_of_their_own(hidden, inter, n_experts, top_k, n_tokens, one):
    import paper_2512_21487_amd as pkg
    gen = torch.Generator(device="cuda").manual_seed(93)
    normal = lambda n, std: torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    tokens, routed = normal(n_tokens * hidden, 1.0), normal(n_experts * 3 * inter * hidden, 0.02)
    scores = torch.empty((n_tokens, n_experts), dtype=torch.float32, device="cuda").normal_(generator=gen)
    out = torch.zeros(n_tokens * hidden, dtype=torch.bfloat16, device="cuda")
    ctx = pkg.MoeEp(hidden=hidden, inter=inter, n_experts=n_experts, n_local=n_experts, max_tokens=n_tokens, max_top_k=top_k, max_chunks=1)
    ctx.forward(tokens, scores, routed, None, top_k, n_tokens=n_tokens, out=out)
    torch.cuda.synchronize()
    assert (ctx.last_tile_shape("routed_down_gemm")["waves_n"] == 8) == one and out.any()
    ctx.destroy()
