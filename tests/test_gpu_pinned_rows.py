"""The first chunk of pinned host rows: the gate's launch brings them in (router.hip), or, where they do not start on 16 bytes, a copy
does; the bits are those of rows that are on the GPU already."""
import numpy as np
import pytest

from workloads import make_inputs, tiny_workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pinned(a, offset=0):
    """`a` in pinned host memory, `offset` elements behind the start of an allocation."""
    flat = torch.empty(a.numel() + offset, dtype=a.dtype, pin_memory=True)
    flat[offset:].copy_(a.reshape(-1))
    return flat[offset:].view(a.shape)


@pytest.mark.parametrize("offset", [0, 2])
@pytest.mark.parametrize("n_shared", [0, 1])
@pytest.mark.parametrize("n_tokens,hidden", [(1, 64), (63, 192), (64, 256), (65, 192), (333, 320), (2100, 1024)])
def test_rows_from_host_memory(monkeypatch, n_tokens, hidden, n_shared, offset):
    """From fewer bytes than one copy workgroup takes at once to many rounds of all of them; shared experts apart and beside."""
    import gpu_util as g
    import paper_2512_21487_amd as pkg
    wl = tiny_workload(name="pinned_rows", n_tokens=n_tokens, hidden=hidden, inter=128, n_experts=20, local_begin=3, n_local=11, top_k=3,
                       n_shared=n_shared, shared_inter=192 if n_shared else 0)
    inp = make_inputs(wl, seed=85)
    d = g.DeviceInputs(wl, inp)
    want = g.run_forward(g.make_ctx(wl), wl, d)
    tokens, logits = _pinned(d.tokens.cpu().reshape(n_tokens, hidden), offset), _pinned(d.logits.cpu().reshape(n_tokens, wl.n_experts), offset // 2)
    for merge in ("0", "1"):
        monkeypatch.setenv("MOE_EP_MERGE", merge)
        ctx = pkg.MoeEp(hidden=hidden, inter=128, n_experts=20, local_begin=3, n_local=11, n_shared=n_shared, shared_inter=192 if n_shared else 0,
                        max_tokens=n_tokens, max_top_k=3, max_chunks=2, io_mode=pkg.IO_PINNED_HOST)
        out = torch.zeros((n_tokens, hidden), dtype=tokens.dtype, pin_memory=True)
        for r in (1, 2, 1):   # and behind a forward whose rows came in on a stream of their own
            out.zero_()
            ctx.forward(tokens, logits, d.routed, d.shared if n_shared else None, 3, r, 0, n_tokens=n_tokens, out=out)
            torch.cuda.synchronize()
            assert np.array_equal(out.numpy().view(np.uint16), want.reshape(n_tokens, hidden)), f"r = {r}"
        ctx.destroy()
    assert want.any()
