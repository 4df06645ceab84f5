"""The counters of launches of both projections, on the CPU: how many a context has, and a model of the order in which the multiplying
wavefronts of loader_gemm.hip tell that a gate/up tile's activation is in memory: in every interleaving a tile is counted once, behind its
last wavefront."""
import ctypes
import os
import re

import pytest

import paper_2512_21487_amd as pkg

SOURCE = os.path.join(os.path.dirname(pkg.__file__), "csrc", "loader_gemm.hip")


def wavefront(tiles, steps):
    """What a multiplying wavefront does with `tiles` gate/up tiles of `steps` K steps in a row, then a down tile or nothing: None is a
    hand-over, which all wavefronts meet at, a number the tile that it tells of.  A tile's last K step has a hand-over where another gate/up
    tile follows; the tile before is told of behind the K loop, the last one right behind its own."""
    todo = [None]
    for it in range(tiles):
        todo += [None] * (steps if it + 1 < tiles else steps - 1)
        if it > 0:
            todo.append(it - 1)
    return todo + [tiles - 1, None]


def faults(tiles, steps, slots, waves=3):
    """Tiles that some interleaving counts before every wavefront has told of them, or another number of times than once."""
    todo = wavefront(tiles, steps)
    start = ((0,) * waves, (0,) * slots, (0,) * tiles)
    seen, stack, bad = {start}, [start], set()
    while stack:
        at, added, counted = stack.pop()
        if all(i == len(todo) for i in at):
            bad.update(t for t in range(tiles) if counted[t] != 1)
        after = []
        if all(i < len(todo) and todo[i] is None for i in at):
            after.append((tuple(i + 1 for i in at), added, counted))
        for w, i in enumerate(at):
            if i == len(todo) or todo[i] is None:
                continue
            t = todo[i]
            now = at[:w] + (i + 1,) + at[w + 1:]
            last = added[t % slots] % waves == waves - 1
            if last and any(t in todo[j:] for j in now):
                bad.add(t)
            after.append((now, added[:t % slots] + ((added[t % slots] + 1) % waves,) + added[t % slots + 1:],
                          counted[:t] + (counted[t] + last,) + counted[t + 1:]))
        for state in after:
            if state not in seen:
                seen.add(state)
                stack.append(state)
    return bad


@pytest.mark.parametrize("steps", [1, 2, 3])
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 7])
def test_every_tile_is_counted_once_behind_its_last_wavefront(tiles, steps):
    with open(SOURCE) as f:
        source = f.read()
    slots = re.search(r"constexpr int kLdTold = (\d+);", source)
    assert slots and "s_waves + it % kLdTold" in source, "the numbers that tiles take in turn"
    assert not faults(tiles, steps, int(slots.group(1)))


def test_two_numbers_in_turn_are_too_few_for_one_step():
    assert faults(3, 1, 2) and not faults(3, 2, 2)


@pytest.mark.parametrize("max_tokens,top_k,n_local,n_shared,row_tiles", [
    (1, 1, 1, 0, 1), (4096, 6, 64, 2, 192 + 64 + 32), (16384, 8, 4, 0, 512 + 4), (260096, 8, 128, 0, 1 << 14),
    (262144, 8, 128, 0, 1 << 14),      # its largest call has more, its small ones do not
    (1 << 22, 64, 512, 2, 1 << 14)])
def test_a_context_of_any_size_has_counters(max_tokens, top_k, n_local, n_shared, row_tiles):
    count = pkg.load_library()._ZN6moe_ep17context_row_tilesERK13moe_ep_config
    count.restype = ctypes.c_longlong
    cfg = pkg.MoeEpConfig(hidden=64, inter=64, n_experts=512, local_begin=0, n_local=n_local, n_shared=n_shared, shared_inter=64 if n_shared else 0,
                          max_tokens=max_tokens, max_top_k=top_k, max_chunks=1, io_mode=pkg.IO_DEVICE, device=0)
    assert count(ctypes.byref(cfg)) == row_tiles
