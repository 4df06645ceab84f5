"""Host-only checks of the kernels' launchers: what they refuse before anything is launched (no GPU is used)."""
import ctypes
import os

import pytest

import paper_2512_21487_amd as pkg

# the pointers are made up: a launch that is not refused must find no GPU to run on
pytestmark = pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="host-only checks")

INVALID_VALUE = 1   # hipErrorInvalidValue


class GemmArgs(ctypes.Structure):   # csrc/kernels.h
    _fields_ = [("A", ctypes.c_void_p), ("W", ctypes.c_void_p), ("C", ctypes.c_void_p), ("offset", ctypes.c_void_p),
                *((n, ctypes.c_int) for n in ("G", "dense_rows", "K", "N", "lda", "ldc", "ldw")),
                ("w_group_stride", ctypes.c_longlong), ("w_up_offset", ctypes.c_longlong), ("kseg_len", ctypes.c_int),
                ("w_kseg_stride", ctypes.c_longlong), ("c_group_col_stride", ctypes.c_int), ("a_row_map", ctypes.c_void_p),
                ("a_row_div", ctypes.c_int), ("a_src_rows", ctypes.c_int), ("max_units", ctypes.c_int), ("epi", ctypes.c_int),
                ("row_weight", ctypes.c_void_p), ("row_assignment", ctypes.c_void_p), ("Wp", ctypes.c_void_p)]


class GateArgs(ctypes.Structure):
    _fields_ = [("scores", ctypes.c_void_p), *((n, ctypes.c_int) for n in ("Tn", "E", "k", "e0")),
                *((n, ctypes.c_void_p) for n in ("idx", "w", "count", "offset", "pos", "perm"))]


@pytest.mark.parametrize("max_tokens,dense_rows", [(4, 17), (4, 64), (17, 4), (33, 4), (3, 4)])
def test_a_gate_inside_a_launch_without_one_is_refused(max_tokens, dense_rows):
    """The gate/up projection routes by itself in tiles of one block of 16 rows only: asked to in any other tile (or with
    more tokens than its groups can have rows), the launch must not run without the gate."""
    launch = pkg.load_library()._ZN6moe_ep18launch_narrow_gemmERKNS_8GemmArgsEPS1_bidixP12ihipStream_tPiPKNS_8GateArgsE
    M, H, k, A = 2048, 1408, 6, 0x1000
    routed = GemmArgs(A=A, W=A, C=A, offset=A, G=64, K=M, N=H, lda=M, ldc=H, ldw=M, w_group_stride=3 * H * M, w_up_offset=H * M, kseg_len=M,
                      a_row_map=A, a_row_div=k, a_src_rows=max_tokens)
    shared = GemmArgs(A=A, W=A, C=A, G=2, dense_rows=dense_rows, K=M, N=H, lda=M, ldc=2 * H, ldw=M, w_group_stride=3 * H * M, w_up_offset=H * M,
                      kseg_len=M, c_group_col_stride=H)
    gate = GateArgs(scores=A, Tn=4, E=64, k=k, e0=0, idx=A, w=A, count=A, offset=A, pos=A, perm=A)
    kind = ctypes.c_int()
    rc = launch(ctypes.byref(routed), ctypes.byref(shared), ctypes.c_bool(True), 256, ctypes.c_double(max_tokens * k / 64), max_tokens,
                ctypes.c_longlong(max_tokens * k), None, ctypes.byref(kind), ctypes.byref(gate))
    assert rc == INVALID_VALUE


def test_compute_units_left_to_the_link():
    """A sixteenth of the device at most, whatever its size: a launch beside a copy always has some."""
    beside = pkg.load_library()._ZN6moe_ep17units_beside_linkEi
    assert [beside(n) for n in (256, 304, 64, 32, 16, 8, 1)] == [240, 288, 60, 30, 15, 8, 1]


@pytest.mark.parametrize("tokens,top_k,local,inter,inside", [
    (1, 6, 64, 1408, True), (4, 6, 64, 1408, True), (4, 6, 20, 1536, True), (4, 8, 16, 1536, True), (4, 8, 128, 768, True),
    (4, 64, 64, 64, True),         # many rounds, a tile in four compute units
    (1, 64, 64, 1536, False),      # many rounds, six tiles on every compute unit
    (4, 33, 128, 1536, False),
    (4, 33, 16, 1536, True),       # few experts here
    (1, 33, 32, 7168, False),      # few, but many columns
    (4, 16, 256, 7168, False),
    (1, 8, 8, 4096, True),
])
def test_gate_of_many_rounds_takes_a_launch_of_its_own(tokens, top_k, local, inter, inside):
    pays = pkg.load_library()._ZN6moe_ep16narrow_gate_paysEiiiii
    pays.restype = ctypes.c_bool
    assert pays(tokens, top_k, local, inter, 256) == inside


@pytest.mark.parametrize("experts,chunks,shared_first,with_gate", [
    (256, 1, False, True), (256, 1, True, True), (256, 2, False, True), (256, 2, True, False), (257, 1, False, False), (512, 4, True, False)])
def test_first_chunk_comes_in_with_the_gate(experts, chunks, shared_first, with_gate):
    rule = pkg.load_library()._ZN6moe_ep19rows_come_with_gateEiib
    rule.restype = ctypes.c_bool
    assert rule(experts, chunks, ctypes.c_bool(shared_first)) == with_gate


@pytest.mark.parametrize("up,down,counters,refused", [
    (True, False, False, False), (False, True, False, False),   # a launch of one projection deals its tiles
    (True, True, False, True), (True, True, True, False)])
def test_counters_are_for_launches_of_both_projections(up, down, counters, refused):
    launch = pkg.load_library()._ZN6moe_ep18launch_loader_gemmEPKNS_8GemmArgsES2_S2_S2_iPiP12ihipStream_t
    M, H, A = 1024, 512, 0x1000
    gate_up = GemmArgs(A=A, W=A, C=A, offset=A, G=8, K=M, N=H, lda=M, ldc=H, ldw=M, w_group_stride=3 * H * M, w_up_offset=H * M, kseg_len=M)
    out = GemmArgs(A=A, W=A, C=A, offset=A, G=8, K=H, N=M, lda=H, ldc=M, ldw=H, w_group_stride=3 * H * M, kseg_len=H)
    rc = launch(ctypes.byref(gate_up) if up else None, None, ctypes.byref(out) if down else None, None, 256, ctypes.c_void_p(A if counters else None), None)
    assert rc != 0 and (rc == INVALID_VALUE) == refused
