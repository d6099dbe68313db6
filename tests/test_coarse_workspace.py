"""Which form of the coarse step's gradient sums the workspace query asks for:
float atomics (a few bytes per ray) for small batches and for those whose
sorted records would take more than 1 GiB."""

import ctypes

import pytest


def _lib():
    from paper_2111_11215_amd import _lib
    return _lib, _lib.load()


def _bytes(B, capacity, n):
    mod, lib = _lib()
    box = mod.make_box((-1, -1, -1), (1, 1, 1), (n, n, n))
    return lib.dvgo_coarse_step_workspace_bytes(B, capacity, ctypes.byref(box)), lib.dvgo_coarse_workspace_bytes(B)


@pytest.mark.parametrize("rays,slots,n", [
    (0, 0, 100), (1, 344, 100), (256, 137, 40), (256, 344, 100), (256, 441, 128), (512, 344, 160),   # small batches
    (1 << 20, 344, 100), (65536, 344, 100), (1 << 23, 255, 100), (8192, 1 << 18, 256)])              # large ones
def test_atomic_form(rays, slots, n):
    want, small = _bytes(rays, rays * slots, n)
    assert want == small


@pytest.mark.parametrize("rays,slots,n", [(1024, 137, 40), (1024, 344, 100), (1024, 441, 128), (8192, 344, 100),
                                          (12288, 441, 128), (32768, 344, 100)])
def test_sorted_form(rays, slots, n):
    want, small = _bytes(rays, rays * slots, n)
    assert 72 * rays * slots + 8 * (n - 1) ** 3 <= want - small <= min(1 << 30, 72 * rays * slots + 9 * (n - 1) ** 3 + 4096)


def test_invalid_arguments():
    mod, lib = _lib()
    assert lib.dvgo_coarse_step_workspace_bytes(8, 100, None) == 0
    box = mod.make_box((-1, -1, -1), (1, 1, 1), (1, 4, 4))
    assert lib.dvgo_coarse_step_workspace_bytes(8, 100, ctypes.byref(box)) == 0
