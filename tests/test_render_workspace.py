"""The workspace of a render's backward by precision: the branch bits of the
float32 network's adjoint (32 bytes per slot) are asked of its callers only."""

import ctypes

import pytest

SLOTS = 1 << 22
OK, CAPACITY = 0, -4


def _call(precision, nbytes):
    """dvgo_render_bwd without rays (nothing is launched) on a workspace of
    nbytes; precision None: no network."""
    from paper_2111_11215_amd import _lib
    lib = _lib.load()
    f = _lib.Field()
    f.density = f.feat = 16
    f.channels = 12
    f.box = _lib.make_box((-1, -1, -1), (1, 1, 1), (4, 4, 4))
    m = _lib.Mlp()
    for nm in ("w1", "b1", "w2", "b2", "w3", "b3"):
        setattr(m, nm, 16)
    m.hidden = 128
    m.precision = precision or 0
    fake, nul, bg = ctypes.c_void_p(16), None, (ctypes.c_float * 3)(1, 1, 1)
    return lib.dvgo_render_bwd(ctypes.byref(f), None if precision is None else ctypes.byref(m), fake, fake, nul, fake,
                               fake, fake, fake, fake, fake, fake, SLOTS, 0, 0.1, bg, fake, nul, nul, nul, fake, fake,
                               fake, fake, nbytes, nul)


def _sizes(slots):
    from paper_2111_11215_amd import _lib
    lib = _lib.load()
    box = _lib.make_box((-1, -1, -1), (1, 1, 1), (4, 4, 4))
    return [fn(0, slots, 12, ctypes.byref(box)) for fn in (lib.dvgo_render_workspace_bytes,
                                                           lib.dvgo_render_bf16_workspace_bytes)]


def test_bytes_per_slot():
    (f1, b1), (f2, b2) = _sizes(SLOTS), _sizes(2 * SLOTS)
    assert f2 - f1 == 188 * SLOTS and b2 - b1 == 156 * SLOTS


@pytest.mark.parametrize("precision,short", [(0, CAPACITY), (1, OK), (None, OK)])
def test_smaller_workspace(precision, short):
    full, small = _sizes(SLOTS)
    assert _call(precision, full) == OK
    assert _call(precision, small) == short
    assert _call(precision, small - 1) == CAPACITY
