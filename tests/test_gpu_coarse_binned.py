"""The coarse step's two routes for the grid gradients, sorted records with a
vertex gather and float atomics, on the same inputs: the workspace given
decides (dvgo_coarse_step_workspace_bytes or dvgo_coarse_workspace_bytes).
Sizes at the edges: one ray, ragged batches, rays of more than the four
64-sample steps whose values are cached, a truncated sample list, Morton
order, a box of unequal sides, and gradients accumulated onto existing ones.

Both sum the same float32 terms in different orders: n terms at a vertex
differ by at most n 2^-24 of their absolute sum, a few 1e-6 of the largest
entry at the tens of samples per vertex here; 1e-5 normwise and 3e-5 of the
largest entry.  Loss and colour come from the same kernel code: 1e-6."""

import numpy as np
import pytest

import synth
from tests.helpers import assert_close, np_of, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rays,morton,cap", [
    ((24, 24, 24), 1, False, None), ((24, 24, 24), 333, True, None), ((160, 160, 160), 257, False, None),
    ((33, 20, 41), 1000, False, None), ((24, 24, 24), 500, False, 7777), ((2, 2, 2), 64, False, None)])
def test_binned_route_matches_atomics(gpu_lib, monkeypatch, n, rays, morton, cap):
    import torch
    from paper_2111_11215_amd import api
    lib = api.load()
    rng = np.random.default_rng(rays)
    dens = to_dev(rng.uniform(-3, 3, n).astype(np.float32))
    rgb = to_dev(rng.uniform(-2, 2, n + (3,)).astype(np.float32))
    o, d, *_ = synth.draw_pixels_with_replacement(rng, synth.hemisphere_cameras(20, 1), 800, 800, 1000.0, rays)
    step = 1.0 / (max(n) - 1)
    ms = int(np.ceil(2 * np.sqrt(3) / step)) + 1
    s = api.sample_rays(to_dev(o), to_dev(d), to_dev(rng.random(rays).astype(np.float32)), synth.BOX_MIN,
                        synth.BOX_MAX, step, ms, morton=morton, capacity=cap)
    tgt = to_dev(rng.random((rays, 3)).astype(np.float32))
    g0, c0 = rng.normal(size=n).astype(np.float32) * 1e-4, rng.normal(size=n + (3,)).astype(np.float32) * 1e-4

    def step_once():
        gd, gc = to_dev(g0), to_dev(c0)
        loss, out = api.coarse_step(dens, rgb, synth.BOX_MIN, synth.BOX_MAX, 0.2, s, tgt, gd, gc, ms, want_rgb=True)
        return [np_of(t) for t in (loss, out, gd, gc)]

    binned = step_once()
    monkeypatch.setattr(lib, "dvgo_coarse_step_workspace_bytes", lambda B, c, b: lib.dvgo_coarse_workspace_bytes(B))
    atomic = step_once()
    assert_close("loss", binned[0], atomic[0], 1e-6)
    assert_close("rgb", binned[1], atomic[1], 1e-6)
    for name, a, b, start in (("grad_density", binned[2], atomic[2], g0), ("grad_rgb", binned[3], atomic[3], c0)):
        assert np.abs(b - start).max() > 0
        assert_close(name, a, b, 1e-5, 3e-5)
