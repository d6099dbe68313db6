"""Coarse steps of several streams accumulate into the same gradients.

Each call adds its sums with float atomics, so calls that overlap lose
nothing.  Two halves of a batch on two streams, several times over, against
the same calls one after the other; equal up to the order of the sums (2 x 8
additions per entry on top of the route's own: 1e-5 normwise, 3e-5 of the
largest entry, as in test_gpu_coarse_binned)."""

import numpy as np
import pytest

import synth
from tests.helpers import assert_close, np_of, to_dev

pytestmark = pytest.mark.gpu


def test_two_streams_share_the_gradients(gpu_lib):
    import torch
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(0)
    n, rays, reps = (64, 64, 64), 1500, 8
    dens = to_dev(rng.uniform(-3, 3, n).astype(np.float32))
    rgb = to_dev(rng.uniform(-2, 2, n + (3,)).astype(np.float32))
    step = 1.0 / 63
    ms = int(np.ceil(2 * np.sqrt(3) / step)) + 1
    parts = []
    for _ in range(2):
        o, d, *_ = synth.draw_pixels_with_replacement(rng, synth.hemisphere_cameras(20, 1), 800, 800, 1000.0, rays)
        s = api.sample_rays(to_dev(o), to_dev(d), to_dev(rng.random(rays).astype(np.float32)), synth.BOX_MIN,
                            synth.BOX_MAX, step, ms)
        parts.append((s, to_dev(rng.random((rays, 3)).astype(np.float32))))

    def run(streams):
        gd, gc = torch.zeros(n, device="cuda"), torch.zeros(n + (3,), device="cuda")
        torch.cuda.synchronize()
        for _ in range(reps):
            for st, (s, tgt) in zip(streams, parts):
                with torch.cuda.stream(st):
                    api.coarse_step(dens, rgb, synth.BOX_MIN, synth.BOX_MAX, 0.2, s, tgt, gd, gc, ms)
        torch.cuda.synchronize()
        return np_of(gd), np_of(gc)

    one = torch.cuda.current_stream()
    want = run([one, one])
    got = run([torch.cuda.Stream(), torch.cuda.Stream()])
    for name, a, b in zip(("grad_density", "grad_rgb"), got, want):
        assert_close(name, a, b, 1e-5, 3e-5)
