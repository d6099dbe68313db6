"""An infinite gradient of one sample reaches its own eight vertices only, as
an infinity: the vertex sums pad their record lists, and nothing of a listed
record may come back through the padding (0 x infinity is NaN).

One sample per ray strictly inside its cell, so that every weight is positive;
dL/dacc of some rays is infinite, and opacity's gradient at a ray's only sample
is dL/dacc T_after step sigmoid, of one sign.  Finite vertices within 1e-5 of the
float64 sum."""

import numpy as np
import pytest

from tests.helpers import assert_close, np_of, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rays,n", [(1, 3), (7, 5), (300, 5), (300, 17)])
def test_infinite_density_gradient(gpu_lib, rays, n):
    import torch
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(rays + n)
    per = 128 // (n - 1)                                        # 64ths of a unit per cell
    q = rng.integers(0, (n - 1), (rays, 3)) * per + rng.integers(1, per, (rays, 3))
    z = q[:, 2] / 64.0
    o = np.stack([-1 + q[:, 0] / 64, -1 + q[:, 1] / 64, np.full(rays, -2.0)], axis=1).astype(np.float32)
    d = np.tile(np.array([0, 0, 1], np.float32), (rays, 1))
    step = 2.0
    s = api.sample_rays(to_dev(o), to_dev(d), to_dev((z / step).astype(np.float32)), (-1.0,) * 3, (1.0,) * 3, step, 1)
    assert int(s.n_kept.item()) == rays
    gA = rng.uniform(0.5, 1.5, rays).astype(np.float32)
    gA[rng.choice(rays, max(1, rays // 60), replace=False)] = np.inf
    shift = 0.25
    grid = api.Grid(torch.zeros((n, n, n), device="cuda"), torch.zeros((n, n, n, 12), device="cuda"), (-1.0,) * 3,
                    (1.0,) * 3, shift)
    out = api.render_fwd(grid, None, s)
    gd = torch.zeros_like(grid.density)
    api.render_bwd(grid, None, s, out["log_t_end"], None, gd, None, None, grad_acc=to_dev(gA))
    sig = np.log1p(np.exp(shift))
    draw = gA.astype(np.float64) * np.exp(-sig * step) * step / (1 + np.exp(-shift))
    ref = np.zeros((n, n, n))
    i0, f = q // per, (q % per) / per
    for c in range(8):
        b = np.array([c >> 2 & 1, c >> 1 & 1, c & 1])
        np.add.at(ref, tuple((i0 + b).T), np.prod(np.where(b, f, 1 - f), axis=1) * draw)
    got = np_of(gd)
    assert np.array_equal(np.isinf(ref), np.isinf(got)) and not np.isnan(got).any()
    ok = np.isfinite(ref)
    if ref[ok].any():
        assert_close("grad_density", got[ok], ref[ok], 1e-5)
