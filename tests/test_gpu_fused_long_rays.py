"""The training step's compositing keeps w_k and the optical depth of a ray's
first 512 samples for its adjoint and log T at the starts of its first 64
steps of 64: rays below, beyond and far beyond both, against the separate
forward, loss and backward calls.  Same colour; loss to float32 rounding
(1e-6), network gradient and grid updates to the summation order (1e-5, as in
test_gpu_fused)."""

import numpy as np
import pytest

from tests.helpers import assert_close, np_of, to_dev
from tests.test_gpu_fused import F32, _clone_grid, _state
from tests.test_gpu_render import _gpu, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("samples,n_rays", [(500, 200), (1100, 100), (5000, 24)])
def test_long_rays_fused_equals_separate(gpu_lib, samples, n_rays):
    import torch
    from paper_2111_11215_amd import api
    P = _problem(4, n_rays=n_rays, bias=-4.0)
    P.step = float(np.linalg.norm(np.asarray(P.box_max) - np.asarray(P.box_min))) / samples
    P.max_samples = samples
    grid, flat, s = _gpu(P, morton=False)
    print(f"  {int(s.n_kept.item())} samples, longest ray {int(np_of(s.n_uniform).max())}", flush=True)
    rng = np.random.default_rng(2)
    state = [*_state(rng, P.density.shape), *_state(rng, P.feat.shape)]
    target = to_dev(P.rays.target.astype(F32))
    ga, gb = _clone_grid(api, grid), _clone_grid(api, grid)
    sa, sb = [x.clone() for x in state], [x.clone() for x in state]
    gma, gmb = torch.zeros_like(flat), torch.zeros_like(flat)
    out = api.render_fwd(ga, flat, s, P.bg, want_depth_acc=False)
    loss_a, g = api.photo_loss(out["rgb"], target)
    api.render_bwd_adam(ga, flat, s, out["log_t_end"], g, *sa, gma, 0.1, 3, bg=P.bg)
    loss_b, rgb_b = api.train_step(gb, flat, s, target, *sb, gmb, 0.1, 3, bg=P.bg)
    assert torch.equal(out["rgb"], rgb_b)
    assert abs(float(loss_a[0]) - float(loss_b[0])) <= 1e-6 * float(loss_a[0])
    assert_close("network gradient", np_of(gmb), np_of(gma), 1e-5)
    for name, p0, pa, pb in (("density", grid.density, ga.density, gb.density), ("feat", grid.feat, ga.feat, gb.feat)):
        assert_close(f"{name} update", np_of(pb - p0), np_of(pa - p0), 1e-5)
    for a, b in zip(sa, sb):
        assert_close("moment", np_of(b), np_of(a), 1e-5)
