"""The fused grid Adam deals chunks of two x-planes (256 vertices at least) to
the eight XCDs: on grids whose chunks reach one XCD, some or all of them, with
a short last one, every vertex has to take exactly one step.  Without samples
the step is the one with a zero gradient, bit for bit that of adam_step; with
them the fused call is compared with the separate ones as in
test_gpu_vertex_gather (1e-5)."""

import numpy as np
import pytest

from tests.helpers import assert_close, np_of, to_dev
from tests.test_gpu_render import F32, _gpu, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hit", [False, True])
@pytest.mark.parametrize("shape", [(2, 2, 2), (5, 5, 5), (8, 8, 8), (9, 8, 16), (12, 12, 12), (17, 16, 16),
                                   (2, 61, 40), (100, 3, 2)])
def test_every_vertex_steps_once(gpu_lib, shape, hit):
    import torch
    from paper_2111_11215_amd import api
    P = _problem(seed=6, n_rays=100, bias=0.3)
    rng = np.random.default_rng(sum(shape))
    P.density = rng.normal(size=shape).astype(F32)
    P.feat = (rng.normal(size=shape + (12,)) * 0.1).astype(F32)
    if not hit:
        P.rays.o = (P.rays.o + 100.0).astype(F32)
    grid, flat, s = _gpu(P, morton=False)
    assert (int(s.n_kept.item()) > 0) == hit
    out = api.render_fwd(grid, flat, s, P.bg)
    g = to_dev(rng.normal(size=(100, 3)).astype(F32))
    state = [to_dev((rng.normal(size=x.shape) * 0.1).astype(F32) ** k) for x in (P.density, P.feat) for k in (1, 2)]
    gd, gf = torch.zeros_like(grid.density), torch.zeros_like(grid.feat)
    api.render_bwd(grid, flat, s, out["log_t_end"], g, gd, gf, torch.zeros_like(flat), bg=P.bg)
    a, b = (api.Grid(grid.density.clone(), grid.feat.clone(), grid.box_min, grid.box_max, grid.act_shift)
            for _ in range(2))
    sa, sb = [x.clone() for x in state], [x.clone() for x in state]
    api.adam_step(a.density, gd, sa[0], sa[1], 0.1, 3)
    api.adam_step(a.feat, gf, sa[2], sa[3], 0.1, 3)
    api.render_bwd_adam(b, flat, s, out["log_t_end"], g, *sb, torch.zeros_like(flat), 0.1, 3, bg=P.bg)
    for p, q in zip([a.density, a.feat] + sa, [b.density, b.feat] + sb):
        if hit:
            assert_close("fused", np_of(q), np_of(p), 1e-5)
        else:
            assert np.array_equal(np_of(q).view(np.uint32), np_of(p).view(np.uint32))
