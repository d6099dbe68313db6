"""Grid gradients of the vertex kernels where their splits end.

A lane quad sums one vertex, lists 32 records at a time and reads 4 of them
ahead; a wavefront takes 16 consecutive vertices across rows and planes.
Grids of a few vertices give cells of hundreds of samples (lists of many
passes), rows shorter than a wavefront's 16 vertices and a ragged last one.
Bounds as in test_gpu_render (float32: 1e-5 in both metrics) with the max
metric of a sum of n terms, n x 2^-24, where a vertex has more than 168; the
fused step against the separate calls as in test_gpu_fused (1e-5)."""

import numpy as np
import pytest

from tests.helpers import assert_close, np_of, to_dev
from tests.test_gpu_render import F32, TOL32, _check_backward, _gpu, _grads, _oracle, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,n_rays", [((2, 2, 2), 40), ((2, 3, 2), 300), ((3, 2, 17), 200), ((5, 4, 33), 300),
                                          ((17, 19, 16), 400), ((33, 3, 65), 64)])
def test_vertex_sums_at_split_edges(gpu_lib, shape, n_rays):
    import torch
    from paper_2111_11215_amd import api
    P = _problem(seed=5, n_rays=n_rays, bias=0.3)
    rng = np.random.default_rng(sum(shape))
    P.density = rng.normal(size=shape).astype(F32)
    P.feat = (rng.normal(size=shape + (12,)) * 0.1).astype(F32)
    grid, flat, s = _gpu(P, morton=False)
    samp, prm, ref, ro = _oracle(P, morton=False)
    n = int(s.n_kept.item())
    print(f"  {n} samples, {np.prod(shape)} vertices", flush=True)
    out = api.render_fwd(grid, flat, s, P.bg)
    g = rng.normal(size=ref["rgb"].shape).astype(F32)
    gd, gf, gm = _grads(api, grid, flat, s, out, g, P)
    ref["_samp"] = samp
    _check_backward(P, prm, ref, ro, gd, gf, gm, g, TOL32, tol_max=max(TOL32, n * 2.0 ** -24))

    # the fused Adam step, with and without an activity mask
    state = [to_dev((rng.normal(size=x.shape) * 0.1).astype(F32) ** k) for x in (P.density, P.feat) for k in (1, 2)]
    a = api.Grid(grid.density.clone(), grid.feat.clone(), grid.box_min, grid.box_max, grid.act_shift)
    sa = [x.clone() for x in state]
    api.adam_step(a.density, to_dev(gd), sa[0], sa[1], 0.1, 3)
    api.adam_step(a.feat, to_dev(gf), sa[2], sa[3], 0.1, 3)
    for masked in (False, True):
        b = api.Grid(grid.density.clone(), grid.feat.clone(), grid.box_min, grid.box_max, grid.act_shift)
        sb = [x.clone() for x in state]
        active = None
        if masked:
            active = torch.zeros(api.grid_active_words(P.density.size), dtype=torch.int32, device="cuda")
            api.grid_active_init(*sb, active)
        api.render_bwd_adam(b, flat, s, out["log_t_end"], to_dev(g), *sb, torch.zeros_like(flat), 0.1, 3, bg=P.bg,
                            active=active)
        for name, p, q in (("density", a.density, b.density), ("feat", a.feat, b.feat)):
            assert_close(name, np_of(q), np_of(p), 1e-5)
        for p, q in zip(sa, sb):
            assert_close("moment", np_of(q), np_of(p), 1e-5)
