"""Vertex sums at the sizes of test_gpu_vertex_gather with the bound of the
fullest vertex: a sum of n float32 terms errs by at most n 2^-24 of their
absolute sum, n the most samples of any one vertex (not of the batch), and
1e-5 where that is smaller.  Network gradients at 1e-5 in both metrics."""

import numpy as np
import pytest

import oracle as O
from tests.helpers import assert_close, check_grid_grad, check_weight_grads, kink_budget, samples_per_vertex
from tests.test_gpu_render import F32, TOL32, ZETA, _gpu, _grads, _oracle, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,n_rays", [((2, 2, 2), 40), ((2, 3, 2), 300), ((3, 2, 17), 200), ((5, 4, 33), 300),
                                          ((17, 19, 16), 400), ((33, 3, 65), 64)])
def test_vertex_sums_by_their_own_records(gpu_lib, shape, n_rays):
    from paper_2111_11215_amd import api
    P = _problem(seed=5, n_rays=n_rays, bias=0.3)
    rng = np.random.default_rng(sum(shape))
    P.density = rng.normal(size=shape).astype(F32)
    P.feat = (rng.normal(size=shape + (12,)) * 0.1).astype(F32)
    grid, flat, s = _gpu(P, morton=False)
    samp, prm, ref, (o, d, j) = _oracle(P, morton=False)
    most = int(samples_per_vertex(ref["cache"]["x"], P.box_min, P.box_max, shape).max())
    tol = max(TOL32, most * 2.0 ** -24)
    print(f"  {int(s.n_kept.item())} samples, at most {most} a vertex: {tol:.1e}", flush=True)
    out = api.render_fwd(grid, flat, s, P.bg)
    g = rng.normal(size=ref["rgb"].shape).astype(F32)
    gd, gf, gm = _grads(api, grid, flat, s, out, g, P)
    gr = O.render_backward(prm, o, d, j, samp, P.step, P.bg, ref, g)
    assert_close("grad_density", gd, gr["density"], TOL32, tol)
    budget, wb, _ = kink_budget(prm, ref, g, ZETA, P.feat.shape, P.box_min, P.box_max)
    check_grid_grad("grad_feat", gf, gr["feat"], budget, TOL32, tol)
    check_weight_grads(gm, gr["Ws"], gr["bs"], wb, TOL32, TOL32)
