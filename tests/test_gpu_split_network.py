"""The float32 network's plane-split kernels at the edges of their tiles.

The forward takes 32 samples per wavefront and deals its tiles differently
when there are fewer than wavefronts; the adjoint takes blocks of 64 samples
(two column tiles), the last one ragged.  Batches of one to a few hundred rays
give sample counts below, at and beyond these sizes; a batch above 65536
samples takes the other dealing.  Bounds as in test_gpu_render: 1e-5 in both
metrics, ReLU-ambiguous samples within their proven budget.

Branch bits: a unit at exactly zero (a row without weights) has no gradient,
and neither do the samples past the last one."""

import numpy as np
import pytest

from tests.helpers import assert_close, np_of, to_dev
from tests.test_gpu_render import (TOL32, _check_backward, _gpu, _grads, _oracle, _problem, _with_position_encoding)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pe_x", [0, 5])
@pytest.mark.parametrize("n_rays", [1, 2, 5, 37, 300, 2600])
def test_split_network_at_tile_edges(gpu_lib, n_rays, pe_x):
    from paper_2111_11215_amd import api
    P = _problem(seed=n_rays, n_rays=n_rays, bias=0.3)
    if pe_x:
        P = _with_position_encoding(P, n_rays)
    grid, flat, s = _gpu(P, morton=False)
    samp, prm, ref, ro = _oracle(P, morton=False)
    print(f"  {int(s.n_kept.item())} samples", flush=True)
    out = api.render_fwd(grid, flat, s, P.bg)
    assert_close("rgb", np_of(out["rgb"]), ref["rgb"], TOL32)
    g = np.random.default_rng(n_rays).normal(size=ref["rgb"].shape).astype(np.float32)
    gd, gf, gm = _grads(api, grid, flat, s, out, g, P)
    ref["_samp"] = samp
    _check_backward(P, prm, ref, ro, gd, gf, gm, g, TOL32)


def test_dead_units_have_no_gradient(gpu_lib):
    """Rows of W1 and W2 without weights or bias: z = 0 exactly, relu' = 0."""
    import torch
    from paper_2111_11215_amd import api
    P = _problem(seed=3, n_rays=64)
    dead = [5, 64, 127]
    for layer in (0, 1):
        P.Ws[layer][dead] = 0.0
        P.bs[layer][dead] = 0.0
    grid, flat, s = _gpu(P, morton=False)
    out = api.render_fwd(grid, flat, s, P.bg)
    assert torch.isfinite(out["rgb"]).all()
    g = np.ones((64, 3), np.float32)
    _, _, gm = _grads(api, grid, flat, s, out, g, P)
    v = api.split_flat(to_dev(gm), api.MLP_SHAPES)
    assert float(v["b2"][dead].abs().max()) == 0.0 and float(v["b1"][dead].abs().max()) == 0.0
    assert float(v["w2"][dead].abs().max()) == 0.0 and float(v["w1"][dead].abs().max()) == 0.0
    assert float(v["b1"].abs().max()) > 0.0
