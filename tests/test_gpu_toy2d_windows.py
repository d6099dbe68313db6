"""The toy's vertex gradient at the edges of its lane groups: a vertex's pixel
window is walked by 4 x 4 or 8 x 8 lanes (more than 16 pixels per vertex),
widened only by the rounding of the pixel coordinates.  Sizes around that
rule, ragged ones, and grids with more vertices than the image has pixels.
Same oracle and bounds as test_gpu_toy2d."""

import numpy as np
import pytest

import oracle as O
import synth
from tests.helpers import np_of, to_dev
from tests.test_gpu_toy2d import MODES, _abs_contrib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("H,W,gh,gw", [(64, 64, 32, 32), (64, 64, 16, 16), (65, 64, 16, 16), (33, 71, 8, 9),
                                       (5, 7, 12, 9), (1, 1, 2, 2), (300, 2, 150, 2), (640, 3, 2, 3)])
def test_vertex_gradient_windows(gpu_lib, mode, H, W, gh, gw):
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(H + 13 * W + gh)
    V = (rng.normal(size=(gh, gw)) * 2.0).astype(np.float32)
    T = synth.binary_image(gw, H, W)
    loss, g = api.toy2d_loss_grad(to_dev(V), to_dev(T), MODES[mode], 1.0)
    L, gref = O.toy2d_loss_grad(V, T, mode, 1.0)
    assert abs(float(np_of(loss)[0]) - L) <= 1e-5 * L
    A, n, C = _abs_contrib(V.astype(np.float64), T, mode, 1.0)
    bound = 1e-5 * np.abs(gref).max() + (n + 8) * 2.0 ** -24 * A + C
    assert np.all(np.abs(np_of(g) - gref) <= bound)
