"""Trilinear gathers at the edges of their split.

A wavefront takes 64 samples, 16 at a time with a lane quad each: sample
counts below and just beyond these from one to a few rays, on grids with odd
extents (density pairs at odd addresses) and with a single cell per axis.
Forward outputs against the oracle, bounds as in test_gpu_render (float32
1e-5; bfloat16 the single-operand bound, for few samples)."""

import numpy as np
import pytest

from tests.test_gpu_render import F32, TOL32, ZETA_BF16, _fwd_keys, _gpu, _oracle, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape,n_rays", [((2, 2, 2), 1), ((3, 5, 7), 2), ((9, 2, 33), 3), ((16, 17, 15), 37)])
def test_gather_at_split_edges(gpu_lib, shape, n_rays, bf16):
    from paper_2111_11215_amd import api
    from paper_2111_11215_amd._lib import DVGO_BF16, DVGO_F32
    P = _problem(seed=9, n_rays=n_rays, bias=0.3)
    rng = np.random.default_rng(sum(shape))
    P.density = rng.normal(size=shape).astype(F32)
    P.feat = (rng.normal(size=shape + (12,)) * 0.1).astype(F32)
    grid, flat, s = _gpu(P, morton=False, bf16=bf16)
    print(f"  {int(s.n_kept.item())} samples", flush=True)
    out = api.render_fwd(grid, flat, s, P.bg, precision=DVGO_BF16 if bf16 else DVGO_F32, use_shadow=bf16)
    _, _, ref, _ = _oracle(P, morton=False, bf16=bf16)
    tol = ZETA_BF16 if bf16 else TOL32
    _fwd_keys(out, ref, ("rgb", "depth", "acc", "log_t_end"), tol)
    dens = api.render_fwd(grid, None, s, P.bg)   # density only
    _fwd_keys(dens, ref, ("depth", "acc", "log_t_end"), TOL32)
