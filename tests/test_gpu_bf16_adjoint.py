"""The bfloat16 network adjoint at the edges of its blocks.

A workgroup takes blocks of 128 samples, two halves of two column tiles each;
batches of one to a few hundred rays give a first block with empty halves and
tiles and a ragged last one, 2600 rays more blocks than workgroups.  Bounds of
test_gpu_render's bfloat16 form; with a few dozen samples a single operand
that rounds to its neighbour (2^-8 of a term) is not averaged out, so the
normwise bound is the one of a single value there."""

import numpy as np
import pytest

from tests.test_gpu_render import TOLBF, ZETA_BF16, _check_backward, _gpu, _grads, _oracle, _problem, _with_position_encoding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pe_x", [0, 5])
@pytest.mark.parametrize("n_rays", [1, 2, 5, 37, 300, 2600])
def test_bf16_adjoint_at_block_edges(gpu_lib, n_rays, pe_x):
    from paper_2111_11215_amd import api
    from paper_2111_11215_amd._lib import DVGO_BF16
    P = _problem(seed=n_rays, n_rays=n_rays, bias=0.3)
    if pe_x:
        P = _with_position_encoding(P, n_rays)
    grid, flat, s = _gpu(P, morton=False, bf16=True)
    samp, prm, ref, ro = _oracle(P, morton=False, bf16=True)
    print(f"  {int(s.n_kept.item())} samples", flush=True)
    out = api.render_fwd(grid, flat, s, P.bg, precision=DVGO_BF16, use_shadow=True)
    g = np.random.default_rng(n_rays).normal(size=ref["rgb"].shape).astype(np.float32)
    gd, gf, gm = _grads(api, grid, flat, s, out, g, P, True)
    ref["_samp"] = samp
    _check_backward(P, prm, ref, ro, gd, gf, gm, g, TOLBF if n_rays >= 300 else ZETA_BF16)
