"""The float32 network where its operands leave the range of the bfloat16
planes: finite values above the largest bfloat16, infinities, gradients of
2^64 and weights of 2^20 and more, which the plain float32 chain takes over.

Values within float32 are held to the oracle at test_gpu_render's bounds, and
an ordinary batch made to take the other adjoint (a huge weight on a unit that
is never active; a gradient scaled by a power of two) to the planes' own
result at the same 1e-5.  With infinities, inputs and pre-activations follow
IEEE arithmetic with a ReLU that gives 0 for NaN, formed here in float64 (no
finite value comes near float32's limits): which outputs are infinite or NaN
is compared exactly, the rest at 1e-5."""

import numpy as np
import pytest

from tests.helpers import assert_close, mlp_flat_np, mlp_unflat, np_of, to_dev
from tests.test_gpu_relu_branches import N, _samples
from tests.test_gpu_render import (F32, TOL32, _check_backward, _gpu, _grads, _oracle, _problem,
                                   _with_position_encoding)

pytestmark = pytest.mark.gpu


def _case(seed, n_rays, pe_x):
    P = _problem(seed=seed, n_rays=n_rays, bias=0.3)
    return _with_position_encoding(P, seed) if pe_x else P


@pytest.mark.parametrize("pe_x", [0, 5])
@pytest.mark.parametrize("n_rays", [1, 37])
def test_plain_adjoint_matches_the_planes(gpu_lib, n_rays, pe_x):
    from paper_2111_11215_amd import api
    P = _case(n_rays, n_rays, pe_x)
    P.Ws[0][9], P.bs[0][9] = 0, -1          # never active, so W2's column 9 meets zeros only
    g = np.random.default_rng(n_rays).normal(size=(n_rays, 3)).astype(F32)

    def grads(scale=1.0):
        grid, flat, s = _gpu(P, morton=False)
        out = api.render_fwd(grid, flat, s, P.bg)
        return [np_of(out["rgb"])] + [np.asarray(x, np.float64) / scale
                                      for x in _grads(api, grid, flat, s, out, g * F32(scale), P)]

    want = grads()
    P.Ws[1][:, 9] = 2.0 ** 21
    heavy = grads()
    P.Ws[1][:, 9] = 0.5
    steep = grads(2.0 ** 70)
    for got in (heavy, steep):
        for name, a, b in zip(("rgb", "grad_density", "grad_feat", "grad_mlp"), got, want):
            assert_close(name, a, b, TOL32)


@pytest.mark.parametrize("pe_x", [0, 5])
def test_finite_values_above_bfloat16(gpu_lib, pe_x):
    """One feature channel of 3.4e38 with first-layer weights of 3e-38."""
    from paper_2111_11215_amd import api
    P = _case(11, 50, pe_x)
    rng = np.random.default_rng(11)
    P.feat[..., 3] = 3.3995e38
    P.Ws[0][:, 3] = (rng.normal(size=128) * 3e-38).astype(F32)
    grid, flat, s = _gpu(P, morton=False)
    samp, prm, ref, ro = _oracle(P, morton=False)
    out = api.render_fwd(grid, flat, s, P.bg)
    assert_close("rgb", np_of(out["rgb"]), ref["rgb"], TOL32)
    g = rng.normal(size=ref["rgb"].shape).astype(F32) * F32(1e-3)
    gd, gf, gm = _grads(api, grid, flat, s, out, g, P)
    ref["_samp"] = samp
    _check_backward(P, prm, ref, ro, gd, gf, gm, g, TOL32)


def _same(name, got, ref):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref)), f"{name}: NaN"
    inf = np.isinf(ref)
    assert np.array_equal(inf, np.isinf(got)) and np.array_equal(got[inf], ref[inf]), f"{name}: infinities"
    ok = np.isfinite(ref)
    print(f"  {name}: {int(ok.sum())} finite, {int(inf.sum())} infinite, {int(np.isnan(ref).sum())} NaN", flush=True)
    if ok.any():
        assert_close(name, got[ok], ref[ok], TOL32)


@pytest.mark.parametrize("case", ["one_unit", "all_units", "weight"])
def test_infinities(gpu_lib, case):
    import torch
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(5)
    feat = (rng.integers(-256, 257, (17, 17, 17, 12)) / 256.0).astype(F32)
    if case != "weight":
        where = rng.random((17, 17, 17)) < 0.02
        feat[where, 3] = np.where(rng.random(int(where.sum())) < 0.7, np.inf, -np.inf)
    with np.errstate(invalid="ignore"):
        o, d, jit, x = _samples(rng, feat, exact=False)
    W1 = np.zeros((128, 39), F32)
    W1[:, :12] = rng.normal(size=(128, 12)) * 0.4
    W2 = (rng.normal(size=(128, 128)) * 0.12).astype(F32)
    W3 = (rng.normal(size=(3, 128)) * 0.2).astype(F32)
    b1, b2, b3 = [(rng.normal(size=k) * 0.3).astype(F32) for k in (128, 128, 3)]
    if case == "one_unit":     # an infinite h1[20], every z2 of either sign infinite, logits of one sign
        W1[:, 3] = 0
        W1[20, 3] = 0.5
        feat[..., 3] = np.where(np.isinf(feat[..., 3]), feat[..., 3], 0.25)
        W3[0], W3[1] = np.abs(W3[0]), -np.abs(W3[1])
        with np.errstate(invalid="ignore"):
            o, d, jit, x = _samples(np.random.default_rng(5), feat, exact=False)
    if case == "weight":
        W2[40, 50] = np.inf
    assert case == "weight" or 0 < np.isfinite(x).all(axis=1).sum() < N
    step, shift, bg = 0.125, 0.5, (0.0, 0.0, 0.0)
    g = rng.normal(size=(N, 3)).astype(F32)
    grid = api.Grid(torch.zeros((17, 17, 17), device="cuda"), to_dev(feat), (-1.0,) * 3, (1.0,) * 3, shift)
    flat = to_dev(mlp_flat_np([W1, W2, W3], [b1, b2, b3]))
    s = api.sample_rays(to_dev(o), to_dev(d), to_dev(jit), (-1.0,) * 3, (1.0,) * 3, step, 1)
    out = api.render_fwd(grid, flat, s, bg)
    gd, gf, gm = torch.zeros_like(grid.density), torch.zeros_like(grid.feat), torch.zeros_like(flat)
    api.render_bwd(grid, flat, s, out["log_t_end"], to_dev(g), gd, gf, gm, bg)
    got = mlp_unflat(np_of(gm))

    W1d, W2d, W3d, xd = [np.asarray(v, np.float64) for v in (W1[:, :12], W2, W3, x)]
    dot = lambda a, b: np.array([[np.sum(r * c) for c in b.T] for r in a])   # (a product that keeps 0 inf = NaN)
    with np.errstate(invalid="ignore", over="ignore"):
        z1 = dot(xd, W1d.T) + b1
        h1 = np.fmax(z1, 0)
        z2 = dot(h1, W2d.T) + b2
        h2 = np.fmax(z2, 0)
        c = 1 / (1 + np.exp(-(dot(h2, W3d.T) + b3)))
        w = 1 - np.exp(-np.log1p(np.exp(shift)) * step)
        dz3 = w * g * c * (1 - c)
        dz2 = np.where(z2 > 0, dot(dz3, W3d), 0)
        dz1 = np.where(z1 > 0, dot(dz2, W2d), 0)
        want = [dot(dz1.T, xd), dz1.sum(0), dot(dz2.T, h1), dz2.sum(0), dot(dz3.T, h2), dz3.sum(0)]
    _same("rgb", np_of(out["rgb"]), w * c)
    for name, a, ref in zip(("W1", "b1", "W2", "b2", "W3", "b3"), got, want):
        _same(name, a[:, :12] if name == "W1" else a, ref)
