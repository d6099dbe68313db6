"""ReLU branches of the float32 network's adjoint at units within rounding of
zero, with units beside them that have neither weights nor bias.

One sample per ray at points where the interpolation is exact (corners, cells
and feature values are small dyadic numbers) and a first layer without view
weights, so that every pre-activation's plain float32 chain (fused
multiply-adds in input order; layer 2 takes the units of each eight in the
order 0 4 1 5 2 6 3 7) can be formed here bit for bit.  Each of 96 units has a
bias that puts it within rounding of zero in a sample of its own.  The
gradient is compared with a float64 adjoint whose branches are that chain's.

Bound: contractions of 3, 128 and 128 terms and the sum over the samples, each
term rounded once, (3 + 128 + 128 + N) 2^-24 of the sum of the absolute terms;
a branch taken the other way moves its unit's entry by about 1e-3 of it.  (W2's
gradient shows no more branches than b2's, and its factor h1 is as inexact as
it is small where a unit is near zero.)"""

import numpy as np
import pytest

from tests.helpers import mlp_flat_np, mlp_unflat, np_of, to_dev

pytestmark = pytest.mark.gpu
F32, F64 = np.float32, np.float64
N, DEAD = 96, [0, 7, 64, 127]
ORDER2 = [8 * g + u for g in range(16) for u in (0, 4, 1, 5, 2, 6, 3, 7)]


def _chain(W, b, x, order):
    """acc = fma(W[:, k], x[:, k], acc) over k, float32; x [N, K] -> [N, units]."""
    acc = np.broadcast_to(b.astype(F32), (x.shape[0], b.size)).copy()
    for k in order:
        acc = (W[:, k].astype(F64)[None] * x[:, k].astype(F64)[:, None] + acc.astype(F64)).astype(F32)
    return acc


def _samples(rng, feat, exact=True):
    """Rays along z through dyadic points of the box, and their features."""
    n = feat.shape[0]
    q = rng.integers(0, 2 * 64 - 8, (N, 3))           # position = -1 + q/64, 8 per cell
    q[:, 2] %= 8                                       # z from the jitter: within the first cell
    i0, f = q // 8, (q % 8) / 8.0
    x = np.zeros((N, feat.shape[-1]))
    for c in range(8):
        o = np.array([c >> 2 & 1, c >> 1 & 1, c & 1])
        ii = i0 + o
        x += np.prod(np.where(o, f, 1 - f), axis=1)[:, None] * feat[ii[:, 0], ii[:, 1], ii[:, 2]]
    assert n == 17 and (not exact or np.array_equal(x, x.astype(F32)))
    o = np.stack([-1 + q[:, 0] / 64, -1 + q[:, 1] / 64, np.full(N, -2.0)], axis=1).astype(F32)
    d = np.tile(np.array([0, 0, 1], F32), (N, 1))
    return o, d, (q[:, 2] / 8).astype(F32), x.astype(F32)


@pytest.mark.parametrize("pe_x", [0, 5])
@pytest.mark.parametrize("dead", [[], DEAD])
def test_branches_near_zero_follow_the_plain_chain(gpu_lib, dead, pe_x):
    import torch
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(7 + pe_x)
    feat = (rng.integers(-256, 257, (17, 17, 17, 12)) / 256.0).astype(F32)
    o, d, jit, x = _samples(rng, feat)
    W1 = np.zeros((128, 72 if pe_x else 39), F32)
    W1[:, :12] = rng.normal(size=(128, 12)) * 0.4
    W2 = (rng.normal(size=(128, 128)) * 0.12).astype(F32)
    W3 = (rng.normal(size=(3, 128)) * 0.2).astype(F32)
    b1, b2, b3 = [(rng.normal(size=k) * 0.3).astype(F32) for k in (128, 128, 3)]
    near = [u for u in range(128) if u % 4 != 3 and u not in DEAD][:N // 2]
    for s, u in enumerate(near):
        b1[u] = -(W1[u, :12].astype(F64) @ x[s])
    W1[dead], b1[dead] = 0, 0
    h1 = np.maximum(_chain(W1[:, :12], b1, x, range(12)), 0)
    for s, u in enumerate(near):
        b2[u] = -(W2[u].astype(F64) @ h1[N // 2 + s])
    W2[dead], b2[dead] = 0, 0
    z1 = _chain(W1[:, :12], b1, x, range(12))
    z2 = _chain(W2, b2, h1, ORDER2)
    rows = np.arange(N // 2)
    close = [np.abs(z1[rows, near]).max() / np.abs(z1).max(), np.abs(z2[N // 2 + rows, near]).max() / np.abs(z2).max()]
    print(f"  largest of the near-zero units, of its layer: {close[0]:.1e} {close[1]:.1e}", flush=True)

    step, shift, bg = 0.125, 0.5, (0.0, 0.0, 0.0)
    grid = api.Grid(torch.zeros((17, 17, 17), device="cuda"), to_dev(feat), (-1.0,) * 3, (1.0,) * 3, shift)
    flat = to_dev(mlp_flat_np([W1, W2, W3], [b1, b2, b3]))
    s = api.sample_rays(to_dev(o), to_dev(d), to_dev(jit), (-1.0,) * 3, (1.0,) * 3, step, 1)
    assert int(s.n_kept.item()) == N
    g = rng.normal(size=(N, 3)).astype(F32)
    out = api.render_fwd(grid, flat, s, bg)
    gd, gf, gm = torch.zeros_like(grid.density), torch.zeros_like(grid.feat), torch.zeros_like(flat)
    api.render_bwd(grid, flat, s, out["log_t_end"], to_dev(g), gd, gf, gm, bg)
    got = mlp_unflat(np_of(gm))

    W1d, W2d, W3d, xd = W1[:, :12].astype(F64), W2.astype(F64), W3.astype(F64), x.astype(F64)
    m1, m2 = z1 > 0, z2 > 0
    h1d = (xd @ W1d.T + b1) * m1
    h2d = (h1d @ W2d.T + b2) * m2
    c = 1 / (1 + np.exp(-(h2d @ W3d.T + b3)))
    w = 1 - np.exp(-np.log1p(np.exp(shift)) * step)
    dz3 = w * g * c * (1 - c)
    dz2 = (dz3 @ W3d) * m2
    dz1 = (dz2 @ W2d) * m1
    a2 = np.abs(dz3) @ np.abs(W3d)
    a1 = a2 @ np.abs(W2d)
    tol = (3 + 128 + 128 + N) * 2.0 ** -24
    sums = (("b1", got[1], dz1.sum(0), a1.sum(0)), ("W1", got[0][:, :12], dz1.T @ xd, a1.T @ np.abs(xd)),
            ("b2", got[3], dz2.sum(0), a2.sum(0)))
    beyond = []
    for name, a, ref, size in sums:
        excess = np.abs(a - ref) - tol * size
        print(f"  {name}: {int((excess > 0).sum())} entries beyond the bound, worst error "
              f"{np.max(np.abs(a - ref) / np.maximum(size, 1e-30)):.2e} of the terms (allowed {tol:.2e})", flush=True)
        beyond += [name] * bool(np.any(excess > 0))
    assert not beyond
    for name, a in (("W1", got[0]), ("b1", got[1]), ("W2", got[2]), ("b2", got[3])):
        assert not np.any(a[dead]), name
