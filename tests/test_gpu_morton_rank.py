"""The Morton order's counting kernel at the edges of its tiles (64 rays per
workgroup, sixteen slices of the keys rounded up to 16) and at its limit of
32768 rays: the permutation equals a stable sort by the documented key, formed
here in the same float32 recipe."""

import numpy as np
import pytest

from tests.helpers import np_of, to_dev

pytestmark = pytest.mark.gpu
F32 = np.float32


def _keys(o, d, s):
    tm = (np_of(s.t_near) + np_of(s.t_far)) * F32(0.5)
    m = o + tm[:, None] * d
    q = np.clip(np.floor((m - F32(-1)) * F32(16)), 0, 31).astype(np.int64)
    key = np.zeros(len(o), np.int64)
    for b in range(5):
        for c in range(3):
            key |= ((q[:, c] >> b) & 1) << (3 * b + 2 - c)
    return np.where(np_of(s.valid) != 0, key, 1 << 15)


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 255, 257, 1000, 4097, 32768])
def test_morton_permutation(gpu_lib, B):
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(B)
    o = rng.normal(size=(B, 3))
    o = (4 * o / np.linalg.norm(o, axis=1, keepdims=True)).astype(F32)
    d = -o / 4 + 0.3 * rng.normal(size=(B, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(F32)
    o[B // 2:] = o[: B - B // 2]      # equal keys: the ray id decides
    d[B // 2:] = d[: B - B // 2]
    s = api.sample_rays(to_dev(o), to_dev(d), None, (-1, -1, -1), (1, 1, 1), 0.05, 80, morton=True)
    assert np.array_equal(np_of(s.perm), np.argsort(_keys(o, d, s), kind="stable"))
