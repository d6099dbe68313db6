"""Ray offsets and sample list of large batches at the limits of their paths:
counts summed by every workgroup (up to 16384 rays), by groups of 1024 rays
(up to 2^20), the single scan beyond.  Without masks a ray keeps its uniform
samples, so the lists follow from n_uniform by a prefix sum: whole numbers,
equal."""

import numpy as np
import pytest

from tests.helpers import np_of, to_dev

pytestmark = pytest.mark.gpu
F32 = np.float32


@pytest.mark.parametrize("B,morton", [(16384, False), (16385, False), (17408, False), (17409, False), (20001, True),
                                      (32768, True), (1 << 20, False), ((1 << 20) + 1, False)])
def test_offsets_at_path_limits(gpu_lib, B, morton):
    from paper_2111_11215_amd import api
    rng = np.random.default_rng(B)
    o = rng.normal(size=(B, 3))
    o = (3 * o / np.linalg.norm(o, axis=1, keepdims=True)).astype(F32)
    d = -o / 3 + 0.35 * rng.normal(size=(B, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(F32)
    s = api.sample_rays(to_dev(o), to_dev(d), None, (-1, -1, -1), (1, 1, 1), 0.5, 7, morton=morton)
    perm, n = np_of(s.perm), np_of(s.n_uniform)
    assert np.array_equal(np.sort(perm), np.arange(B)) and (morton or np.array_equal(perm, np.arange(B)))
    assert n.min() == 0 and n.max() > 3
    counts = n[perm]
    off = np.concatenate([[0], np.cumsum(counts)])
    assert np.array_equal(np_of(s.ray_offset), off) and int(np_of(s.n_kept)[0]) == off[-1]
    total = int(off[-1])
    assert np.array_equal(np_of(s.sample_ray)[:total], np.repeat(perm, counts))
    assert np.array_equal(np_of(s.sample_k)[:total], np.arange(total) - np.repeat(off[:-1], counts))
