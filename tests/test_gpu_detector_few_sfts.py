"""Detector inputs of few SFTs, whose lanes take several sky points side by
side: SFT counts around the powers of two that set the lanes, sky points
around a block's share, an unknown site, against the FP64 oracle (the bounds
of the work-unit shape)."""
import numpy as np
import pytest

import oracle
import synth.workloads as sw
from tests.test_gpu_detector import EARTH, SITES, _device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sft,n_sky", [(1, 1), (1, 255), (1, 257), (2, 1000), (3, 64), (5, 33), (63, 9), (64, 65),
                                         (65, 130), (128, 5), (128, 129), (129, 66), (256, 3), (257, 65)])
def test_few_sfts(n_sft, n_sky):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(1000 * n_sft + n_sky)
    t = np.sort(sw.EPOCH + rng.uniform(0, 3.0e7, n_sft))
    idx = rng.integers(0, 2, n_sft).astype(np.int32)
    sky = rng.normal(size=(n_sky, 3))
    sky /= np.linalg.norm(sky, axis=1, keepdims=True)
    pos, vel, a, b, _ = _device(torch, EARTH, t, idx, sky)
    rp, rv, ra, rb = oracle.detector_inputs(EARTH, SITES, t, idx, sky)
    assert np.max(np.abs(pos - rp)) < 1e-11 and np.max(np.abs(vel - rv)) < 1e-17
    assert np.max(np.abs(a - ra)) < 3e-7 and np.max(np.abs(b - rb)) < 3e-7
    bad = idx.copy()
    bad[-1] = -1
    pos, vel, a, b, _ = _device(torch, EARTH, t, bad, sky)
    for x in (pos[-1], vel[-1], a[:, -1], b[:, -1]):
        assert np.all(np.isnan(x))
    assert np.max(np.abs(a - ra)[:, :-1], initial=0) < 3e-7
