"""Ranking and redrawing at the edges of their work split (4 hypotheses per
wavefront, 16 and 256 per block): against the oracle with ties and NaN losses,
poses within one float32 ulp per update, optimiser rows exactly."""
import math
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2210_10108_amd import synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 3, 5, 15, 16, 17, 63, 65, 255, 256, 257, 513, 3001])
@pytest.mark.parametrize("kind", ["ties", "nan"])
def test_resample_block_edges(K, kind):
    import torch
    from paper_2210_10108_amd import pnerf
    sys.stderr.write(f"[gpu] resample K={K} {kind}\n")
    sys.stderr.flush()
    w = synth.WORKLOADS["tiny32"]
    poses = synth.perturb_poses(synth.ground_truth_pose(w, 0), K, 40, 0.3, 1)
    rng = np.random.default_rng(K)
    mom = rng.normal(size=(K, 6)).astype(np.float32)
    # many equal losses; or every third NaN, infinities of both signs beside them
    loss = rng.integers(0, max(2, K // 8), K).astype(np.float32)
    if kind == "nan":
        loss[::3] = np.nan
        loss[1::7] = np.inf
        loss[2::11] = -np.inf
    for keep in (0.0, 0.3, 1.0):
        p_ref, m_ref, _ = O.resample(poses, mom, loss, keep, math.radians(5), 0.03, 1234, 3)
        p, m = G.to_dev(poses), G.to_dev(mom)
        pnerf.resample_hypotheses(p, m, G.to_dev(loss), keep, math.radians(5), 0.03, 1234, 3)
        torch.cuda.synchronize()
        assert np.array_equal(m.cpu().numpy(), m_ref)
        assert np.allclose(p.cpu().numpy(), p_ref, atol=1e-6, rtol=0)
