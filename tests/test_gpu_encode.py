"""The encoding kernel at the edges of its work split, per sample against the
oracle (per-sample tolerances of test_gpu_parity): wavefronts whose samples
span more rays than the LDS slots hold, samples clamped to the box, levels
grouped per work queue (many small tables), one queue per large dense level,
hashed levels only and dense levels only, and the last partial runs of 32."""
import dataclasses
import math
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2210_10108_amd import synth
from tests import gpu_common as G
from tests.test_gpu_parity import check_full

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    sys.stderr.write(f"[gpu] {request.node.nodeid}\n")
    sys.stderr.flush()


@pytest.fixture(scope="module")
def pn():
    from paper_2210_10108_amd import pnerf
    pnerf.lib()
    return pnerf


def one_cell(R):
    occ = np.zeros((R, R, R), bool)
    occ[R // 2, R // 2, R // 2] = True
    return synth.pack_bits(occ)


# (levels, log2 table, n_max, storage, dense coarse levels)
FIELDS = {
    "grouped_hashed": (16, 10, 64, "f32", 0),
    "grouped_both": (12, 14, 64, "f16", 1),
    "all_dense": (8, 18, 48, "f32", 1),
    "large_dense": (4, 22, 150, "f32", 1),
    "smallest_table": (4, 4, 64, "f16", 0),
    # the last level is dense and fills its table: 256^3 = 2^24 vertices
    "largest_dense": (4, 24, 255, "f16", 1),
}


def case_of(monkeypatch, field, K, P, camera=(2.5, 40.0), **kw):
    L, log2, n_max, dtype, dense = FIELDS[field]
    w = dataclasses.replace(synth.WORKLOADS["tiny32"], name=field, n_levels=L, log2_table=log2,
                            n_max=n_max, param_dtype=dtype, cam_radius=camera[0],
                            focal=camera[1], max_rot_deg=20.0 * 2.5 / camera[0])
    monkeypatch.setitem(synth.WORKLOADS, field, w)
    return G.make_case(field, K=K, P=P, dense_coarse_levels=dense, **kw)


def check(pn, case):
    of = O.OracleField(case.spec)
    obs = G.oracle_observation(of, case.gt, case.pix, case.intr)
    ref = of.render_loss_grad(case.poses, case.pix, obs, case.intr, per_sample=True)
    stats, _ = check_full(pn, case, obs, ref, of)
    assert stats["samples"] == int(ref["march"][0][-1])
    return ref


@pytest.mark.parametrize("field", sorted(FIELDS))
@pytest.mark.parametrize("K,P", [(3, 97), (1, 11)])
def test_encode_level_groups(pn, monkeypatch, field, K, P):
    check(pn, case_of(monkeypatch, field, K, P))


@pytest.mark.parametrize("field", ["grouped_hashed", "all_dense"])
def test_encode_wavefront_of_many_rays(pn, monkeypatch, field):
    # one cell of 8^3 is set: most rays keep no sample, the others a few
    case = case_of(monkeypatch, field, 2, 4000, march_mode=1, step=math.sqrt(3) / 256,
                   max_samples=64, t_stop=0.0, occ_res=8, occ_bits=one_cell(8))
    ref = check(pn, case)
    ray = np.repeat(np.arange(8000), np.diff(ref["march"][0]))
    assert len(ray) > 128
    spans = [ray[min(s + 63, len(ray) - 1)] - ray[s] for s in range(0, len(ray), 64)]
    assert max(spans) >= 64  # more rays than slots


@pytest.mark.parametrize("field", ["grouped_hashed", "all_dense"])
def test_encode_clamped_samples(pn, monkeypatch, field):
    # the first samples of a ray, so close to the box, and the camera so far
    # from it, that rounding puts some of them outside it
    case = case_of(monkeypatch, field, 4, 256, camera=(40.0, 1000.0), march_mode=1, step=2e-6,
                   max_samples=3, t_stop=0.0)
    ref = check(pn, case)
    off, t = ref["march"][0], ref["march"][1]
    f = np.float32
    clamped = 0
    for r in np.flatnonzero(np.diff(off)):
        pose, pix = case.poses[r // 256], case.pix.reshape(-1)[r]
        c = np.array([(pix % 32 + 0.5 - 16) / 1000, (pix // 32 + 0.5 - 16) / 1000, 1])
        d = pose[:, :3].astype(np.float64) @ c
        d = (d / np.linalg.norm(d)).astype(f)
        for s in range(off[r], off[r + 1]):
            p = pose[:, 3] + f(t[s]) * d
            clamped += bool(np.any(np.abs(p) > f(0.5)))
    assert clamped > 0
