"""GPU sampler against the oracle where its passes have edges: vocabularies around
one entry per thread (1024), one group maximum per thread (256) and the largest
(16384), top-k from 2 to the limit, rows with more exact ties than the candidate
list holds, zeros of both signs, NaN entries (they count as -inf) and rows with
fewer finite entries than top-k.  Choices are equal unless the draw sits within
1e-5 of a cumulative boundary (one-ulp differences of the exponentials).
"""
import numpy as np
import pytest

from oracle import sample as osample
from paper_2607_21042_amd import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [2, 64, 255, 256, 257, 1023, 1024, 1025, 4099, 16383, 16384])
def test_sampler_edges(V):
    import torch
    from paper_2607_21042_amd import ftts
    B = 48
    z = workload.random_logits(B, V, seed=V)
    rng = np.random.default_rng(V)
    z[0:6] = np.round(z[0:6] * 2) / 2                 # many exact ties
    z[6:12] = 0.25                                     # one value: more candidates than the list holds at V > 1024
    z[12:18] = np.where(rng.random((6, V)) < 0.5, np.float32(0.0), np.float32(-0.0))
    z[18:24, V // 2:] = -np.inf
    z[24:30][rng.random((6, V)) < 0.3] = np.nan
    z[24:30, V - 1] = 3.0
    z[30:36] = -np.inf                                 # one finite entry
    z[30:36, V // 3] = -7.0
    z[36:42] = -1.0 - np.arange(V, dtype=np.float32)[None] * 1e-3  # the best entries side by side
    ref = np.where(np.isnan(z), np.float32(-np.inf), z)
    u = workload.uniforms(1, B, seed=V + 1)[0]
    zt, ut = torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda()
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    for (T, k, p) in [(1.0, 1, 1.0), (0.8, 2, 0.9), (0.8, 30, 0.8), (1.3, 63, 1.0), (1.7, 64, 0.95)]:
        if k > V:
            continue
        print(f"sampler edges: V={V} T={T} k={k} p={p}", flush=True)
        ftts.sample(zt, ftts.Sampling(T, k, p), ut, out)
        got = out.cpu().numpy()
        for b in range(B):
            want, det = osample.sample(ref[b], T, k, p, u[b])
            assert got[b] == want or osample.near_boundary(det), (T, k, p, b, got[b], want)
