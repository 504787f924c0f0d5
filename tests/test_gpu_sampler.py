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


@pytest.mark.parametrize("V", [2, 64, 256, 257, 320, 1023, 1024, 8194, 16384])
def test_sampler_wave_threshold_edges(V):
    """Top-k on both sides of the 16 waves' maxima and of the number of waves that a row
    reaches, with ties, entries side by side and rows in few waves."""
    import torch
    from paper_2607_21042_amd import ftts
    B = 40
    z = workload.random_logits(B, V, seed=V + 1)
    z[0:8] = np.round(z[0:8] * 2) / 2
    z[8:16] = -1.0 - np.arange(V, dtype=np.float32)[None] * 1e-3
    z[16:24] = -np.inf
    z[16:24, V // 2:V // 2 + 70] = workload.random_logits(8, V, seed=V + 2)[:, V // 2:V // 2 + 70]
    z[24:28] = 0.5
    u = workload.uniforms(1, B, seed=V + 3)[0]
    zt, ut = torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda()
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    for k in (2, 3, 4, 5, 6, 15, 16, 17):
        if k > V:
            continue
        print(f"sampler wave threshold: V={V} k={k}", flush=True)
        ftts.sample(zt, ftts.Sampling(0.9, k, 0.9), ut, out)
        got = out.cpu().numpy()
        for b in range(B):
            want, det = osample.sample(z[b], 0.9, k, 0.9, u[b])
            assert got[b] == want or osample.near_boundary(det), (k, b, got[b], want)


@pytest.mark.parametrize("V", [64, 100, 200, 1025, 8194])
def test_sampler_few_finite_entries(V):
    """Rows with 0 .. k + 2 finite entries, in one run or scattered, the rest -inf
    (and a few led by +inf, whose exponentials are NaN): the ranks past the finite
    entries go to the lowest-index -inf ones."""
    import torch
    from paper_2607_21042_amd import ftts
    rng = np.random.default_rng(V)
    for T, k, p in [(0.8, 2, 0.9), (0.8, 30, 0.8), (1.7, 64, 1.0)]:
        n_finite = [n for n in (0, 1, 2, 3, k // 2, k - 1, k, k + 1, k + 2) if n <= V]
        z = np.full((3 * len(n_finite), V), -np.inf, np.float32)
        for i, n in enumerate(n_finite):
            at = int(rng.integers(0, V - n + 1))
            z[3 * i, at:at + n] = rng.standard_normal(n)
            z[3 * i + 1, rng.permutation(V)[:n]] = rng.standard_normal(n)
            z[3 * i + 2, V - n:] = rng.standard_normal(n)
            z[3 * i + 2, V // 2] = np.inf
        B = z.shape[0]
        u = workload.uniforms(1, B, seed=V + k)[0]
        out = torch.empty(B, dtype=torch.int32, device="cuda")
        print(f"sampler with few finite entries: V={V} k={k}", flush=True)
        ftts.sample(torch.from_numpy(z).cuda(), ftts.Sampling(T, k, p), torch.from_numpy(u).cuda(), out)
        got = out.cpu().numpy()
        for b in range(B):
            with np.errstate(invalid="ignore"):
                want, det = osample.sample(z[b], T, k, p, u[b])
            assert got[b] == want or osample.near_boundary(det), (T, k, p, b, got[b], want)


def us_per_call(z, k, temperature=0.8, calls=100):
    import torch
    from paper_2607_21042_amd import ftts
    u = torch.from_numpy(workload.uniforms(1, z.shape[0], seed=9)[0]).cuda()
    out = torch.empty(z.shape[0], dtype=torch.int32, device="cuda")
    ftts.sample(z, ftts.Sampling(temperature, k, 0.8), u, out)
    best = 1e9
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(calls):
            ftts.sample(z, ftts.Sampling(temperature, k, 0.8), u, out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1000 / calls)
    return best


def test_short_and_masked_rows_take_the_fast_path():
    """A row of fewer than 4 k entries, or masked to a short run, costs no more than a
    full row of 8194: the ranked list serves both (k rounds of block argmax, which only
    a crowd of exact ties takes, would be several times slower).  The bar of 1.5 leaves
    room for timing noise: these rows read less and rank about as many entries."""
    import torch
    full = torch.from_numpy(workload.random_logits(32, 8194, seed=5)).cuda()
    masked = torch.full_like(full, float("-inf"))
    masked[:, 4000:4090] = full[:, 4000:4090]
    t = {name: us_per_call(z, 30) for name, z in
         (("full", full), ("short", full[:, :100].contiguous()), ("masked", masked))}
    print(f"sampler us per call: {t}", flush=True)
    assert t["short"] <= 1.5 * t["full"] and t["masked"] <= 1.5 * t["full"], t


def test_small_top_k_over_many_rows_stays_near_the_read():
    """1024 rows of 16384 fill the chip and are bound by reading the logits, which the
    greedy choice does and little else: a small top-k adds a few short steps (measured
    1.2 of greedy's time; 1.8 with a threshold from all 256 group maxima)."""
    import torch
    z = torch.from_numpy(workload.random_logits(1024, 16384, seed=6)).cuda()
    t = {k: us_per_call(z, k) for k in (1, 2, 5)}
    print(f"sampler us per call of 1024 rows: {t}", flush=True)
    assert max(t[2], t[5]) <= 1.5 * t[1], t


def test_rows_masked_with_a_finite_value_take_the_ranked_list():
    """A run of 90 entries, the rest at float32's lowest value or at -1e4: the crowd of
    equal entries may not send the row to k rounds of block argmax (57 us for 32 rows)."""
    import torch
    full = torch.from_numpy(workload.random_logits(32, 8194, seed=5)).cuda()
    t = {"full": us_per_call(full, 30, temperature=1.0)}
    for low in (float(np.finfo(np.float32).min), -1e4):
        for V, at in ((8194, 4000), (1024, 500)):
            z = torch.full((32, V), low, device="cuda")
            z[:, at:at + 90] = full[:, at:at + 90]
            t[low, V] = us_per_call(z, 30, temperature=1.0)
    print(f"sampler us per call: {t}", flush=True)
    assert max(t.values()) <= 2 * t["full"], t


@pytest.mark.parametrize("low", [-np.inf, float(np.finfo(np.float32).min), -1e4])
@pytest.mark.parametrize("k", [2, 9, 16, 30, 32, 64])
def test_sampler_masked_rows_around_the_lines(k, low):
    """V = 16384 with all but some entries masked, by -inf or a finite value: runs whose threads number 127 to 129
    (the line for taking every entry above -inf), longer runs, and entries at the same
    few threads' slots only (2048 of them: more than the candidate list holds)."""
    import torch
    from paper_2607_21042_amd import ftts
    V = 16384
    src = workload.random_logits(1, V, seed=k)[0]
    rows = []
    for n in (127, 128, 129, 300, 1000, 1025):
        for at in (0, 1000, V - n):
            z = np.full(V, low, np.float32)
            z[at:at + n] = src[at:at + n]
            rows.append(z)
    for threads in (4, 64, 128, 129, 200):
        z = np.full(V, low, np.float32)
        keep = np.arange(V) % 1024 < threads
        z[keep] = src[keep]
        rows.append(z)
    z = np.stack(rows)
    u = workload.uniforms(1, len(rows), seed=k + 1)[0]
    out = torch.empty(len(rows), dtype=torch.int32, device="cuda")
    print(f"sampler, masked rows around the lines: k={k}", flush=True)
    ftts.sample(torch.from_numpy(z).cuda(), ftts.Sampling(1.1, k, 0.95), torch.from_numpy(u).cuda(), out)
    got = out.cpu().numpy()
    for b in range(len(rows)):
        want, det = osample.sample(z[b], 1.1, k, 0.95, u[b])
        assert got[b] == want or osample.near_boundary(det), (k, b, got[b], want)
