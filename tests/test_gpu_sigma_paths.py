"""The sigma selector at the edges of its kernels' ranges.

Low-pass residual: the register transform serves kappa <= 64, the general one
the rest; both against numpy's FFT (fp64: a 4096-point transform's error is a
few ulps of the block's norm, so 1e-12 of it is far above rounding and far
below a wrong bin).  Tier selection: exact, against a stable sort, where the
keys fit the LDS list, need a sampled bracket, miss it, or overflow it.
"""
import numpy as np
import pytest
import torch

import paper_2609_03949_amd as vkv

pytestmark = pytest.mark.gpu
N = vkv.SIGMA_BLOCK


@pytest.mark.parametrize("kappa,B,nblk,stride", [(1, 1, 1, 576), (2, 2, 3, 576), (37, 1, 9, 584), (64, 3, 5, 640),
                                                 (65, 1, 2, 576), (300, 1, 1, 576)])
def test_lowpass_residual(kappa, B, nblk, stride):
    print(f"[sigma-paths] kappa={kappa} B={B} nblk={nblk} stride={stride}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(kappa)
    cache = torch.randn(B, nblk * N, stride, generator=g, device="cuda").to(torch.bfloat16)
    sigma = torch.full((B, nblk * N), -1.0, dtype=torch.float64, device="cuda")
    ws = torch.empty(vkv.sigma_workspace_size(B, nblk), dtype=torch.uint8, device="cuda")
    ctx = vkv.Context(0)
    vkv.sigma_close(ctx, cache, 0, nblk, kappa, ws, sigma)
    x = cache[:, :, 512:576].double().cpu().numpy().reshape(B, nblk, N, 64)
    f = np.fft.rfft(x, axis=2)
    f[:, :, :kappa] = 0
    want = np.linalg.norm(np.fft.irfft(f, n=N, axis=2), axis=3).reshape(B, -1)
    ctx.close()
    assert np.max(np.abs(sigma.cpu().numpy() - want)) <= 1e-12 * np.linalg.norm(x[0, 0])


def keys(kind, n, lo, rng):
    if kind == "chi":
        return np.sqrt(rng.chisquare(64, n))
    if kind == "ties":
        return np.round(rng.exponential(2.0, n) * 4) / 4
    if kind == "equal":
        return np.full(n, 3.25)
    if kind == "sparse":      # the large keys sit between the sampled places (2048 at even spacing past the sinks)
        v = rng.random(n)
        at = rng.choice(n, n // 10, replace=False)
        v[at] += 100.0
        sampled = lo + max(1, (n - lo) // 2048) * np.arange(2048)
        sampled = sampled[sampled < n]
        v[sampled] = rng.random(len(sampled))
        return v
    if kind == "wide":        # many octaves, zeros and infinities
        v = np.exp(rng.uniform(-600, 600, n))
        v[rng.choice(n, n // 50)] = 0.0
        v[rng.choice(n, 5)] = np.inf
        return v
    return np.sort(rng.random(n))


@pytest.mark.parametrize("kind", ["chi", "ties", "equal", "sparse", "wide", "sorted"])
@pytest.mark.parametrize("n,m,nsink", [(1, 1, 0), (64, 5, 4), (4097, 1, 4), (12288, 700, 0), (12293, 12288, 4),
                                       (131072, 4092, 4), (131073, 1, 0), (150001, 60000, 7), (131072, 131067, 4),
                                       (300000, 30000, 64), (5000, 9000, 4), (3, 2, 9)])
def test_tier_is_the_stable_order(kind, n, m, nsink):
    rng = np.random.default_rng(n + m)
    B = 2
    lo = min(nsink, n)
    v = np.stack([keys(kind, n, lo, rng) for _ in range(B)])
    if kind == "sparse" and (n, m) == (131072, 4092):
        assert np.count_nonzero(v[0] >= 100.0) > m   # the bracket, placed from the sample, lies below them all
    sigma = torch.from_numpy(v).cuda()
    K = vkv.sigma_tier_size(n, m, nsink)
    kept = torch.full((B, K), -7, dtype=torch.int32, device="cuda")
    ctx = vkv.Context(0)
    vkv.sigma_select(ctx, sigma, n, m, nsink, kept)
    got = kept.cpu().numpy()
    ctx.close()
    for b in range(B):
        order = np.argsort(-v[b, lo:], kind="stable")[:K - lo] + lo
        want = np.concatenate([np.arange(lo), np.sort(order)])
        assert np.array_equal(got[b], want)
