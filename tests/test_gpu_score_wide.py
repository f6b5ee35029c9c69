"""The scan where heads x width exceed one wave's query registers (more than 64
heads from 160 dims, any head count from 288 dims): the block's waves share the
heads of every tile.  Selection, theta, the admitted set and the outputs against
the oracle, with every width from 160 to 576 dims, head counts around the parts
(32, 64, 96, 128 heads) and ragged contexts; and the margins-only scan of the
kept step, whose fired set must match the two-buffer form's.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu
SCALE = 1.0 / np.sqrt(192.0)


def build(ctx, B, H, T, W, mode, r, seed, cert):
    cfg = synth.CONFIGS["cfg4"].with_(B=B, H=H, T=T, W=W, k=1, r=r, mode=mode, needles=5)
    wl = synth.make_workload(cfg, "cuda", seed=seed)
    index = torch.empty(B, T, (64 if mode & 1 else 0) + r, dtype=torch.bfloat16, device="cuda")
    sc = [torch.empty(B, T, device="cuda") for _ in range(3)] if cert else [None] * 3
    vkv.digest_build(ctx, wl["cache"], wl["P"], r, bool(mode & 1), index, *sc)
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, mode, r, index=index, index_has_rope=bool(mode & 1),
                    P=wl["P"], eta=sc[0], eps=sc[1], gam=sc[2])
    return wl, step


@pytest.mark.parametrize("H,mode,r", [
    (65, 3, 96), (128, 2, 160), (100, 3, 128), (97, 3, 160), (128, 2, 256), (1, 2, 288), (33, 3, 256), (128, 3, 256),
    (32, 2, 320), (64, 2, 352), (65, 3, 320), (17, 3, 352), (96, 2, 448), (128, 3, 416), (128, 2, 512), (31, 3, 480),
    (128, 3, 512), (40, 3, 512)])
@pytest.mark.parametrize("T,W,admit", [(1031, 7, False), (4500, 100, True), (17, 1, False)])
def test_wide_scan_selects_exactly(H, mode, r, T, W, admit):
    if admit and mode == 2:
        pytest.skip("the bound needs the branch in the key")
    print(f"[score-wide] H={H} mode={mode} r={r} T={T} W={W} admit={admit}", flush=True)
    ctx = vkv.Context(0)
    B = 2
    wl, step = build(ctx, B, H, T, W, mode, r, T + r, admit)
    k = max(1, (T - W) // 9)
    bufs = vkv.Buffers(step, k, two_tier=admit, cert_mult=0.2 if admit else 1.0)
    bufs.run(ctx, step, SCALE)
    torch.cuda.synchronize()
    ctx.close()
    bits = [synth.to_numpy_bits(wl[n]) for n in ("cache", "q_lat", "q_rope", "P")]
    oidx, *sc = oracle.digest_build(bits[0], bits[3], r, with_rope=bool(mode & 1), scalars=admit)
    kw = dict(two_tier=True, eta=sc[0], eps=sc[1], gam=sc[2], cert_mult=0.2) if admit else {}
    res = oracle.step(bits[0], bits[1], bits[2], oidx, bits[3], r, mode, W, k, SCALE, index_has_rope=bool(mode & 1), **kw)
    for b in range(B):
        assert np.array_equal(bufs.sel[b].cpu().numpy(), res["sel"][b])
        assert float(bufs.theta[b]) == float(res["theta"][b])
        if admit:
            n = int(bufs.adm_count[b])
            assert np.array_equal(bufs.adm[b, :n].cpu().numpy(), np.asarray(res["adm"][b])[:n]) and n == len(res["adm"][b])
        o = bufs.out[b].float().cpu().numpy().astype(np.float64)
        w = res["out"][b]
        assert np.max(np.linalg.norm(o - w, axis=1) / np.linalg.norm(w, axis=1)) < 2e-2


@pytest.mark.parametrize("H,r", [(128, 192), (70, 416), (64, 512), (128, 512)])
def test_margins_without_keys(H, r):
    ctx = vkv.Context(0)
    B, T, W, k = 2, 9000, 64, 500
    wl, step = build(ctx, B, H, T, W, 3, r, r, True)
    A = T - W
    kept = torch.stack([torch.randperm(A, generator=torch.Generator().manual_seed(b))[:k].sort().values
                        for b in range(B)]).to(torch.int32).cuda()
    got = []
    for key in (None, torch.empty(B, A, device="cuda")):
        ws = vkv.alloc_workspace(step, k, A)
        ub = torch.empty(B, A, device="cuda")
        smax, arg = torch.empty(B, H, dtype=torch.float64, device="cuda"), torch.empty(B, H, dtype=torch.int32, device="cuda")
        fired = torch.full((B, A), -1, dtype=torch.int32, device="cuda")
        cnt = torch.empty(B, dtype=torch.int32, device="cuda")
        out = torch.empty(B, H, 512, dtype=torch.bfloat16, device="cuda")
        lse = torch.empty(B, H, device="cuda")
        vkv.step_run_kept(ctx, step, ws, k, kept, key, ub, 0.05, smax, arg, 0, fired, cnt, A, SCALE, out, lse)
        torch.cuda.synchronize()
        got.append((ub, fired, cnt, out, lse))
    ctx.close()
    assert all(torch.equal(x, y) for x, y in zip(*got)) and int(got[0][2].sum()) > 0


@pytest.mark.parametrize("H,r,T", [(16, 64, 3000), (128, 64, 3000), (70, 160, 4000), (128, 192, 5000), (40, 512, 3000)])
def test_masked_rows_leave_the_admission_of_the_others(H, r, T):
    """Rows filled with the type's lowest value have an infinite certificate scalar;
    the bound's error term is then infinite, no more, and every row's exact bound
    decides: the other rows' selection and admission are the oracle's."""
    print(f"[score-wide] masked rows H={H} r={r} T={T}", flush=True)
    ctx = vkv.Context(0)
    B, W, k = 2, 8, 100
    cfg = synth.CONFIGS["cfg4"].with_(B=B, H=H, T=T, W=W, k=1, r=r, mode=3, needles=5, basis="orthonormal")
    wl = synth.make_workload(cfg, "cuda", seed=T + r)
    masked = np.arange(3, T, 97)
    wl["cache"][:, torch.from_numpy(masked).cuda()] = float(torch.finfo(torch.bfloat16).min)
    index = torch.empty(B, T, 64 + r, dtype=torch.bfloat16, device="cuda")
    sc = [torch.empty(B, T, device="cuda") for _ in range(3)]
    vkv.digest_build(ctx, wl["cache"], wl["P"], r, True, index, *sc)
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, 3, r, index=index, P=wl["P"], eta=sc[0], eps=sc[1], gam=sc[2])
    A, cm = step.A, 0.2
    ws = vkv.alloc_workspace(step, k)
    sel = torch.empty(B, k, dtype=torch.int32, device="cuda")
    theta = torch.empty(B, dtype=torch.float64, device="cuda")
    ub, adm = torch.empty(B, A, device="cuda"), torch.full((B, A), -1, dtype=torch.int32, device="cuda")
    cnt = torch.empty(B, dtype=torch.int32, device="cuda")
    vkv.query_prep(ctx, step, ws)
    vkv.score(ctx, step, ws, None, ub, cert_mult=cm)
    vkv.select(ctx, step, ws, k, sel, theta)
    vkv.admit(ctx, step, ws, k, sel, theta, ub, adm, cnt, A, cert_mult=cm)
    torch.cuda.synchronize()
    ctx.close()
    bits = [synth.to_numpy_bits(wl[n]) for n in ("cache", "q_lat", "q_rope", "P")]
    # the oracle on the same keys: the masked rows' own keys are what they are
    qt, a, nq, e = oracle.query_prep(bits[1], bits[2], bits[3], r, 3)
    for b in range(B):
        x = oracle.index_rows(bits[0][b], synth.to_numpy_bits(index[b]), 3, r, True)
        s = [v[b].cpu().numpy() for v in sc]
        th = float(theta[b])
        UB = oracle.upper_bounds(qt[b], a[b], nq[b], e[b], x, *s, A, cert_mult=cm)
        want = np.setdiff1d(np.flatnonzero(UB > th), np.concatenate([sel[b].cpu().numpy(), masked]))
        got = np.setdiff1d(adm[b, :int(cnt[b])].cpu().numpy(), masked)
        assert len(want) > 0 and np.array_equal(got, want)
