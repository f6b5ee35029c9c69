"""The one-launch selection of short archives at its edges: row counts around its
register tiles and its upper limit, budgets from 1 to all rows, keys with far
outliers (the histogram must be refined), many ties and duplicated rows.  Bit for
bit against the oracle's selection; and the row flags it leaves, which the
admission reads: a row flagged wrongly would be admitted twice or not at all.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A,k", [(1, 1), (63, 63), (64, 3), (65, 64), (511, 100), (8191, 8191), (8192, 1), (8193, 1024),
                                 (16383, 500), (16384, 16000), (16385, 500)])
@pytest.mark.parametrize("kind", ["plain", "outliers", "ties", "copies"])
def test_short_archives(A, k, kind):
    print(f"[select-small] A={A} k={k} {kind}", flush=True)
    B, H, W = 2, 5, 3
    T = A + W
    cfg = synth.CONFIGS["cfg1"].with_(B=B, H=H, T=T, W=W, k=k, needles=0)
    wl = synth.make_workload(cfg, "cuda", seed=A + k)
    g = torch.Generator(device="cuda")
    g.manual_seed(A)
    if kind == "outliers":
        at = torch.randint(0, A, (3,), generator=g, device="cuda")
        wl["cache"][:, at] *= 4096.0
    if kind == "ties":
        wl["cache"][:, :, 512:] = torch.randint(-1, 2, (B, T, 64), generator=g, device="cuda").to(torch.bfloat16)
        wl["q_rope"][:] = torch.randint(-1, 2, (B, H, 64), generator=g, device="cuda").to(torch.bfloat16)
    if kind == "copies":
        wl["cache"][:, :, 512:] = wl["cache"][:, torch.randint(0, max(1, A // 50), (T,), generator=g, device="cuda"), 512:]
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, synth.MODE_ROPE)
    bufs = vkv.Buffers(step, k)
    ctx = vkv.Context(0)
    bufs.run(ctx, step, cfg.scale)
    torch.cuda.synchronize()
    ctx.close()
    bits = [synth.to_numpy_bits(wl[n]) for n in ("cache", "q_lat", "q_rope")]
    res = oracle.step(bits[0], bits[1], bits[2], None, None, 0, synth.MODE_ROPE, W, k, cfg.scale)
    for b in range(B):
        assert np.array_equal(bufs.sel[b].cpu().numpy(), res["sel"][b])
        assert float(bufs.theta[b]) == float(res["theta"][b])


@pytest.mark.parametrize("A,k", [(1, 1), (64, 63), (65, 3), (4097, 500), (8192, 2000), (8193, 1), (16383, 16000),
                                 (16384, 700), (16385, 700)])
def test_the_flags_the_admission_reads(A, k):
    print(f"[select-small] flags A={A} k={k}", flush=True)
    B, H, W, r, cm = 2, 5, 3, 64, 0.3
    T = A + W
    cfg = synth.CONFIGS["cfg4"].with_(B=B, H=H, T=T, W=W, k=k, needles=0, basis="orthonormal")
    wl = synth.make_workload(cfg, "cuda", seed=A + k)
    index = torch.empty(B, T, 64 + r, dtype=torch.bfloat16, device="cuda")
    sc = [torch.empty(B, T, device="cuda") for _ in range(3)]
    ctx = vkv.Context(0)
    vkv.digest_build(ctx, wl["cache"], wl["P"], r, True, index, *sc)
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, synth.MODE_ROPE_DIGEST, r, index=index, P=wl["P"], eta=sc[0],
                    eps=sc[1], gam=sc[2])
    bufs = vkv.Buffers(step, k, two_tier=True, cert_mult=cm)
    bufs.ws.fill_(1)   # (a flag that is not written reads as a selected row)
    bufs.run(ctx, step, cfg.scale)
    torch.cuda.synchronize()
    ctx.close()
    bits = [synth.to_numpy_bits(wl[n]) for n in ("cache", "q_lat", "q_rope", "P")]
    oidx, *osc = oracle.digest_build(bits[0], bits[3], r, with_rope=True, scalars=True)
    res = oracle.step(bits[0], bits[1], bits[2], oidx, bits[3], r, synth.MODE_ROPE_DIGEST, W, k, cfg.scale, two_tier=True,
                      eta=osc[0], eps=osc[1], gam=osc[2], cert_mult=cm)
    for b in range(B):
        assert np.array_equal(bufs.sel[b].cpu().numpy(), res["sel"][b])
        n = int(bufs.adm_count[b])
        assert n == res["adm_count"][b] and np.array_equal(bufs.adm[b, :n].cpu().numpy(), np.asarray(res["adm"][b])[:n])
