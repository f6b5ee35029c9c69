"""The exact row maximum where its ranges, row classes and merge can go wrong:
copies of the best row in one row class (16 positions apart) and across the
ranges that are scanned in parallel, rows of very different norms, contexts
around the 32-row tiles and the shortest ranges, few and many heads.  Bit for bit
against the fp64 oracle, and the same on every repetition (the ranges of a call
without scratch meet in the outputs in no fixed order).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,T,W,copies", [(1, 1, 1, 0, 0), (1, 17, 31, 3, 4), (2, 16, 33, 33, 2), (1, 128, 257, 0, 12),
                                            (3, 40, 1027, 130, 40), (1, 16, 50021, 77, 300), (2, 128, 9001, 512, 100),
                                            (1, 5, 8192, 8192, 20)])
def test_row_max_over_ranges(B, H, T, W, copies):
    print(f"[row-max] B={B} H={H} T={T} W={W} copies={copies}", flush=True)
    cfg = synth.CONFIGS["cfg1"].with_(B=B, H=H, T=T, W=W, k=0, needles=0, rows="lognormal")
    wl = synth.make_workload(cfg, "cuda", seed=T)
    rng = np.random.default_rng(T)
    cache = wl["cache"]
    q = torch.cat([wl["q_lat"], wl["q_rope"]], 2).double()
    for b in range(B):
        if copies:
            best = int((q[b, 0] @ cache[b].double().T).argmax())
            at = np.concatenate([np.arange(best % 16, min(T, 16 * copies), 16), rng.integers(0, T, copies)])
            cache[b, torch.from_numpy(at).cuda()] = cache[b, best].clone()
    step = vkv.Step(cache, wl["q_lat"], wl["q_rope"], W, synth.MODE_ROPE)
    A = T - W
    lists = torch.from_numpy(np.stack([np.sort(rng.choice(A, A // 3, replace=False)) for _ in range(B)])
                             .astype(np.int32)).cuda() if A >= 3 else None
    ctx = vkv.Context(0)
    smax = torch.empty(B, H, dtype=torch.float64, device="cuda")
    arg = torch.empty(B, H, dtype=torch.int32, device="cuda")
    bits, ql, qr = (synth.to_numpy_bits(t) for t in (cache, wl["q_lat"], wl["q_rope"]))
    for rows, recent in [(None, True), (None, False), (lists, True), (lists, False)]:
        want = [oracle.row_max(ql[b], qr[b], bits[b], np.concatenate(
            [np.arange(A, dtype=np.int32) if rows is None else rows[b].cpu().numpy(),
             np.arange(A, T, dtype=np.int32) if recent else np.zeros(0, np.int32)])) for b in range(B)]
        for _ in range(3):
            smax.fill_(7.0)
            arg.fill_(5)
            vkv.row_max(ctx, step, rows, recent, smax, arg)
            got_s, got_a = smax.cpu().numpy(), arg.cpu().numpy()
            for b in range(B):
                assert np.array_equal(got_s[b], want[b][0])
                assert np.array_equal(got_a[b], want[b][1])
    ctx.close()


@pytest.mark.parametrize("where", ["device", "smax off 8", "argmax off 4", "pinned host"])
def test_outputs_that_take_no_atomics(where):
    """Outputs that are not naturally aligned, or lie in host memory, take one range
    a sequence and plain stores; the result and the bytes around it are the same."""
    B, H, T, W = 2, 24, 6000, 40
    wl = synth.make_workload(synth.CONFIGS["cfg1"].with_(B=B, H=H, T=T, W=W, k=0, needles=3), "cuda", seed=11)
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, synth.MODE_ROPE)
    n = B * H
    so, ao = 8 + (4 if where == "smax off 8" else 0), 8 + (2 if where == "argmax off 4" else 0)
    host = where == "pinned host"
    raw = [torch.full((size,), 0x5A, dtype=torch.uint8, device="cpu" if host else "cuda") for size in (8 * n + 32, 4 * n + 32)]
    if host:
        raw = [t.pin_memory() for t in raw]
    ctx = vkv.Context(0)
    ctx.check(ctx.lib.vkv_row_max(ctx.handle, step.ref, None, 0, 1, raw[0].data_ptr() + so, raw[1].data_ptr() + ao, None))
    torch.cuda.synchronize()
    ctx.close()
    s, a = (t.cpu().numpy() for t in raw)
    assert (s[:so] == 0x5A).all() and (s[so + 8 * n:] == 0x5A).all()
    assert (a[:ao] == 0x5A).all() and (a[ao + 4 * n:] == 0x5A).all()
    gs = np.frombuffer(s[so:so + 8 * n].tobytes(), np.float64).reshape(B, H)
    ga = np.frombuffer(a[ao:ao + 4 * n].tobytes(), np.int32).reshape(B, H)
    bits, ql, qr = (synth.to_numpy_bits(wl[x]) for x in ("cache", "q_lat", "q_rope"))
    for b in range(B):
        ws, wa = oracle.row_max(ql[b], qr[b], bits[b], np.arange(T, dtype=np.int32))
        assert np.array_equal(gs[b], ws) and np.array_equal(ga[b], wa)
