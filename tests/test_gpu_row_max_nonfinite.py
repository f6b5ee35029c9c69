"""The exact row maximum where the fp32 screen has nothing to go by: infinite and
NaN elements, rows filled with the type's lowest value (their squared norm is past
fp32), scores past fp32 whose fp64 value is finite, and heads with a zero query
beside such rows.  Bit for bit against the fp64 oracle (a score that is no number
never is the maximum), over the whole archive, over lists shorter and longer than
the 16 row classes of a tile, in one range and in many.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu
LOWEST = float(torch.finfo(torch.bfloat16).min)


def plant(kind, cache, ql, qr, rng):
    B, T, _ = cache.shape
    H = ql.shape[1]
    some = torch.from_numpy(rng.choice(T, max(1, T // 97), replace=False)).cuda()
    if kind == "inf_query":         # every score of the head is infinite, the sign the row's
        ql[:, H // 2, 3] = float("inf")
    if kind == "huge_query":
        ql[:, 0] *= 2.0 ** 120
    if kind == "nan_query":
        qr[:, H - 1, 5] = float("nan")
    if kind == "inf_rows":
        cache[:, some, 7] = float("inf")
        cache[:, some[0], 9] = -float("inf")
    if kind == "nan_rows":
        cache[:, some, 70] = float("nan")
    if kind in ("masked_rows", "zero_head"):
        cache[:, some] = LOWEST
    if kind == "zero_head":
        ql[:, 0] = 0
        qr[:, 0] = 0
    if kind == "all_masked":
        cache[:] = LOWEST
    if kind == "overflow":          # partial sums past fp32 in both directions, finite in fp64
        ql *= 2.0 ** 60
        qr *= 2.0 ** 60
        cache *= 2.0 ** 62


@pytest.mark.parametrize("B,H,T,W", [(1, 1, 9, 2), (2, 17, 33, 0), (1, 5, 300, 20), (2, 40, 2077, 77), (1, 128, 9001, 64)])
@pytest.mark.parametrize("kind", ["inf_query", "huge_query", "nan_query", "inf_rows", "nan_rows", "masked_rows",
                                  "zero_head", "all_masked", "overflow"])
def test_row_max_without_finite_scores(kind, B, H, T, W):
    print(f"[row-max-nonfinite] {kind} B={B} H={H} T={T} W={W}", flush=True)
    cfg = synth.CONFIGS["cfg1"].with_(B=B, H=H, T=T, W=W, k=0, needles=0)
    wl = synth.make_workload(cfg, "cuda", seed=T)
    rng = np.random.default_rng(T)
    cache, ql, qr = wl["cache"], wl["q_lat"], wl["q_rope"]
    plant(kind, cache, ql, qr, rng)
    step = vkv.Step(cache, ql, qr, W, synth.MODE_ROPE)
    A = T - W
    lists = torch.from_numpy(np.stack([np.sort(rng.choice(A, (A + 1) // 2, replace=False)) for _ in range(B)])
                             .astype(np.int32)).cuda()
    smax = torch.empty(B, H, dtype=torch.float64, device="cuda")
    arg = torch.empty(B, H, dtype=torch.int32, device="cuda")
    bits = [synth.to_numpy_bits(t) for t in (ql, qr, cache)]
    ctx = vkv.Context(0)
    for rows, recent in [(None, True), (None, False), (lists, True), (lists, False)]:
        vkv.row_max(ctx, step, rows, recent, smax, arg)
        got_s, got_a = smax.cpu().numpy(), arg.cpu().numpy()
        for b in range(B):
            every = np.concatenate([np.arange(A) if rows is None else rows[b].cpu().numpy(),
                                    np.arange(A, T) if recent else np.zeros(0)]).astype(np.int32)
            want_s, want_a = oracle.row_max(*(x[b] for x in bits), every)
            assert np.array_equal(got_s[b], want_s)
            assert np.array_equal(got_a[b], want_a)
    ctx.close()
