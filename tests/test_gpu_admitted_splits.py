"""The attention's splits of admitted rows hold at most 1024 rows, whatever
their capacity: a list of admitted rows gives the same bits with a capacity of
1024 rows per workgroup (4096 rows over the 4 workgroups that 64 sequences of 16
heads leave each) and with more than twice that, and the same as the oracle
within the path's tolerance.  (Longer splits for larger capacities would merge
fewer partials, in other bits, and leave a few thousand admitted rows to one
workgroup.)
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

from _checks import LSE_TOL, OUT_TOL, rel_l2

pytestmark = pytest.mark.gpu
SCALE = 1.0 / np.sqrt(192.0)


@pytest.mark.parametrize("n", [0, 1, 1025, 2048, 3333, 4096])
def test_capacity_does_not_change_the_attention(n):
    print(f"[admitted-splits] n={n}", flush=True)
    B, H, T, W, k = 64, 16, 9200, 32, 64
    cfg = synth.CONFIGS["cfg1"].with_(B=B, H=H, T=T, W=W, k=k, needles=0)
    wl = synth.make_workload(cfg, "cuda", seed=n)
    step = vkv.Step(wl["cache"], wl["q_lat"], wl["q_rope"], W, synth.MODE_ROPE)
    rng = np.random.default_rng(n)
    perm = np.stack([rng.permutation(step.A)[:k + n] for _ in range(B)]).astype(np.int32)
    sel, adm = np.sort(perm[:, :k]), np.sort(perm[:, k:])
    ctx = vkv.Context(0)
    got = []
    for cap in (4096, 9000):
        lists = torch.full((B, cap), -1, dtype=torch.int32)
        lists[:, :n] = torch.from_numpy(adm)
        ws = vkv.alloc_workspace(step, k, cap)
        out = torch.empty(B, H, 512, dtype=torch.bfloat16, device="cuda")
        lse = torch.empty(B, H, device="cuda")
        vkv.attend(ctx, step, ws, k, torch.from_numpy(sel).cuda(), lists.cuda(),
                   torch.full((B,), n, dtype=torch.int32, device="cuda"), cap, SCALE, out, lse)
        torch.cuda.synchronize()
        got.append((out, lse))
    ctx.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    for b in (0, B - 1):
        bits = [synth.to_numpy_bits(wl[x][b]) for x in ("q_lat", "q_rope", "cache")]
        o, l = oracle.attend(*bits, oracle.attend_list(sel[b], step.A, T, adm[b]), SCALE)
        assert rel_l2(got[0][0][b].double().cpu().numpy(), o) < OUT_TOL
        assert np.all(np.abs(got[0][1][b].double().cpu().numpy() - l) < LSE_TOL)
