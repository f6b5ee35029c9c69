"""The basis iteration of vkv_sketch_basis against the same iteration written
with numpy (Householder QR with positive diagonal in place of Cholesky QR).

The iteration V <- orth(C V) from the fixed start pattern determines V column
by column, so the bf16 basis must be RNE(s V^T) up to fp64 rounding: each
entry within half a bf16 ulp (8 significant bits: 2^-8 relative) plus 1e-7, which covers the fp64
error (condition number of the columns, below 1e7 here by the kernel's own
check, times 2^-53, with a factor 100).  Ranks around the 64-column panels
(one panel, a 32-column remainder, eight panels), query counts around the
64-query chunks of the second moment.
"""
import numpy as np
import pytest
import torch

import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu


def start_pattern(r):
    h = (np.arange(512 * 512, dtype=np.uint64).reshape(512, 512)[:, :r] + np.uint64(0x5BD1E995)) & np.uint64(0xFFFFFFFF)
    for mul in (0x85EBCA6B, 0xC2B2AE35):
        h = ((h ^ (h >> np.uint64(16 if mul == 0x85EBCA6B else 13))) * np.uint64(mul)) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(16)
    return np.where(h >> np.uint64(31), 1.0, -1.0)


def basis(ctx, q, r, iters):
    ws = torch.empty(vkv.sketch_workspace_size(r), dtype=torch.uint8, device="cuda")
    P = torch.empty(r, 512, dtype=torch.bfloat16, device="cuda")
    energy = torch.empty(2, dtype=torch.float64, device="cuda")
    vkv.sketch_basis(ctx, q, r, iters, ws, P, energy)
    return P.double().cpu().numpy(), energy.cpu().numpy()


@pytest.mark.parametrize("m,r,iters,queries", [
    (100, 32, 0, "gaussian"), (511, 96, 3, "lowrank"), (4097, 64, 8, "lowrank"), (3000, 160, 2, "gaussian"),
    (2500, 512, 1, "gaussian"), (64, 32, 2, "gaussian"), (65, 64, 0, "gaussian"),
])
def test_basis_is_the_iteration(m, r, iters, queries):
    print(f"[sketch-iteration] m={m} r={r} iters={iters} {queries}", flush=True)
    cfg = synth.CONFIGS["cfg0"].with_(queries=queries)
    q = synth.prefix_queries(cfg, m, "cuda")
    ctx = vkv.Context(0)
    P, energy = basis(ctx, q, r, iters)
    ctx.close()
    x = q.double().cpu().numpy()
    C = x.T @ x
    V = start_pattern(r)
    for _ in range(iters + 1):
        V, R = np.linalg.qr(C @ V)
        V = V * np.sign(np.diagonal(R))
    want = (1.0 - 2.0 ** -6) * V.T
    assert np.all(np.abs(P - want) <= 2.0 ** -8 * np.abs(want) + 1e-7)
    assert abs(energy[0] - np.sum(V * (C @ V))) <= 1e-9 * energy[0]
    assert abs(energy[1] - np.trace(C)) <= 1e-12 * energy[1]


@pytest.mark.parametrize("m,r", [(31, 32), (63, 64), (90, 96), (300, 512)])
def test_queries_of_lower_rank_are_refused(m, r):
    q = synth.prefix_queries(synth.CONFIGS["cfg0"], m, "cuda")
    ctx = vkv.Context(0)
    with pytest.raises(vkv.VkvError):
        basis(ctx, q, r, 4)
    ctx.close()
