"""The index build at the edges of its tiles (16 rows), groups (256 rows),
blocks (1 to 4 groups) and basis chunks (64 rows): rows, scalars and the branch
copy bit for bit against the fp64 oracle, and nothing written past a row's
columns or past the last row.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,r,with_rope,cert", [
    (1, 1, 64, True, True), (2, 15, 32, True, True), (1, 16, 64, False, False), (1, 17, 96, True, True),
    (3, 255, 160, True, True), (1, 257, 64, True, True), (2, 272, 512, False, True), (1, 1041, 0, True, True),
    (520, 257, 64, True, True), (700, 529, 32, True, False), (1100, 513, 64, True, True),
    (1, 1041, 512, True, False), (2, 272, 96, False, False), (520, 300, 64, True, False),
])
def test_index_build_edges(B, T, r, with_rope, cert):
    print(f"[digest-edges] B={B} T={T} r={r} rope={with_rope} cert={cert}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(B + T)
    # rows spread over many octaves, with zeros: other summation orders give other bits
    cache = torch.randn(B, T, 576, generator=g, device="cuda")
    cache = (cache * torch.exp2(torch.randint(-12, 12, (B, T, 576), generator=g, device="cuda").float()))
    cache[:, ::7, ::5] = 0
    cache = cache.to(torch.bfloat16)
    P = synth.make_basis("orthonormal", r)
    cols = (64 if with_rope else 0) + r
    ld = cols + 8
    index = torch.full((B, T + 1, ld), 3.0, dtype=torch.bfloat16, device="cuda")
    sc = [torch.full((B * T + 1,), -5.0, device="cuda") for _ in range(3)] if cert else [None] * 3
    ctx = vkv.Context(0)
    Pd = P.cuda() if P is not None else None
    ptr = lambda t: None if t is None else t.data_ptr()   # noqa: E731
    ctx.check(ctx.lib.vkv_digest_build(ctx.handle, ptr(cache), B, T, 576, T * 576, ptr(Pd), r, int(with_rope),
                                       ptr(index), ld, (T + 1) * ld, ptr(sc[0]), ptr(sc[1]), ptr(sc[2]), None))
    torch.cuda.synchronize()
    ctx.close()
    assert torch.all(index[:, T] == 3.0) and torch.all(index[:, :, cols:] == 3.0)
    if cert:
        assert all(float(s[B * T]) == -5.0 for s in sc)
    for b in sorted({0, B // 2, B - 1}):
        bits = synth.to_numpy_bits(cache[b:b + 1])
        idx, eta, eps, gam = oracle.digest_build(bits, synth.to_numpy_bits(P) if r else None, r, with_rope=with_rope,
                                                 scalars=cert)
        got = synth.to_numpy_bits(index[b:b + 1, :T, :cols].contiguous())
        assert np.array_equal(got, np.asarray(idx).reshape(got.shape))
        if cert:
            for s, want in zip(sc, (eta, eps, gam)):
                assert np.array_equal(s[b * T:(b + 1) * T].cpu().numpy(), np.asarray(want).reshape(-1))


@pytest.mark.parametrize("name,r,ok", [("identity", 64, True), ("identity", 512, True), ("above", 64, False),
                                       ("overlap", 96, False), ("inside", 160, True), ("zero", 32, True),
                                       ("nan", 64, False)])
def test_contractivity_verdict(name, r, ok):
    """Bases on, above and inside the bound: exact row sums of 1 pass (the sequential
    check), anything above does not, and the quick check alone serves the rest."""
    P = torch.eye(512, dtype=torch.float64)[:r]
    if name == "above":
        P[3, 3] = 1.0078125                       # the next bf16 above 1
    if name == "overlap":
        P[1, 0] = 2.0 ** -20                      # row sums 1 + 2^-20 and above
    if name == "inside":
        P = P * 0.75
        P[:, 300] += 2.0 ** -10
    if name == "zero":
        P = P * 0
    if name == "nan":
        P[5, 7] = float("nan")
    T = 40
    cache = torch.randn(1, T, 576, device="cuda").to(torch.bfloat16)
    index = torch.full((1, T, 64 + r), 3.0, dtype=torch.bfloat16, device="cuda")
    sc = [torch.full((1, T), -5.0, device="cuda") for _ in range(3)]
    ctx = vkv.Context(0)
    if ok:
        vkv.digest_build(ctx, cache, P.to(torch.bfloat16).cuda(), r, True, index, *sc)
        torch.cuda.synchronize()
        assert all(bool((s >= 0).all()) for s in sc)
    else:
        with pytest.raises(vkv.VkvError) as e:
            vkv.digest_build(ctx, cache, P.to(torch.bfloat16).cuda(), r, True, index, *sc)
        assert e.value.code == -5 and bool((index == 3.0).all()) and all(bool((s == -5.0).all()) for s in sc)
    ctx.close()
