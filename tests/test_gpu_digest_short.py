"""The index builds that have a kernel of their own: no digest (r = 0: the branch
copy and eta >= ||c||), around its 64-row blocks, and short sequences without a
certificate (up to 128 rows), around its 16-row tiles, 32- and 128-row blocks and
64-row basis chunks, against the long form just above.  Bit for bit against the fp64
oracle, and nothing written past a row's columns or past the last row.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_03949_amd as vkv
from paper_2609_03949_amd import synth

pytestmark = pytest.mark.gpu


def check(B, T, r, with_rope, cert, has_index=True, stride=576):
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * B + T)
    # rows spread over many octaves, with zeros: other summation orders give other bits
    cache = torch.randn(B, T, stride, generator=g, device="cuda")
    cache = cache * torch.exp2(torch.randint(-12, 12, (B, T, stride), generator=g, device="cuda").float())
    cache[:, ::7, ::5] = 0
    cache = cache.to(torch.bfloat16)
    P = synth.make_basis("orthonormal", r) if r else None
    cols = (64 if with_rope else 0) + r
    ld = cols + 8
    index = torch.full((B, T + 1, ld), 3.0, dtype=torch.bfloat16, device="cuda")
    sc = [torch.full((B * T + 1,), -5.0, device="cuda") for _ in range(3)] if cert else [None] * 3
    Pd = P.cuda() if r else None
    ptr = lambda t: None if t is None else t.data_ptr()   # noqa: E731
    ctx = vkv.Context(0)
    ctx.check(ctx.lib.vkv_digest_build(ctx.handle, ptr(cache), B, T, stride, T * stride, ptr(Pd), r, int(with_rope),
                                       ptr(index) if has_index else None, ld, (T + 1) * ld, *(ptr(x) for x in sc), None))
    torch.cuda.synchronize()
    ctx.close()
    assert torch.all(index[:, T] == 3.0) and torch.all(index[:, :, cols:] == 3.0)
    if cert:
        assert all(float(x[B * T]) == -5.0 for x in sc)
    for b in sorted({0, B // 2, B - 1}):
        bits = synth.to_numpy_bits(cache[b:b + 1, :, :576].contiguous())
        idx, *want = oracle.digest_build(bits, synth.to_numpy_bits(P) if r else None, r, with_rope=with_rope, scalars=cert)
        if has_index and cols:
            got = synth.to_numpy_bits(index[b:b + 1, :T, :cols].contiguous())
            assert np.array_equal(got, np.asarray(idx).reshape(got.shape))
        if cert:
            for x, w in zip(sc, want):
                assert np.array_equal(x[b * T:(b + 1) * T].cpu().numpy(), np.asarray(w).reshape(-1))


@pytest.mark.parametrize("B,T,with_rope,cert,has_index", [
    (1, 1, True, True, True), (3, 63, True, False, True), (2, 64, True, True, True), (1, 65, False, True, True),
    (2, 1000, True, True, False), (300, 129, True, True, True)])
@pytest.mark.parametrize("stride", [576, 640])
def test_index_without_a_digest(B, T, with_rope, cert, has_index, stride):
    print(f"[digest-plain] B={B} T={T} rope={with_rope} cert={cert} index={has_index} stride={stride}", flush=True)
    check(B, T, 0, with_rope, cert, has_index, stride)


@pytest.mark.parametrize("B,T,r,with_rope", [
    (1, 1, 64, True), (1, 16, 32, False), (2, 17, 96, True), (3, 31, 512, True), (1, 32, 160, True), (5, 33, 64, True),
    (64, 127, 64, True), (65, 128, 64, True), (300, 128, 32, False), (257, 17, 96, True), (260, 65, 160, True),
    (2, 129, 96, True)])
@pytest.mark.parametrize("stride", [576, 640])
def test_short_index_without_a_certificate(B, T, r, with_rope, stride):
    print(f"[digest-short] B={B} T={T} r={r} rope={with_rope} stride={stride}", flush=True)
    check(B, T, r, with_rope, False, True, stride)
