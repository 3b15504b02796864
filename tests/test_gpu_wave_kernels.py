"""Kernels whose wavefronts split the reduction (projections) or the keys
(fp32 attention), at the edges of their tiles and chunks, against fp64."""
import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(77)


# fp32 projections: 16 x 16 tiles (with fewer K chunks than waves; element by
# element where a row is no multiple of 16 bytes), 32 x 32 and 64 x 64 tiles,
# each with a ragged last tile and a short last chunk
@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (16, 16, 16), (17, 33, 20), (33, 18, 132), (9, 50, 7), (40, 24, 1),
                                   (33, 500, 1021), (500, 300, 36), (460, 512, 256), (1000, 800, 52), (770, 1030, 130)])
def test_projection_f32_edges(M, N, K):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[gemm f32] M={M} N={N} K={K}")
    A = RNG.standard_normal((M, K)).astype(np.float32)
    W = RNG.standard_normal((N, K)).astype(np.float32)
    bias = RNG.standard_normal(N).astype(np.float32)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias
    out = vla.debug_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda(), bias=torch.from_numpy(bias).cuda())
    torch.cuda.synchronize()
    # each of the K products and sums rounds once: |error| <= K 2^-24 sum |a w|,
    # in practice its square root; a few of those
    bound = 4 * np.sqrt(K) * 2.0 ** -24 * (np.abs(A) @ np.abs(W).T + np.abs(bias))
    assert (np.abs(out.cpu().numpy() - ref) <= bound + 1e-7).all()


def test_projection_f32_keeps_inf_and_nan_in_their_rows():
    """A short last chunk (K = 20) is filled with zeros on both sides: an
    infinity or NaN of one row reaches that row's outputs only, as such."""
    import torch
    from paper_2609_12075_amd import vla
    A, W = torch.ones(18, 20), torch.ones(24, 20)
    A[3, 19], A[17, 16] = float("inf"), float("nan")
    out = vla.debug_gemm(A.cuda(), W.cuda()).cpu()
    assert torch.isinf(out[3]).all() and torch.isnan(out[17]).all()
    keep = [m for m in range(18) if m not in (3, 17)]
    assert (out[keep] == 20).all()


# fewer keys than one tile, fewer tiles than waves, one more than a round of
# tiles, grouped heads whose rows share a tile, head dims of each padding
@pytest.mark.parametrize("B,Hq,Hkv,Lq,hd,len0,len1", [
    (1, 1, 1, 1, 8, 1, 0), (2, 4, 4, 8, 64, 15, 2), (1, 4, 2, 9, 64, 16, 0), (1, 6, 2, 17, 72, 120, 9),
    (1, 4, 1, 5, 128, 129, 0), (2, 2, 1, 16, 200, 250, 7), (1, 2, 2, 33, 256, 40, 1)])
def test_attention_f32_edges(B, Hq, Hkv, Lq, hd, len0, len1):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[attn f32] B={B} Hq={Hq} Hkv={Hkv} Lq={Lq} hd={hd} len0={len0} len1={len1}")
    g = torch.Generator().manual_seed(hd + len0)
    rnd = lambda *s: torch.randn(*s, generator=g)
    q, k0, v0 = rnd(B, Hq, Lq, hd), rnd(B, Hkv, len0, hd), rnd(B, Hkv, len0, hd)
    k1, v1 = (rnd(B, Hkv, len1, hd), rnd(B, Hkv, len1, hd)) if len1 else (None, None)
    c = lambda t: None if t is None else t.cuda()
    got = vla.debug_attention(c(q), c(k0), c(v0), c(k1), c(v1)).cpu()
    k, v = (x if y is None else torch.cat([x, y], 2) for x, y in ((k0, k1), (v0, v1)))
    k, v = (x.double().repeat_interleave(Hq // Hkv, 1) for x in (k, v))
    p = torch.softmax(q.double() @ k.transpose(2, 3) / hd ** 0.5, -1)
    ref = (p @ v).transpose(1, 2).reshape(B, Lq, Hq * hd)
    np.testing.assert_allclose(got.numpy(), ref.numpy(), rtol=1e-4, atol=2e-6)
