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


# bf16: one shape or more per tile of the plan (weight rows x activation rows
# 16 x 16, 32 x 16, 32 x 32 with a one- and a two-slot ring, 32 x 64, 64 x 64),
# with ragged last tiles, fewer chunks than waves, and K ending inside a chunk
BF16_SHAPES = [(1, 16, 8), (17, 100, 72), (50, 1000, 1096), (40, 1700, 200), (61, 2000, 1016), (100, 1500, 1240),
               (330, 1030, 1032), (300, 1300, 136), (520, 1600, 1032), (64, 9000, 4104)]


def _plan_of(M, N, K, **kw):
    from paper_2609_12075_amd import vla
    p = vla.gemm_plan(M, N, K, 0, **kw)
    return p["tile_n"], p["tile_m"], p["stages"]


def test_bf16_shapes_cover_every_tile():
    got = {_plan_of(*s, out_bf16=True) for s in BF16_SHAPES}
    assert got >= {(16, 16, 2), (32, 16, 2), (32, 32, 1), (32, 32, 2), (32, 64, 2), (64, 64, 2)}, got


@pytest.mark.parametrize("M,N,K", BF16_SHAPES)
@pytest.mark.parametrize("rms", [False, True])
def test_projection_bf16_edges(M, N, K, rms):
    """Aligned operands (direct loads) and, up to 64 rows, operands whose base
    is 2 bytes off a 16-byte boundary (the gather kernel) against fp64."""
    import torch
    from paper_2609_12075_amd import vla
    log(f"[wave bf16] M={M} N={N} K={K} rms={rms} plan={_plan_of(M, N, K, rms=rms)}")
    g = torch.Generator().manual_seed(M + N + K)
    A = torch.randn(M, K, generator=g).bfloat16()
    W = (torch.randn(N, K, generator=g) * 0.05).bfloat16()
    bias = torch.randn(N, generator=g)
    x = A.double()
    scale = 1 / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6) if rms else 1.0
    ref = (scale * (x @ W.double().t()) + bias.double()).numpy()

    def off(t, by):          # the same matrix `by` bf16 elements past an aligned address
        flat = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
        flat[by:by + t.numel()] = t.cuda().flatten()
        return flat[by:by + t.numel()].view(t.shape)

    for by in ((0, 1) if M <= 64 else (0,)):
        a, w = off(A, by), off(W, by)
        out = vla.debug_gemm_rms(a, w, bias=bias.cuda(), eps=1e-6) if rms else vla.debug_gemm(a, w, bias=bias.cuda())
        torch.cuda.synchronize()
        # fp32 sums of K exact bf16 products: a few times sqrt(K) roundings of a term
        np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=1e-4, atol=1e-5 * (np.sqrt(K) * 0.05 + 1))


# patch extraction by vectors of 4, 2 and 1 pixels, with (112 of 108) and
# without columns to fill; end to end against the oracle
@pytest.mark.parametrize("patch,hw,bf16", [(8, 24, False), (6, 12, True), (5, 15, False), (5, 15, True)])
def test_patch_sizes(patch, hw, bf16):
    from paper_2609_12075_amd import synth
    from tests.test_gpu_parity import check_parity
    cfg = synth.CONFIGS["tiny"].with_(name=f"tiny-p{patch}-{bf16}", patch=patch, img_hw=hw, n_img=2, action_dim=8,
                                      dtype=synth.DTYPE_BF16 if bf16 else synth.DTYPE_F32)
    check_parity(cfg, 3)


# bf16 attention whose waves split the keys: every head-dim padding, output
# dims whole and shared by two and four blocks, one key, whole and ragged last
# tiles in both segments, more tiles than waves, rows that end inside a tile,
# and on both sides of its limits (1024 keys; 256, 512 or 2048 blocks); many
# row tiles at head dims 72 and 80, whose last subtiles are skipped
@pytest.mark.parametrize("B,Hq,Hkv,Lq,hd,len0,len1", [
    (1, 1, 1, 1, 8, 1, 0), (2, 32, 32, 17, 32, 296, 0), (3, 6, 2, 9, 24, 33, 5), (33, 32, 32, 17, 32, 40, 0),
    (1, 15, 5, 50, 64, 240, 50), (2, 6, 2, 11, 40, 31, 1), (1, 5, 1, 50, 64, 1024, 0), (1, 5, 1, 50, 64, 1024, 1),
    (1, 16, 16, 256, 72, 256, 0), (1, 16, 16, 257, 72, 64, 0), (4, 16, 16, 257, 72, 70, 3), (17, 16, 16, 64, 80, 65, 0), (1, 4, 2, 7, 128, 999, 17),
    (1, 8, 1, 50, 256, 816, 50), (1, 2, 1, 3, 200, 17, 0), (2, 2, 2, 33, 136, 15, 3), (4, 8, 1, 50, 256, 97, 20),
    (8, 8, 1, 50, 256, 64, 9), (1, 8, 1, 296, 256, 296, 0), (3, 8, 1, 400, 256, 50, 0)])
def test_attention_bf16_edges(B, Hq, Hkv, Lq, hd, len0, len1):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[attn bf16] B={B} Hq={Hq} Hkv={Hkv} Lq={Lq} hd={hd} len0={len0} len1={len1}")
    g = torch.Generator().manual_seed(hd + len0 + B)
    rnd = lambda *s: torch.randn(*s, generator=g).bfloat16()
    q, k0, v0 = rnd(B, Hq, Lq, hd), rnd(B, Hkv, len0, hd), rnd(B, Hkv, len0, hd)
    k1, v1 = (rnd(B, Hkv, len1, hd), rnd(B, Hkv, len1, hd)) if len1 else (None, None)
    c = lambda t: None if t is None else t.cuda()
    got = vla.debug_attention(c(q), c(k0), c(v0), c(k1), c(v1)).cpu().double()
    k, v = (x if y is None else torch.cat([x, y], 2) for x, y in ((k0, k1), (v0, v1)))
    k, v = (x.double().repeat_interleave(Hq // Hkv, 1) for x in (k, v))
    p = torch.softmax(q.double() @ k.transpose(2, 3) / hd ** 0.5, -1)
    rows = lambda o: o.transpose(1, 2).reshape(B, Lq, Hq * hd)
    ref, mag = rows(p @ v), rows(p @ v.abs())
    # bf16 (8 significant bits) rounds each probability and the output by at
    # most 2^-8 of itself (half a unit of 2^-7); fp32 scores, exponentials and
    # sums add a few 2^-22 of the summed magnitudes
    bound = 2.0 ** -8 * 1.01 * (mag + ref.abs())
    assert ((got - ref).abs() <= bound).all(), float(((got - ref).abs() / bound).max())


# fp32 models whose action expert normalises its input rows inside the
# projections: widths below, at and past a K chunk of the eight waves, batches
# whose rows end inside a tile
@pytest.mark.parametrize("d,horizon,batch", [(64, 3, 1), (96, 8, 3), (320, 17, 2)])
def test_f32_folded_norms(d, horizon, batch):
    from paper_2609_12075_amd import synth
    from tests.test_gpu_parity import check_parity
    check_parity(synth.CONFIGS["tiny"].with_(name=f"tiny-d{d}-h{horizon}", act_d=d, horizon=horizon), batch)
