"""Kernels that the dispatch reaches at sizes that no other kernel test has:
each shape states the plan it is there for, so that a change of the dispatch
cannot leave the kernel without a test unnoticed."""
import numpy as np
import pytest

from oracle import vla as O
from tests.gpu_util import log

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(31)


def _bf16(a):
    return O.bf16_round(np.asarray(a, np.float32))


def _plan(M, N, K, mode=0, **kw):
    from paper_2609_12075_amd import vla
    p = vla.gemm_plan(M, N, K, mode, **kw)
    return p["kind"], p["tile_n"], p["tile_m"], p["stages"], p["kg"], p["splits"]


# residual projections: 64 x 64 tiles with two wave groups and one K range
# (the update from registers), whole and ragged, also three-stage; 128 x 128
# tiles whose stages are requested early (rows that end inside a line over more
# than 512 blocks) and late
@pytest.mark.parametrize("M,N,K,plan", [
    (816, 2048, 2048, (4, 64, 64, 2, 2, 1)), (811, 2044, 2040, (4, 64, 64, 2, 2, 1)), (1024, 1152, 1152, (4, 64, 64, 2, 2, 1)),
    (9000, 1160, 1080, (1, 128, 128, 2, 1, 1)), (1500, 5000, 1000, (1, 128, 128, 2, 1, 1)),
])
def test_residual_routes(M, N, K, plan):
    """x += gate * (A W^T + bias) with the bf16 copy, against fp64 on sampled
    rows; the copy is x rounded, and rows that are only 4-byte aligned (the
    per-element epilogue) give the same bits."""
    import torch
    from paper_2609_12075_amd import vla
    log(f"[resid route] M={M} N={N} K={K}")
    assert _plan(M, N, K, 1) == plan
    A, W = _bf16(RNG.standard_normal((M, K))), _bf16(RNG.standard_normal((N, K)) * 0.05)
    x0 = RNG.standard_normal((M, N)).astype(np.float32)
    bias, gate = (RNG.standard_normal(N) * 0.1).astype(np.float32), (1 + 0.1 * RNG.standard_normal(N)).astype(np.float32)
    At, Wt = (torch.from_numpy(t).to(torch.bfloat16).cuda() for t in (A, W))
    bt, gt, x = (torch.from_numpy(t).cuda() for t in (bias, gate, x0.copy()))
    xb = vla.debug_resid_copy(At, Wt, x, bias=bt, gate=gt)
    xw = torch.zeros(M, N + 5, device="cuda")
    xw[:, 1:1 + N] = torch.from_numpy(x0).cuda()
    vla.debug_resid_copy(At, Wt, xw[:, 1:1 + N], bias=bt, gate=gt)
    torch.cuda.synchronize()
    assert torch.equal(xb, x.to(torch.bfloat16)) and torch.equal(x, xw[:, 1:1 + N])
    rows = np.unique(np.concatenate([np.arange(20), RNG.integers(0, M, 60), np.arange(M - 20, M)]))
    ref = x0[rows].astype(np.float64) + (A[rows].astype(np.float64) @ W.astype(np.float64).T + bias) * gate
    np.testing.assert_allclose(x.cpu().numpy()[rows], ref, rtol=1e-4, atol=1e-4)


# stores: register-pipelined 64 x 32 tiles without and with K ranges, 64 x 64
# tiles with one wave group, with two and three stages, with two and K ranges;
# with the RMSNorm of the rows folded in: few rows of long K, three stages, 64 x
# 64 and 128 x 64 tiles with one group
@pytest.mark.parametrize("M,N,K,rms,plan", [
    (1100, 720, 64, False, (0, 64, 32, 2, 1, 1)), (40, 1000, 8192, False, (0, 64, 32, 2, 1, "split")),
    (5, 300, 8200, False, (0, 64, 32, 2, 1, "split")), (1000, 2200, 504, False, (1, 64, 64, 2, 1, 1)),
    (200, 3000, 200, False, (4, 64, 64, 3, 2, 1)), (1, 200, 4304, False, (4, 64, 64, 3, 2, "split")),
    (1010, 1000, 4304, False, (4, 64, 64, 2, 2, "split")), (1000, 2200, 504, True, (1, 64, 64, 2, 1, 1)),
    (5, 33, 4304, True, (1, 64, 64, 2, 1, 1)), (200, 3000, 200, True, (4, 64, 64, 3, 2, 1)),
    (65, 8192, 4304, True, (1, 128, 64, 2, 1, 1)),
])
def test_store_routes(M, N, K, rms, plan):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[store route] M={M} N={N} K={K} rms={rms}")
    got = _plan(M, N, K, rms=rms)
    assert got[:5] + ("split" if got[5] > 1 else 1,) == plan, got
    A, W = _bf16(RNG.standard_normal((M, K))), _bf16(RNG.standard_normal((N, K)) * 0.05)
    bias = RNG.standard_normal(N).astype(np.float32)
    t = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    b = torch.from_numpy(bias).cuda()
    out = vla.debug_gemm_rms(t(A), t(W), bias=b, eps=1e-6) if rms else vla.debug_gemm(t(A), t(W), bias=b)
    torch.cuda.synchronize()
    A64 = A.astype(np.float64)
    r = 1 / np.sqrt((A64 * A64).mean(1, keepdims=True) + 1e-6) if rms else 1.0
    ref = r * (A64 @ W.astype(np.float64).T) + bias
    np.testing.assert_allclose(out.cpu().numpy(), ref, rtol=1e-4, atol=1e-5 * (np.sqrt(K) * 0.05 + 1))


# the reduce of a split residual projection with the row norm that follows, at
# each row width it is compiled for (to 256, 512, 1024, 2048), ragged widths,
# after 64 x 32, 64 x 64, 128 x 64 and 128 x 128 partial tiles
@pytest.mark.parametrize("M,N,K,kind", [
    (5, 64, 8192, 0), (100, 256, 8192, 1), (40, 300, 4304, 2), (130, 512, 8192, 0), (100, 720, 8192, 1),
    (200, 1024, 4304, 2), (800, 1000, 8192, 0), (5, 1152, 8192, 1), (300, 2048, 4304, 0)])
def test_split_residual_with_norm(M, N, K, kind):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[split norm] M={M} N={N} K={K} kind={kind}")
    assert vla.gemm_plan(M, N, K, 1, norm_follows=True)["splits"] > 1
    A, W = _bf16(RNG.standard_normal((M, K))), _bf16(RNG.standard_normal((N, K)) * 0.02)
    x0 = RNG.standard_normal((M, N)).astype(np.float32)
    bias = (RNG.standard_normal(N) * 0.1).astype(np.float32)
    g = (1 + 0.1 * RNG.standard_normal(N)).astype(np.float32) if kind != 1 else None
    b = (0.1 * RNG.standard_normal(N)).astype(np.float32) if kind == 2 else None
    x_ref = x0.astype(np.float64) + A.astype(np.float64) @ W.astype(np.float64).T + bias
    if kind == 0:
        z_ref = O.rmsnorm(x_ref, g.astype(np.float64), 1e-6)
    else:
        z_ref = O.layernorm(x_ref, None, None, 1e-6)
        z_ref = z_ref * (1 + g) + b if kind == 2 else z_ref
    t = lambda a: None if a is None else torch.from_numpy(a).cuda()
    x = t(x0.copy())
    z = vla.debug_resid_norm(t(A).to(torch.bfloat16), t(W).to(torch.bfloat16), x, kind, g=t(g), b=t(b), bias=t(bias))
    torch.cuda.synchronize()
    np.testing.assert_allclose(x.cpu().numpy(), x_ref, rtol=1e-4, atol=1e-4)
    # z: bf16 of fp32 statistics and an fp32 row
    np.testing.assert_allclose(z.float().cpu().numpy(), z_ref, rtol=2.0 ** -8 * 1.01, atol=1e-4)


# attention on blocks of 64 rows: head dims to 32 with a ring of four tiles and
# more tiles than slots; key ranges over blocks and their merge at each lane
# count; two key groups with ragged segments; the narrow subtiles of 72 and 80;
# and the splitting waves at head dim 256 with two blocks a CU
@pytest.mark.parametrize("shape,plan", [
    ((9, 32, 32, 128, 32, 305, 0), ("direct", 32, 32, 1, 1)), ((5, 32, 32, 128, 24, 290, 9), ("direct", 32, 32, 1, 1)),
    ((1, 2, 2, 40, 32, 1500, 3), ("direct", 32, 32, 1, "split")), ((1, 5, 1, 50, 64, 1100, 7), ("direct", 64, 64, 2, "split")),
    ((1, 4, 2, 40, 128, 1101, 30), ("direct", 128, 128, 2, "split")), ((1, 2, 2, 33, 72, 1030, 0), ("direct", 128, 128, 2, "split")),
    ((1, 8, 1, 50, 256, 1201, 50), ("direct", 256, 256, 2, "split")), ((2, 4, 2, 21, 200, 1025, 2), ("direct", 256, 256, 2, "split")),
    ((24, 8, 1, 100, 256, 150, 7), ("direct", 256, 256, 2, 1)), ((6, 16, 16, 257, 80, 140, 3), ("direct", 128, 80, 1, 1)),
    ((16, 15, 5, 240, 64, 257, 0), ("direct", 64, 64, 1, 1)), ((40, 4, 1, 130, 128, 129, 0), ("direct", 128, 128, 1, 1)),
    ((16, 8, 1, 50, 256, 300, 50), ("wave", 256, 256, 1, 1)), ((2, 8, 1, 50, 256, 70, 9), ("wave", 256, 64, 1, 1)),
    ((5, 8, 1, 50, 256, 70, 9), ("wave", 256, 128, 1, 1)), ((40, 32, 32, 16, 32, 200, 0), ("wave", 32, 32, 1, 1)),
])
def test_attention_routes(shape, plan):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[attn route] {shape} {plan}")
    B, Hq, Hkv, Lq, hd, len0, len1 = shape
    p = vla.attention_plan(*shape)
    assert (p["kernel"], p["hdp"], p["dims"], p["groups"], "split" if p["splits"] > 1 else 1) == plan, p
    g = torch.Generator().manual_seed(hd + len0 + B)
    rnd = lambda *s: torch.randn(*s, generator=g).bfloat16()
    q, k0, v0 = rnd(B, Hq, Lq, hd), rnd(B, Hkv, len0, hd), rnd(B, Hkv, len0, hd)
    k1, v1 = (rnd(B, Hkv, len1, hd), rnd(B, Hkv, len1, hd)) if len1 else (None, None)
    c = lambda t: None if t is None else t.cuda()
    got = vla.debug_attention(c(q), c(k0), c(v0), c(k1), c(v1)).cpu().double()
    k, v = (x if y is None else torch.cat([x, y], 2) for x, y in ((k0, k1), (v0, v1)))
    k, v = (x.double().repeat_interleave(Hq // Hkv, 1) for x in (k, v))
    pr = torch.softmax(q.double() @ k.transpose(2, 3) / hd ** 0.5, -1)
    rows = lambda o: o.transpose(1, 2).reshape(B, Lq, Hq * hd)
    ref, mag = rows(pr @ v), rows(pr @ v.abs())
    # bf16 (8 significant bits) rounds each probability and the output by at
    # most 2^-8 of itself (half a unit of 2^-7); fp32 scores, exponentials and
    # sums add a few 2^-22 of the summed magnitudes
    bound = 2.0 ** -8 * 1.01 * (mag + ref.abs())
    assert ((got - ref).abs() <= bound).all(), float(((got - ref).abs() / bound).max())


# fp32 products whose rows the direct loads cannot take: 16 x 16 and 32 x 32
# tiles whose waves split K, 64 x 64 ones (long K), and tiles of one wave alone,
# 32 x 32 and 64 x 32, each ragged, with K below, at and past a piece, and rows
# of 4-byte alignment only
@pytest.mark.parametrize("M,N,K", [(33, 50, 9), (270, 250, 70), (700, 300, 1021), (600, 610, 7), (530, 500, 33),
                                   (610, 600, 130), (2000, 900, 1), (2010, 899, 30), (1500, 1300, 61)])
def test_f32_rows_of_any_length(M, N, K):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[gather f32] M={M} N={N} K={K}")
    A, W = RNG.standard_normal((M, K)).astype(np.float32), RNG.standard_normal((N, K)).astype(np.float32)
    bias = RNG.standard_normal(N).astype(np.float32)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + bias

    def off(a):              # the same matrix one float past an aligned address
        flat = torch.zeros(a.size + 4, device="cuda")
        flat[1:1 + a.size] = torch.from_numpy(a).cuda().flatten()
        return flat[1:1 + a.size].view(a.shape)

    out = vla.debug_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda(), bias=torch.from_numpy(bias).cuda())
    out1 = vla.debug_gemm(off(A), off(W), bias=torch.from_numpy(bias).cuda())
    torch.cuda.synchronize()
    # each of the K products and sums rounds once: |error| <= K 2^-24 sum |a w|,
    # in practice its square root; a few of those
    bound = 4 * np.sqrt(K) * 2.0 ** -24 * (np.abs(A) @ np.abs(W).T + np.abs(bias)) + 1e-7
    assert (np.abs(out.cpu().numpy() - ref) <= bound).all()
    if K % 4:
        assert torch.equal(out, out1)


# the same products as residual updates: fp32 models with MLP widths that are
# no multiple of four (64 x 64, 32 x 32 and 64 x 32 tiles in the LLM, 16 x 16 in
# the action expert)
@pytest.mark.parametrize("llm_d,llm_mlp,act_mlp", [(512, 1030, 129), (512, 510, 514), (1024, 130, 129)])
def test_f32_models_with_odd_mlp_widths(llm_d, llm_mlp, act_mlp):
    from paper_2609_12075_amd import synth
    from tests.test_gpu_parity import check_parity
    check_parity(synth.CONFIGS["tiny"].with_(name=f"tiny-{llm_d}-{llm_mlp}", llm_d=llm_d, llm_mlp=llm_mlp, act_mlp=act_mlp,
                                             n_text=128, max_batch=8), 8)


# short K and many tiles: 32 x 32 and 64 x 32 tiles of one wave for aligned rows
# too, as stores and (width of the action expert, batch) with the folded norm
@pytest.mark.parametrize("M,N,K", [(830, 840, 4), (1000, 700, 96), (1500, 1300, 20), (2100, 900, 128)])
def test_f32_short_k_many_tiles(M, N, K):
    import torch
    from paper_2609_12075_amd import vla
    log(f"[alone f32] M={M} N={N} K={K}")
    A, W = RNG.standard_normal((M, K)).astype(np.float32), RNG.standard_normal((N, K)).astype(np.float32)
    out = vla.debug_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda())
    bound = 4 * np.sqrt(K) * 2.0 ** -24 * (np.abs(A) @ np.abs(W).T) + 1e-7
    assert (np.abs(out.cpu().numpy() - A.astype(np.float64) @ W.astype(np.float64).T) <= bound).all()


@pytest.mark.parametrize("act_d,batch", [(64, 128), (96, 130), (128, 210)])
def test_f32_folded_norms_of_short_rows(act_d, batch):
    from oracle import vla as OV
    from paper_2609_12075_amd import synth
    from tests.gpu_util import check_chunk, oracle_params, run
    cfg = synth.CONFIGS["tiny"].with_(name=f"tiny-a{act_d}-b{batch}", act_d=act_d, max_batch=batch)
    inp = synth.make_inputs(cfg, batch)
    act, _ = run(cfg, inp)
    rows = [0, batch // 2, batch - 1]
    ref, _ = OV.run(cfg, oracle_params(cfg), inp, rows=rows)
    check_chunk(act[rows], ref, inp["noise"][rows], 1e-4, cfg.name)


@pytest.mark.parametrize("kw,stages", [({}, 2), ({"act_mlp": 129, "llm_mlp": 514}, 0), ({"max_batch": 64}, 2)])
def test_f32_plans_name_what_is_launched(kw, stages):
    """A replay of an fp32 model's projections reports the tile and waves of
    the kernel that it launches."""
    from paper_2609_12075_amd import synth, vla
    cfg = synth.CONFIGS["tiny"].with_(name="tiny-plans", **kw)
    m = vla.Model(cfg, synth.make_weights(cfg))
    with open(vla._LIB_PATH, "rb") as f:
        names = f.read()
    for which in range(4):
        flops, p = m.replay_gemm(which, cfg.max_batch, 0)
        where = (which, p, vla.Model.kernel_symbol(p))
        assert p["f32"] == 1 and p["kind"] == 2 and p["splits"] == 1, where
        assert vla.Model.kernel_symbol(p).encode() in names, where
        assert p["tile_n"] in (16, 32, 64) and p["tile_m"] in (16, 32, 64) and p["kg"] in (1, 4, 8), where
    assert m.replay_gemm(3, cfg.max_batch, 0)[1]["stages"] == stages          # the down projection: K = act_mlp
    m.close()


# patch extraction of very many images: more rows of blocks than a launch
# holds, and (17 GB of pixels, one a thread) more threads than fit one dimension
@pytest.mark.parametrize("batch,hw,patch", [(4000, 8, 8), (4000, 245, 49)])
def test_very_many_images(batch, hw, patch):
    import torch
    from paper_2609_12075_amd import synth, vla
    cfg = synth.CONFIGS["tiny"].with_(name=f"tiny-many-{hw}", n_img=6, img_hw=hw, patch=patch, n_text=2, llm_d=64, n_q=1, n_kv=1,
                                      llm_mlp=64, act_d=64, act_mlp=64, max_batch=batch)
    if torch.cuda.mem_get_info()[0] < 8 * batch * 6 * 3 * hw * hw + (8 << 30):
        pytest.skip("the card has not enough free memory for the pixels and their patches")
    log(f"[images] {6 * batch} of {hw} x {hw}, patches of {patch}")
    g = torch.Generator(device="cuda").manual_seed(7)
    pix = torch.rand(batch, 6, 3, hw, hw, generator=g, device="cuda")
    text = torch.randint(0, cfg.vocab, (batch, 2), generator=g, device="cuda", dtype=torch.int32)
    w = synth.make_weights(cfg)
    m = vla.Model(cfg, w)
    kv = m.alloc_kv(batch)
    m.prefill(batch, pix, text, kv)
    torch.cuda.synchronize()
    got = kv.view(torch.float32).view(cfg.llm_layers, 2, batch, 1, cfg.prefix_len, cfg.head_dim)
    P = O.params(cfg, w)
    for b in (0, batch // 2, batch - 1):
        ref = O.prefill_row(cfg, P, pix[b].cpu().numpy(), text[b].cpu().numpy(), None)
        for l in range(cfg.llm_layers):
            for i, what in enumerate("kv"):
                r, x = ref[what][l], got[l, i, b].cpu().numpy()
                assert np.linalg.norm(x - r) <= 1e-4 * np.linalg.norm(r), (b, l, what)
    m.close()


@pytest.mark.parametrize("patch,bf16", [(8, False), (8, True), (6, True), (5, False)])
def test_pixels_at_any_float(patch, bf16):
    """Pixels one float past an aligned address give the same bits."""
    import torch
    from paper_2609_12075_amd import synth, vla
    cfg = synth.CONFIGS["tiny"].with_(name=f"tiny-px{patch}-{bf16}", patch=patch, img_hw=3 * patch, action_dim=8,
                                      dtype=synth.DTYPE_BF16 if bf16 else synth.DTYPE_F32)
    m = vla.Model(cfg, synth.make_weights(cfg))
    inp = synth.make_inputs(cfg, 3)
    text, pix = torch.from_numpy(inp["text_ids"]).cuda(), torch.from_numpy(inp["pixels"]).cuda()
    flat = torch.zeros(pix.numel() + 4, device="cuda")
    flat[1:1 + pix.numel()] = pix.flatten()
    kvs = []
    for p in (pix, flat[1:1 + pix.numel()].view(pix.shape)):
        kvs.append(m.alloc_kv(3))
        m.prefill(3, p, text, kvs[-1])
    torch.cuda.synchronize()
    assert torch.equal(kvs[0], kvs[1])
    m.close()
