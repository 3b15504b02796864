"""The projection planner (host logic, no GPU): plans of the model's
projection shapes that were chosen by measurement, and invariants every plan
must satisfy (K covered by non-empty ranges, the split workspace respected,
each kernel kind within the shapes it serves)."""
import itertools

import pytest

from paper_2609_12075_amd import vla

STORE, RESID, GEGLU, QKV, EULER = 0, 1, 2, 3, 4
SPLIT_FLOATS = 16 << 20          # the split-K workspace of a model's stage (floats)


def plan(M, N, K, mode=STORE, **kw):
    return vla.gemm_plan(M, N, K, mode, **kw)


def test_few_rows_long_k_take_k_ranges_on_staged_tiles():
    """The GR00T-like LLM MLP down at batch 1 (296 rows, K = 16384): LDS-staged
    tiles with K ranges, not the register tiles with one K loop per tile."""
    p = plan(296, 2048, 16384, RESID, norm_follows=True)
    assert p["kind"] == 1 and p["splits"] >= 2, p


@pytest.mark.parametrize("M", [256, 512, 768])
def test_vit_mlp_down_two_group_tiles_with_k_ranges(M):
    """The ViT MLP down (K = 4304) at 256-768 rows: two-group K-steps of 128
    with two K ranges."""
    p = plan(M, 1152, 4304, RESID, norm_follows=True)
    assert (p["kind"], p["splits"], p["bk"], p["kg"]) == (4, 2, 128, 2), p


def test_k_past_4096_needs_k_ranges_on_two_group_tiles():
    """At 1024 rows the same product would take one 34-step range on the
    two-group tiles (measured slower): it stays on the staged tiles."""
    p = plan(1024, 1152, 4304, RESID, norm_follows=True)
    assert p["kind"] != 4, p


def test_small_m_kernel_for_one_action_chunk():
    p = plan(50, 8192, 1024, GEGLU, out_bf16=True, rms=True)
    assert p["kind"] == 2 and p["splits"] == 1, p


def test_large_tiles_for_the_pi0_gate_up_at_batch_8():
    p = plan(6528, 32768, 2048, GEGLU, out_bf16=True)
    assert (p["kind"], p["tile_n"], p["tile_m"], p["splits"]) == (3, 256, 256, 1), p


@pytest.mark.parametrize("M,N,K", [(800, 3840, 720), (50, 2560, 1024), (400, 2560, 1024), (3000, 5120, 960)])
def test_folded_norm_never_splits_k(M, N, K):
    p = plan(M, N, K, GEGLU if N % 2 == 0 else STORE, out_bf16=True, rms=True)
    assert p["splits"] == 1 and p["kind"] in (1, 2, 4), p


MS = [1, 17, 50, 64, 65, 100, 256, 296, 512, 768, 1024, 1632, 4096, 6528]
NS = [16, 720, 1152, 2048, 3840, 8192, 32768]
KS = [64, 720, 1152, 2048, 4304, 8192, 16384]


@pytest.mark.parametrize("mode", [STORE, RESID])
def test_plan_invariants(mode):
    for M, N, K in itertools.product(MS, NS, KS):
        p = plan(M, N, K, mode, norm_follows=mode == RESID)
        s, ks, kind = p["splits"], p["ksplit"], p["kind"]
        where = (M, N, K, mode, p)
        assert kind in (0, 1, 2, 3, 4), where
        assert 1 <= s <= 16 and ks > 0, where
        assert s * ks >= K and (s - 1) * ks < K, where            # K covered, no empty range
        if s > 1:
            assert ks % p["bk"] == 0, where                        # ranges end on K-step boundaries
            assert s * M * ((N + 3) & ~3) <= SPLIT_FLOATS, where   # partials fit the workspace
        if kind == 2:
            assert M <= 64 and s == 1, where
        if kind == 3:
            assert s == 1 and p["tile_n"] == 256 and p["tile_m"] in (224, 256) and M >= 256 and K >= 512, where
        if kind == 4:
            assert M <= 1024 and p["bk"] == 128 and p["kg"] == 2, where
            assert K <= 4096 or s > 1, where


def test_bad_arguments_are_rejected():
    assert vla.lib().vla_debug_gemm_plan(0, 16, 64, 0, 0, 0, 0, (vla.ctypes.c_int * 8)()) == vla.VLA_EINVAL
    assert vla.lib().vla_debug_gemm_plan(16, 15, 64, GEGLU, 1, 0, 0, (vla.ctypes.c_int * 8)()) == vla.VLA_EINVAL
    assert vla.lib().vla_debug_gemm_plan(16, 16, 60, 0, 0, 0, 0, (vla.ctypes.c_int * 8)()) == vla.VLA_EINVAL
    assert vla.lib().vla_debug_gemm_plan(16, 16, 64, RESID, 0, 1, 0, (vla.ctypes.c_int * 8)()) == vla.VLA_EINVAL


@pytest.mark.parametrize("shape,kernel", [
    # (B, Hq, Hkv, Lq, hd, len0, len1): head dims 33-128 to one block of 16
    # rows a CU and 1024 keys
    ((4, 15, 5, 50, 64, 240, 50), "wave"), ((8, 15, 5, 50, 64, 240, 50), "direct"), ((1, 16, 16, 256, 72, 256, 0), "wave"),
    ((1, 16, 16, 257, 72, 256, 0), "direct"), ((1, 5, 1, 50, 64, 974, 50), "wave"), ((1, 5, 1, 50, 64, 975, 50), "direct"),
    # over 128 likewise; at 256 to two blocks a CU where the keys are enough
    # and the blocks of 64 rows filled
    ((8, 8, 1, 50, 256, 816, 50), "wave"), ((16, 8, 1, 50, 256, 816, 50), "wave"), ((16, 8, 1, 50, 256, 100, 50), "direct"),
    ((20, 8, 1, 50, 256, 270, 50), "direct"), ((20, 8, 1, 50, 256, 271, 50), "wave"), ((21, 8, 1, 50, 256, 816, 50), "direct"),
    ((16, 16, 16, 17, 256, 800, 0), "direct"), ((8, 8, 1, 50, 200, 816, 50), "wave"), ((16, 8, 1, 50, 200, 816, 50), "direct"),
    # to 32 by blocks and keys: blocks of 16 rows that are whole, nearly empty
    # second ones, and four to a block of 64
    ((8, 32, 32, 16, 32, 64, 0), "wave"), ((64, 32, 32, 16, 32, 300, 0), "wave"), ((65, 32, 32, 16, 32, 300, 0), "direct"),
    ((3, 32, 32, 17, 32, 296, 0), "wave"), ((32, 32, 32, 17, 32, 296, 0), "wave"), ((32, 32, 32, 17, 32, 17, 0), "direct"),
    ((8, 16, 16, 128, 32, 100, 0), "direct"), ((8, 16, 16, 128, 32, 600, 0), "wave"), ((16, 16, 16, 128, 32, 100, 0), "direct"),
    ((16, 16, 16, 128, 8, 1000, 0), "direct"), ((4, 16, 16, 128, 32, 200, 0), "wave"),
])
def test_attention_of_few_row_tiles(shape, kernel):
    """The measured sides of the rule that splits an attention's keys over a
    block's waves: with many blocks or few keys the blocks of 64 rows are
    faster (up to 1.9 times)."""
    assert vla.attention_plan(*shape)["kernel"] == kernel, vla.attention_plan(*shape)


def test_attention_plan_invariants():
    for B, Hkv, G, Lq, hd, keys in itertools.product([1, 3, 16, 40], [1, 5, 16], [1, 3, 8], [1, 17, 50, 300],
                                                     [8, 32, 40, 64, 72, 80, 128, 200, 256], [1, 33, 300, 1024, 1025, 3000]):
        p = vla.attention_plan(B, Hkv * G, Hkv, Lq, hd, keys)
        where = (B, Hkv, G, Lq, hd, keys, p)
        assert p["hdp"] >= hd and p["kernel"] in ("wave", "direct"), where
        if p["kernel"] == "wave":
            assert p["splits"] == 1 and p["hdp"] // p["dims"] in (1, 2, 4), where
            # the reciprocal divisions hold for block and row indices to 2^16 each
            assert -(-G * Lq // 16) * Hkv * B <= 2048, where
        else:
            assert p["dims"] >= hd and p["groups"] in (1, 2) and 1 <= p["splits"] <= 16, where
            if p["splits"] > 1:                                     # keys covered, no empty range
                assert p["splits"] * p["kchunk"] >= keys > (p["splits"] - 1) * p["kchunk"], where
        f = vla.attention_plan(B, Hkv * G, Hkv, Lq, hd, keys, bf16=False)
        assert f["kernel"] == "f32" and f["hdp"] >= hd, where
    bad = (vla.ctypes.c_int * 6)()
    assert vla.lib().vla_debug_attention_plan(1, 3, 2, 4, 64, 1, 8, 0, bad) == vla.VLA_EINVAL
    assert vla.lib().vla_debug_attention_plan(1, 2, 2, 4, 60, 1, 8, 0, bad) == vla.VLA_EINVAL
    assert vla.lib().vla_debug_attention_plan(1, 2, 2, 4, 64, 1, 0, 8, bad) == vla.VLA_EINVAL


@pytest.mark.parametrize("mode,rms", [(STORE, False), (RESID, False), (GEGLU, True), (QKV, True), (EULER, True)])
def test_plans_name_kernels_of_the_library(mode, rms):
    """The kernel that a plan names (the profiler's name of it) is one that
    the library holds; waves that split K are reported under two kinds."""
    with open(vla._LIB_PATH, "rb") as f:
        names = f.read()
    for M, N, K in itertools.product([1, 50, 100, 300, 800, 3000, 7000], [16, 720, 1152, 2048, 8192], [64, 720, 2048, 4304, 8192]):
        out_bf16 = mode in (GEGLU, QKV)
        p = dict(plan(M, N, K, mode, out_bf16=out_bf16, rms=rms), mode=mode, rms=int(rms), f32=0)
        assert vla.Model.kernel_symbol(p).encode() in names, (M, N, K, p, vla.Model.kernel_symbol(p))
        if p["kind"] == 0 and p["kg"] > 1:
            assert M > 64 and p["splits"] == 1 and p["ksplit"] >= K and p["stages"] in (1, 2), (M, N, K, p)
