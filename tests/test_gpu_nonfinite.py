"""Infinities and NaN in the inputs of the attention kernels: they reach the
outputs that depend on them, as what they are, and leave every other output's
bits as they were."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu


def _inputs(B, Hq, Hkv, Lq, hd, len0, len1, dtype):
    import torch
    g = torch.Generator().manual_seed(hd + len0 + Lq)
    rnd = lambda *s: torch.randn(*s, generator=g).to(dtype)
    t = {"q": rnd(B, Hq, Lq, hd), "k0": rnd(B, Hkv, len0, hd), "v0": rnd(B, Hkv, len0, hd)}
    if len1:
        t.update(k1=rnd(B, Hkv, len1, hd), v1=rnd(B, Hkv, len1, hd))
    return t


def _run(t, shape):
    from paper_2609_12075_amd import vla
    B, Hq, Hkv, Lq, hd = shape[:5]
    d = {n: x.cuda() for n, x in t.items()}
    o = vla.debug_attention(d["q"], d["k0"], d["v0"], d.get("k1"), d.get("v1")).cpu()
    return o.view(B, Lq, Hq, hd).transpose(1, 2)          # [B][Hq][Lq][hd]


# fp32; bf16: waves that split the keys (one block a row tile, and at head dim
# 256 four blocks that share it), direct-load tiles (one key group, two, two
# with key ranges over blocks and their merge)
SHAPES = [
    ("f32", (2, 4, 2, 9, 64, 35, 2)), ("f32", (1, 2, 1, 19, 136, 16, 1)), ("f32", (2, 2, 2, 5, 256, 131, 0)),
    ("bf16", (2, 6, 2, 11, 64, 45, 4)), ("bf16", (1, 4, 1, 21, 32, 300, 0)), ("bf16", (2, 2, 1, 9, 256, 50, 3)),
    ("bf16", (8, 15, 5, 240, 64, 150, 7)), ("bf16", (4, 8, 2, 300, 128, 70, 0)), ("bf16", (40, 8, 1, 100, 256, 100, 9)),
    ("bf16", (1, 5, 1, 50, 64, 1024, 5)), ("bf16", (1, 4, 1, 50, 256, 1101, 20)),
]


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_nonfinite_query_and_value(dtype, shape):
    import torch
    log(f"[attn nonfinite] {dtype} {shape}")
    B, Hq, Hkv, Lq, hd, len0, len1 = shape
    G = Hq // Hkv
    clean = _inputs(*shape, torch.float32 if dtype == "f32" else torch.bfloat16)
    want = _run(clean, shape)
    assert torch.isfinite(want.float()).all()

    # a NaN in one query: its row alone is NaN
    t = {n: x.clone() for n, x in clean.items()}
    t["q"][B - 1, Hq - 1, Lq // 2, hd - 1] = float("nan")
    got = _run(t, shape)
    assert torch.isnan(got[B - 1, Hq - 1, Lq // 2].float()).all()
    got[B - 1, Hq - 1, Lq // 2] = want[B - 1, Hq - 1, Lq // 2]
    assert torch.equal(got, want)

    # an infinity in the last key's values (the first request and KV head):
    # one output dim of that head's queries is infinite, with its sign. Keys
    # past the end, which fill the last tile, must not turn it into a NaN.
    t = {n: x.clone() for n, x in clean.items()}
    t["v1" if len1 else "v0"][0, 0, -1, 3] = -float("inf")
    got = _run(t, shape)
    assert (got[0, :G, :, 3].float() == -float("inf")).all(), got[0, :G, :, 3]
    got[0, :G, :, 3] = want[0, :G, :, 3]
    assert torch.equal(got, want)

    # a NaN in a key: the rows of that request and KV head are NaN
    t = {n: x.clone() for n, x in clean.items()}
    t["k0"][0, Hkv - 1, len0 // 2, 0] = float("nan")
    got = _run(t, shape)
    assert torch.isnan(got[0, (Hkv - 1) * G:].float()).all()
    got[0, (Hkv - 1) * G:] = want[0, (Hkv - 1) * G:]
    assert torch.equal(got, want)
