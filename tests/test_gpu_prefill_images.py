"""The block images a chunked prefill leaves in its workspace, against the oracle's reconstruction.

A call of many query rows reconstructs every visible 32-token block into the
workspace (192 D bytes: keys as binary16 hi and lo halves, then the values, in
fragment order), where a test can read them: the keys' precision shows there
alone, behind the roundings of probabilities and values in the outputs.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_04263_amd import configs, synth

from gpu_util import assert_close, dev_bf16, image, prefill_ranges
from test_gpu_append import CASES

pytestmark = pytest.mark.gpu

FORMATS = {
    "kivi": CASES["kivi"],
    "perch_k4v2_window64": CASES["perch_k4v2_window64"],
    "perch8_meta16": CASES["perch8_meta16"],
    # eight key groups per token: hi + lo keys instead of exact codes
    "affine_g32_d256": (configs.make_format(4, 4, k_group=32, v_group=32), 256),
}

B, H, G, N, C = 4, 8, 4, 293, 260  # 32 units of 1040 rows: the workspace path at every head size


def scaled_kv(seed, B, n, H, D, scale):
    """Keys times powers of two (exact in bf16; one, or one per token), and values."""
    K, V = synth.kv_tokens(seed, B, n, H, D)
    return synth.to_bf16_bits(synth.bf16_bits_to_f32(K) * np.asarray(scale, dtype=np.float32).reshape(1, -1, 1, 1)), V


def images(name, seed, scale=1.0):
    """The oracle's cache, and the bits of the images' key halves hi and lo, [B, H, blocks, 32, D]."""
    from paper_2609_04263_amd import kvq
    fmt, D = FORMATS[name]
    K, V = scaled_kv(seed, B, N, H, D, scale)
    ref = oracle.Cache(fmt, B, H, D, N)
    ref.append(K, V)
    gc = kvq.Cache(fmt, B, H, D, N)
    gc.append(dev_bf16(K), dev_bf16(V))
    assert np.array_equal(image(gc), ref.image), "cache images differ"
    assert prefill_ranges(gc, C, H * G) == 0
    Q = synth.normal_bf16(seed, ("chunk-q",), (B, C, H * G, D))
    O = torch.empty((B, C, H * G, D), dtype=torch.float32, device="cuda")
    ws = torch.full((gc.prefill_workspace_bytes(),), 0xFF, dtype=torch.uint8, device="cuda")
    sm = 1.0 / np.sqrt(D) / scale
    gc.prefill_attn(dev_bf16(Q), C, H * G, sm, O, ws)
    assert_close(O.cpu().numpy(), ref.prefill_attn(Q, sm), what=name)
    img = ws.cpu().numpy().reshape(B, H, -1, 192 * D)

    def part(i):  # channels 8 P .. 8 P + 7 of token t are 16 bytes at 512 P + 16 t
        h = np.ascontiguousarray(img[..., 64 * D * i:64 * D * (i + 1)]).view(np.uint16)
        h = h.reshape(B, H, -1, D // 8, 32, 8).transpose(0, 1, 2, 4, 3, 5)
        return np.ascontiguousarray(h).reshape(B, H, -1, 32, D)

    return ref, part(0), part(1)


def f64(bits):
    return bits.view(np.float16).astype(np.float64)


@pytest.mark.parametrize("name", list(FORMATS))
def test_hi_lo_keys(name):
    ref, hi, lo = images(name, seed=900)
    k = ref.dequant()[0]
    got = (f64(hi) + f64(lo)).reshape(B, H, -1, k.shape[-1])[:, :, :N]
    # hi and lo rounded to nearest (2^-23), after one fp32 rounding of c s + z
    # (2^-24); lo subnormal below 2^-14 (2^-25)
    bound = (2.0 ** -23 + 2.0 ** -24) * np.abs(k) + 2.0 ** -25
    over = np.abs(got - k) > bound
    assert not over.any(), f"{name}: {over.sum()} of {k.size} keys"


ROTATING = {
    "hadamard": CASES["hadamard"],
    "had_affine_window": CASES["had_affine_window"],
    "kvarn_sink": CASES["kvarn_sink"],
    "had_d64_g32": (configs.make_format(4, 4, k_group=32, v_group=32, rotate=64), 64),
    "had8_d128": (configs.make_format(8, 8, k_group=64, v_group=64, rotate=128), 128),
    "had_perch_window": (configs.make_format(4, 2, k_axis=1, k_group=32, v_group=32, residual=32, flush=32,
                                             rotate=128), 128),
}
FORMATS.update(ROTATING)


def fwht64(x):
    """The normalized Hadamard transform of the last axis in 64 bits."""
    D = x.shape[-1]
    h = 1
    while h < D:
        v = x.reshape(*x.shape[:-1], D // (2 * h), 2, h)
        x = np.stack((v[..., 0, :] + v[..., 1, :], v[..., 0, :] - v[..., 1, :]), axis=-2).reshape(x.shape)
        h *= 2
    return x / np.sqrt(D)


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -14, 2.0 ** 9])
@pytest.mark.parametrize("name", list(ROTATING))
def test_rotated_keys_keep_their_precision_at_any_magnitude(name, scale):
    ref, hi, lo = images(name, seed=910, scale=scale)
    D = hi.shape[-1]
    # octet j's exponent: bit 14 of the lo halves of channel D / 2 of its eight tokens
    octets = (B, H, -1, 8)
    bits = ((lo[..., D // 2] >> 14) & 1).reshape(octets).astype(np.int64)
    ef = (bits << np.arange(8)).sum(axis=-1).repeat(8, axis=-1)
    lo = lo.copy()
    lo[..., D // 2] &= 0xBFFF
    assert np.abs(f64(lo)).max() <= 1.0 and np.abs(f64(hi)).max() <= 4096.0
    got = (f64(hi) + f64(lo)).reshape(B, H, -1, D) * 2.0 ** (ef[..., None] - 134.0)
    want = np.zeros_like(got)
    want[:, :, :N] = fwht64(ref.dequant()[0])  # (stored rotated)
    octet_max = np.abs(want).max(axis=-1).reshape(octets).max(axis=-1).repeat(8, axis=-1)
    # the split; then a transform in fp32 (log2 D stages and the product, each
    # rounding within 2^-24 of the vector's length) of keys rounded once
    length = np.sqrt((want ** 2).sum(axis=-1, keepdims=True))
    bound = 2.0 ** -23 * np.abs(want) + 2.0 ** -25 * octet_max[..., None] + (np.log2(D) + 2) * 2.0 ** -24 * length
    over = np.abs(got - want) > bound
    assert not over.any(), f"{name}: {over.sum()} of {want.size} keys"


SHAPES = pytest.mark.parametrize("shape", [dict(b=1, h=1, g=2, n=1493, c=23), dict(b=B, h=H, g=G, n=N, c=C)],
                                 ids=["fused", "workspace"])


def relative_error(name, seed, scale, sm, b, h, g, n, c):
    from paper_2609_04263_amd import kvq
    fmt, D = FORMATS[name]
    K, V = scaled_kv(seed, b, n, h, D, scale)
    ref = oracle.Cache(fmt, b, h, D, n)
    ref.append(K, V)
    gc = kvq.Cache(fmt, b, h, D, n)
    gc.append(dev_bf16(K), dev_bf16(V))
    Q = synth.normal_bf16(seed, ("chunk-q",), (b, c, h * g, D))
    O = torch.empty((b, c, h * g, D), dtype=torch.float32, device="cuda")
    gc.prefill_attn(dev_bf16(Q), c, h * g, sm / np.sqrt(D), O, gc.prefill_workspace())
    want = ref.prefill_attn(Q, sm / np.sqrt(D))
    return np.linalg.norm(O.cpu().numpy() - want) / np.linalg.norm(want)


# Probabilities and values are rounded to binary16, 2^-11 each; nothing else may
# show in the outputs.
@SHAPES
@pytest.mark.parametrize("name", list(ROTATING))
def test_rotated_outputs_of_small_keys(name, shape):
    # the scores of ordinary keys, from keys of 2^-14 and a softmax scale of 2^14
    assert relative_error(name, 920, 2.0 ** -14, 2.0 ** 14, **shape) <= 2.0 ** -10


@SHAPES
@pytest.mark.parametrize("name", list(ROTATING))
def test_rotated_outputs_of_mixed_magnitudes(name, shape):
    # octets with different exponents in one block
    scale = 2.0 ** -(5.0 * (np.arange(shape["n"]) // 8 % 3))
    assert relative_error(name, 925, scale, 1.0, **shape) <= 2.0 ** -10


def test_rotated_keys_beyond_binary16():
    # codes and scales hold keys of 2^20; a softmax that one key takes whole
    from paper_2609_04263_amd import kvq
    fmt, D = FORMATS["hadamard"]
    K, V = scaled_kv(930, 1, 320, 2, D, 2.0 ** 20)
    ref = oracle.Cache(fmt, 1, 2, D, 320)
    ref.append(K, V)
    gc = kvq.Cache(fmt, 1, 2, D, 320)
    gc.append(dev_bf16(K), dev_bf16(V))
    Q = synth.normal_bf16(931, ("chunk-q",), (1, 40, 4, D))
    O = torch.empty((1, 40, 4, D), dtype=torch.float32, device="cuda")
    gc.prefill_attn(dev_bf16(Q), 40, 4, 1.0, O, gc.prefill_workspace())
    assert torch.isfinite(O).all()
    assert_close(O.cpu().numpy(), ref.prefill_attn(Q, 1.0), what="keys of 2^20")


CODED = {name: CASES[name] for name in ("tiny_b1", "tiny_b16", "affine2_g128", "gqa12b", "g256", "affine8", "tiny_meta16",
                                        "sym4_window")}
CODED["affine_g32_d128"] = (configs.make_format(4, 4, k_group=32, v_group=32), 128)
FORMATS.update(CODED)


@pytest.mark.parametrize("name", list(CODED))
def test_code_blocks_keep_scales_and_offsets_as_stored(name):
    # a code block's lo half: the groups' scales, then their offsets, each the
    # stored value in fp32, so that a score takes one rounding per group
    ref, _, lo = images(name, seed=950)
    fmt, D = FORMATS[name]
    ng, blocks = D // fmt["k_group"], (ref.n_coded + 31) // 32
    meta = np.float16 if fmt["meta_fp16"] else np.float32

    def stored(section):
        return ref.section(section).view(meta).reshape(B, H, -1, 32 * ng)[:, :, :blocks].astype(np.float32)

    # part() put the bytes in token order: back to the order of the image
    raw = lo.reshape(B, H, -1, 32, D // 8, 8).transpose(0, 1, 2, 4, 3, 5).reshape(B, H, -1, 32 * D)
    got = np.ascontiguousarray(raw).view(np.float32)[:, :, :blocks]
    live = np.arange(32 * blocks).reshape(blocks, 1, 32) < ref.n_coded
    live = np.broadcast_to(live, (blocks, ng, 32)).reshape(blocks, 32 * ng)
    s = stored(1)
    z = stored(2) if fmt["k_mode"] == 0 else -np.float32(2 ** (fmt["k_bits"] - 1)) * s
    assert (got[..., :32 * ng] == s)[:, :, live].all()
    assert (got[..., 32 * ng:64 * ng] == z)[:, :, live].all()
