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

from gpu_util import assert_close, dev_bf16, image
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


def images(name, seed, scale=1.0):
    """The oracle's cache, and the bits of the images' key halves hi and lo, [B, H, blocks, 32, D]."""
    from paper_2609_04263_amd import kvq
    fmt, D = FORMATS[name]
    K, V = synth.kv_tokens(seed, B, N, H, D)
    if scale != 1.0:  # a power of two, exact
        K = synth.to_bf16_bits((K.astype(np.uint32) << 16).view(np.float32) * np.float32(scale))
    ref = oracle.Cache(fmt, B, H, D, N)
    ref.append(K, V)
    gc = kvq.Cache(fmt, B, H, D, N)
    gc.append(dev_bf16(K), dev_bf16(V))
    assert np.array_equal(image(gc), ref.image), "cache images differ"
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
