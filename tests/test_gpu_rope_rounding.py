"""The bf16 rebuild's per-head norm and rotation, bit for bit: with zero key
weights a projected key is its bias, so a stored K follows from the bias, the
gain and the position by the fp32 operations listed here, each correctly rounded
(HIP's square root and division are), and one rounding to bf16.  No tolerance:
one FMA placed elsewhere, or the squares summed in another order, flips some ten
of the stored values."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_14635_amd import harness as Hn  # noqa: E402
from paper_2608_14635_amd import kvr  # noqa: E402
from paper_2608_14635_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu
HEADS = 16


def fma(a, b, c):
    """fp32 a * b + c with one rounding (the 64-bit significand of a long double
    holds the product and the sum but for ties no input here comes near)."""
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(np.float32)


def expected(k, gain, n, s):
    """K rows [n, HEADS, 128] as bf16 bits of keys k [HEADS, 128]."""
    if gain is not None:
        part = np.zeros((HEADS, 8), np.float32)
        v = k.reshape(HEADS, 8, 16)
        for i in range(16):  # a chain of FMAs over each part's 16 dims
            part = fma(v[..., i], v[..., i], part)
        while part.shape[1] > 1:  # the parts pairwise
            part = part[:, 0::2] + part[:, 1::2]
        inv = np.float32(1) / np.sqrt(part / np.float32(128) + np.float32(s.rms_eps))
        k = k * inv * gain
    angle = np.arange(n, dtype=np.float64)[:, None] * np.power(float(s.rope_theta), -np.arange(0, 128, 2) / 128.0)
    c, t = (f(angle).astype(np.float32)[:, None] for f in (np.cos, np.sin))
    c, t, a, b = np.broadcast_arrays(c, t, k[:, :64], k[:, 64:])
    out = np.concatenate([fma(a, c, -(b * t)), fma(a, t, b * c)], -1)
    return torch.from_numpy(out).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("n", [300, 2000])
@pytest.mark.parametrize("norm", [False, True])
def test_stored_keys_follow_from_their_bias(norm, n):
    s = dataclasses.replace(W.TINY_BF16, num_layers=1, hidden=256, num_q_heads=HEADS, num_kv_heads=HEADS, vocab=64,
                            qkv_bias=True, qk_norm=norm)
    host_w = W.host_weights(s, seed=831)
    lw = host_w["layers"][0]
    lw["wk"][:] = 0
    wl = W.small_workload(s, [n], seed=832, other_live_frac=0.0)
    model = Hn.device_model_from_host(s, host_w)
    arena = Hn.DeviceArena(wl)
    arena.bind()
    ws, nbytes = Hn.alloc_workspace(s, 1, n, n)
    kvr.kv_rebuild(model.weights, wl.tokens, wl.lens, wl.block_tables, arena.handle, ws.data_ptr(), nbytes,
                   Hn.stream_ptr())
    torch.cuda.synchronize()
    p = np.arange(n)
    shp = (2, wl.num_blocks, wl.block_size, HEADS, 128)
    got = arena.to_host().reshape(shp)[0, wl.block_tables[0, p // wl.block_size], p % wl.block_size]
    arena.release()
    want = expected(W.bf16_bits_to_f32(lw["bk"]).reshape(HEADS, 128),
                    W.bf16_bits_to_f32(lw["k_norm"]) if norm else None, n, s)
    print(f"norm={norm} n={n}: {int((got != want).sum())} of {got.size} values differ", flush=True)
    assert np.array_equal(got, want)
