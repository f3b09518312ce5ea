"""The fp32 matrix-core products and attention at the sizes where they can go
wrong: every head size, FFN widths that end inside a 16-column group and a
32-wide K tile, requests around the 16-query, 32- and 64-row tiles, batches large
enough for the 64 x 64 tiles, against the CPU oracle (fp64 sums).  Tolerance: the
rebuild's 1e-4; sums of at most 768 products of fp32 values differ by about
1e-6 of the largest."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_14635_amd import harness as Hn  # noqa: E402
from paper_2608_14635_amd import kvr  # noqa: E402
from paper_2608_14635_amd import workloads as W  # noqa: E402

import parity_util as PU  # noqa: E402

pytestmark = pytest.mark.gpu

BASE = dataclasses.replace(W.TINY_F32, hidden=128, vocab=200)
SHAPES = {
    "d16": dataclasses.replace(BASE, num_q_heads=16, num_kv_heads=8, head_dim=16, ffn_dim=8),
    "d16_bias": dataclasses.replace(BASE, num_q_heads=8, num_kv_heads=8, head_dim=16, ffn_dim=56, qkv_bias=True),
    "d32_norm": dataclasses.replace(BASE, num_q_heads=8, num_kv_heads=4, head_dim=32, ffn_dim=40, qk_norm=True),
    "d64_norm_bias": dataclasses.replace(BASE, num_q_heads=6, num_kv_heads=2, head_dim=64, ffn_dim=344,
                                         qk_norm=True, qkv_bias=True),
    "d128_norm": dataclasses.replace(BASE, num_q_heads=4, num_kv_heads=1, head_dim=128, ffn_dim=264, qk_norm=True),
    "d128": dataclasses.replace(BASE, num_q_heads=2, num_kv_heads=2, head_dim=128, ffn_dim=768),
}


def rebuild(wl, model, image):
    arena = Hn.DeviceArena(wl, host_image=image)
    arena.bind()
    ws, n = Hn.alloc_workspace(wl.shape, wl.num_requests, wl.total_tokens, wl.total_tokens, fill=0xFF)
    kvr.kv_rebuild(model.weights, wl.tokens, wl.lens, wl.block_tables, arena.handle, ws.data_ptr(), n,
                   Hn.stream_ptr())
    torch.cuda.synchronize()
    arena.release()
    return arena.to_host()


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("lens", [[1, 15, 16, 17, 63, 64, 65], [129, 300]])
def test_f32_edges(oracle_lib, name, lens):
    shape = SHAPES[name]
    wl = W.small_workload(shape, lens, seed=711, other_live_frac=0.2)
    print(f"{name} lens={lens}", flush=True)
    host_w = W.host_weights(shape, seed=712)
    image = W.host_arena(wl)
    got = rebuild(wl, Hn.device_model_from_host(shape, host_w), image)
    want = image.copy()
    oracle_lib.rebuild(shape, host_w, wl.tokens, wl.lens, wl.block_tables, want, wl.block_size, wl.num_blocks)
    _, rep = PU.compare(wl, got, want, image)
    print("  ", rep, flush=True)
    assert rep["unwritten_changed"] == 0 and rep["written_nonfinite"] == 0 and rep["worst"] <= 1e-4


def test_f32_large_tiles_keep_the_bits():
    """A request in a batch large enough for the 64 x 64 tiles holds the bits it has alone."""
    shape = SHAPES["d64_norm_bias"], SHAPES["d128"]
    for s in shape:
        wl = W.small_workload(s, [70, 200] + [900] * 20, seed=721, other_live_frac=0.0)
        model = Hn.device_model_from_host(s, W.host_weights(s, seed=722))
        image = W.host_arena(wl)
        shp = (s.num_layers, 2, wl.num_blocks, wl.block_size, -1)
        whole = rebuild(wl, model, image).reshape(shp)
        off = wl.request_offsets()
        for r in (0, 1, 2):
            one = dataclasses.replace(wl, lens=wl.lens[r:r + 1].copy(), tokens=wl.tokens[off[r]:off[r + 1]].copy(),
                                      block_tables=wl.block_tables[r:r + 1].copy())
            alone = rebuild(one, model, image).reshape(shp)
            p = np.arange(int(wl.lens[r]))
            blk, sl = wl.block_tables[r, p // wl.block_size], p % wl.block_size
            assert np.array_equal(whole[:, :, blk, sl], alone[:, :, blk, sl]), (s.head_dim, r)


def poisoned(shape, host_w, kind):
    """Token 0's row, made to give a layer-0 K and V of NaN, or a V of infinities
    over a finite K: hidden dim 0 is token 0's own, and Wv's column of it is huge."""
    host_w["embed"][:, 0] = 0.0
    host_w["embed"][0, 0] = np.inf if kind == "nan" else 1.0
    if kind == "inf_v":
        host_w["layers"][0]["wv"][:, 0] = 3e38


# the poisoned token on both sides of the edges of the 16-key pieces and the 64-key
# tiles, in a request that ends inside one
@pytest.mark.parametrize("kind", ["nan", "inf_v"])
@pytest.mark.parametrize("name", ["d16", "d64_norm_bias", "d128"])
def test_f32_later_keys_that_are_not_finite(oracle_lib, name, kind):
    """Earlier positions keep their bits whatever a later key's values are, and the
    rows that are not finite are the oracle's."""
    shape, n = SHAPES[name], 141
    wl = W.small_workload(shape, [n], seed=731, other_live_frac=0.0)
    wl.tokens[wl.tokens == 0] = 1
    host_w = W.host_weights(shape, seed=732)
    poisoned(shape, host_w, kind)
    model = Hn.device_model_from_host(shape, host_w)
    image = W.host_arena(wl)
    p = np.arange(n)
    shp = (shape.num_layers, 2, wl.num_blocks, wl.block_size, -1)
    rows = lambda a: PU.to_float(a.reshape(shp)[:, :, wl.block_tables[0, p // wl.block_size], p % wl.block_size], W.F32)
    clean = rows(rebuild(wl, model, image))
    assert np.isfinite(clean).all()
    for t in (0, 1, 15, 16, 40, 63, 64, 79, 127, 128, 140):
        print(f"{name} {kind}: position {t}", flush=True)
        bad = dataclasses.replace(wl, tokens=wl.tokens.copy())
        bad.tokens[t] = 0
        got = rows(rebuild(bad, model, image))
        want = image.copy()
        oracle_lib.rebuild(shape, host_w, bad.tokens, bad.lens, bad.block_tables, want, bad.block_size, bad.num_blocks)
        want = rows(want)
        assert np.array_equal(got[:, :, :t].view(np.uint32), clean[:, :, :t].view(np.uint32))
        assert np.array_equal(np.isfinite(got), np.isfinite(want))
        assert not np.isfinite(got[1, :, t + 1:]).any()
