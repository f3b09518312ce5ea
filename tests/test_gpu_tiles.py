"""The bf16 products pick their tile by the row and column counts: a request
rebuilt alone (small tiles), in a batch of short requests and in a long batch
(256 x 256 tiles) holds the same bits, for plain, q/k-normed and biased heads."""
import dataclasses
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_14635_amd import harness as Hn  # noqa: E402
from paper_2608_14635_amd import kvr  # noqa: E402
from paper_2608_14635_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def rebuild(wl, model):
    arena = Hn.DeviceArena(wl)
    arena.bind()
    ws, n = Hn.alloc_workspace(wl.shape, wl.num_requests, wl.total_tokens, wl.total_tokens, fill=0xFF)
    kvr.kv_rebuild(model.weights, wl.tokens, wl.lens, wl.block_tables, arena.handle, ws.data_ptr(), n,
                   Hn.stream_ptr())
    torch.cuda.synchronize()
    arena.release()
    return arena


def rows_of(wl, arena, r):
    p = np.arange(int(wl.lens[r]))
    blk = torch.as_tensor(wl.block_tables[r, p // wl.block_size].astype(np.int64), device="cuda")
    return arena.bits[:, :, blk, torch.as_tensor(p % wl.block_size, device="cuda")]


# lengths that end inside, on and just past the 32-, 64-, 128- and 256-row tiles
LENS = [1, 64, 65, 130, 250, 257, 520, 1030, 2050]


@pytest.mark.parametrize("name", ["llama8b", "qwen3_8b", "qwen25_1_5b", "tiny_bf16"])
def test_a_request_keeps_its_bits_whatever_the_tile(name):
    shape = W.SHAPES[name].with_layers(2)
    wl = W.small_workload(shape, LENS, seed=611, other_live_frac=0.1)
    model = Hn.device_model_random(shape, seed=612, gain_std=0.1)
    print(f"{name}: {wl.total_tokens} tokens in one call", flush=True)
    whole = rebuild(wl, model)
    off = wl.request_offsets()
    for r, n in enumerate(LENS):
        one = dataclasses.replace(wl, lens=wl.lens[r:r + 1].copy(), tokens=wl.tokens[off[r]:off[r + 1]].copy(),
                                  block_tables=wl.block_tables[r:r + 1].copy())
        print(f"  {n} tokens alone", flush=True)
        alone = rebuild(one, model)
        a, b = rows_of(wl, whole, r), rows_of(one, alone, 0)
        assert torch.isfinite(b.view(torch.bfloat16)).all()
        assert torch.equal(a, b), f"{n} tokens: {(a != b).sum().item()} values differ"
    print("  in two long calls", flush=True)
    long = W.small_workload(shape, LENS + [9000], seed=611, other_live_frac=0.1)
    long = dataclasses.replace(long, tokens=np.concatenate([wl.tokens, long.tokens[wl.total_tokens:]]))
    big = rebuild(long, model)
    for r, n in enumerate(LENS):
        assert torch.equal(rows_of(wl, whole, r), rows_of(long, big, r)), f"{n} tokens in the long call"
    sys.stdout.flush()


@pytest.mark.parametrize("name", ["llama8b", "qwen3_8b", "qwen25_1_5b"])
def test_columns_shared_out_over_two_tiles_keep_their_bits(name):
    """Products whose last round of tiles would be mostly empty take two kinds of
    tile: q/k/v at 3000 rows (9000 for the 1.5B shape), the residual products at
    4400 and gate/up at 1003; in one call of all the rows there is one kind."""
    lens = [1003, 3000, 4400, 9000]
    shape = W.SHAPES[name].with_layers(2)
    wl = W.small_workload(shape, lens, seed=613, other_live_frac=0.1)
    model = Hn.device_model_random(shape, seed=614, gain_std=0.1)
    whole = rebuild(wl, model)
    off = wl.request_offsets()
    for r, n in enumerate(lens):
        print(f"{name}: {n} tokens alone", flush=True)
        one = dataclasses.replace(wl, lens=wl.lens[r:r + 1].copy(), tokens=wl.tokens[off[r]:off[r + 1]].copy(),
                                  block_tables=wl.block_tables[r:r + 1].copy())
        a, b = rows_of(wl, whole, r), rows_of(one, rebuild(one, model), 0)
        assert torch.equal(a, b), f"{n} tokens: {(a != b).sum().item()} values differ"
