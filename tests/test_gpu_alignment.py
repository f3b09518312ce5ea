"""Weights, biases, gains, the LM head and the arena may start on any 4-byte
boundary: rebuilds and decode steps over copies 4 bytes past a 16-byte boundary
hold the bits of those over aligned ones."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_14635_amd import harness as Hn  # noqa: E402
from paper_2608_14635_amd import kvr  # noqa: E402
from paper_2608_14635_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

BASE = dataclasses.replace(W.TINY_F32, hidden=128, vocab=192)
SHAPES = {
    "f32_d16": dataclasses.replace(BASE, num_q_heads=16, num_kv_heads=8, head_dim=16, ffn_dim=56, qkv_bias=True),
    "f32_d64": dataclasses.replace(BASE, num_q_heads=6, num_kv_heads=2, head_dim=64, ffn_dim=344, qk_norm=True,
                                   qkv_bias=True),
    "f32_d128": dataclasses.replace(BASE, num_q_heads=2, num_kv_heads=1, head_dim=128, ffn_dim=264),
    "bf16": dataclasses.replace(W.TINY_BF16.with_layers(2), vocab=1024, qkv_bias=True),
    "bf16_norm": dataclasses.replace(W.TINY_BF16.with_layers(2), vocab=1024, qk_norm=True, qkv_bias=True),
}


def shifted(t, nbytes):
    """A copy of t that starts nbytes past a 16-byte boundary."""
    n = nbytes // t.element_size()
    raw = torch.empty(t.numel() + 16, dtype=t.dtype, device="cuda")
    assert raw.data_ptr() % 16 == 0
    out = raw[n:n + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("name", list(SHAPES))
def test_results_do_not_depend_on_alignment(name):
    shape = SHAPES[name]
    lens = [1, 70, 300]
    wl = W.small_workload(shape, [n + 1 for n in lens], seed=851, other_live_frac=0.0)
    toks = wl.tokens[:sum(lens)]
    ln = np.array(lens, np.int32)
    base = Hn.device_model_random(shape, seed=852, gain_std=0.1)
    head = Hn.device_head_random(shape, seed=853)
    got = []
    for by in (0, 4):
        print(f"{name}: {by} bytes past a boundary", flush=True)
        embed = shifted(base.embed, by)
        layers = [{k: shifted(t, by) for k, t in lw.items()} for lw in base.layers]
        model = Hn.model_view(shape, embed, layers)
        hd = {k: shifted(t, by) for k, t in head.items()}
        bits = shifted(torch.zeros(wl.arena_elems(), dtype=torch.int32 if shape.dtype == W.F32 else torch.int16,
                                   device="cuda"), by)
        handle = kvr.kv_arena_bind(bits.data_ptr(), bits.numel() * bits.element_size(), shape, wl.block_size,
                                   wl.num_blocks)
        ws, n = Hn.alloc_workspace(shape, len(lens), sum(lens), sum(lens), fill=0xFF)
        kvr.kv_rebuild(model.weights, toks, ln, wl.block_tables, handle, ws.data_ptr(), n, Hn.stream_ptr())
        torch.cuda.synchronize()
        rebuilt = bits.clone()
        n = kvr.kv_decode_workspace_bytes(shape, len(lens), max(lens) + 1)
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        nxt = torch.zeros(len(lens), dtype=torch.int32, device="cuda")
        logits = torch.zeros(len(lens), shape.vocab, dtype=torch.float32, device="cuda")
        kvr.kv_decode_step(model.weights, hd["final_norm"].data_ptr(), hd["lm_head"].data_ptr(),
                           np.array([1, 2, 3], np.int32), ln, wl.block_tables, handle, ws.data_ptr(), n,
                           nxt.data_ptr(), logits.data_ptr(), Hn.stream_ptr())
        torch.cuda.synchronize()
        kvr.kv_arena_release(handle)
        assert torch.isfinite(logits).all()
        got.append((rebuilt, bits, nxt, logits.view(torch.int32)))
    for a, b in zip(*got):
        assert torch.equal(a, b)
