"""Decode steps at the edges of their kernels' ranges, against the oracle: more
requests than one wave of the range scan (64) and than the few-row products (64),
ragged contexts on both sides of a key range's length, vocabularies that end on
each column block of the row-major LM head, per-head norms with few rows, and a
logits buffer that is only 4-byte aligned.  Tolerances as in test_gpu_decode."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_14635_amd import harness as Hn  # noqa: E402
from paper_2608_14635_amd import kvr  # noqa: E402
from paper_2608_14635_amd import workloads as W  # noqa: E402

import parity_util as PU  # noqa: E402
import test_gpu_decode as TD  # noqa: E402

pytestmark = pytest.mark.gpu

T2 = W.TINY_BF16.with_layers(2)
CASES = {
    "130req_ragged": (dataclasses.replace(T2, vocab=1024), [1 + (37 * i) % 701 for i in range(130)], 0),
    "66req_vocab_128": (dataclasses.replace(T2, vocab=896), [1 + (11 * i) % 90 for i in range(66)], 0),
    "5req_vocab_16": (dataclasses.replace(T2, vocab=1008), [63, 64, 65, 127, 129], 0),
    "33req_vocab_32": (dataclasses.replace(T2, vocab=992), [1 + (5 * i) % 140 for i in range(33)], 0),
    "3req_norm": (dataclasses.replace(T2, vocab=1024, qk_norm=True), [2, 200, 17], 0),
    "20req_norm_bias": (dataclasses.replace(T2, vocab=1024, qk_norm=True, qkv_bias=True),
                        [1 + (7 * i) % 60 for i in range(20)], 0),
    "70req_norm": (dataclasses.replace(T2, vocab=1024, qk_norm=True), [1 + (7 * i) % 60 for i in range(70)], 0),
    # vocabularies large enough for 256 x 256 tiles: row-major and transposed
    "300req_vocab_152064": (dataclasses.replace(T2, num_layers=1, hidden=256, vocab=152064), [1 + i % 5 for i in range(300)], 1),
    "3req_vocab_152065": (dataclasses.replace(T2, num_layers=1, hidden=256, vocab=152065), [2, 40, 17], 1),
    "4req_unaligned_logits": (dataclasses.replace(T2, vocab=1024), [3, 40, 15, 16], 1),
}


# the general attention kernel in bf16 (blocks that hold no whole 16-key tiles) over
# several ranges a request; it and the matrix-core kernel where the number of
# requests changes the length of the ranges
KERNELS = {
    "b8_ragged": (T2, [1, 63, 64, 65, 700, 1500, 129], 8),
    "b24_ragged": (T2, [1, 63, 64, 65, 700, 1500, 129], 24),
    "b8_130req": (T2.with_layers(1), [1 + (37 * i) % 301 for i in range(130)], 8),
    "f32_95req": (W.TINY_F32.with_layers(1), [1 + (37 * i) % 301 for i in range(95)], 16),
    "f32_96req": (W.TINY_F32.with_layers(1), [1 + (37 * i) % 301 for i in range(96)], 16),
    "g16_65req": (dataclasses.replace(T2.with_layers(1), num_q_heads=32), [1 + (37 * i) % 301 for i in range(65)], 16),
}


@pytest.mark.parametrize("name", list(KERNELS))
def test_decode_kernels_and_ranges(oracle_lib, name):
    shape, prefix, block_size = KERNELS[name]
    check_step(oracle_lib, name, shape, prefix, 0, block_size)


# more requests than two probes of the range lookup tell apart
def test_decode_of_4100_requests(oracle_lib):
    shape = dataclasses.replace(T2, num_layers=1, hidden=256, ffn_dim=256, vocab=128)
    check_step(oracle_lib, "4100 requests", shape, [1 + (i * i) % 11 for i in range(4100)], 0)


@pytest.mark.parametrize("name", list(CASES))
def test_decode_edges(oracle_lib, name):
    check_step(oracle_lib, name, *CASES[name])


def check_step(oracle_lib, name, shape, prefix, shift, block_size=16):
    tol = PU.TOL[shape.dtype]
    wl = TD.resume_workload(shape, prefix, steps=2, seed=801, block_size=block_size)
    R = len(prefix)
    TD.say(f"{name}: {R} requests")
    host_w, head = W.host_weights(shape, seed=802), W.host_head_weights(shape, seed=803)
    model = Hn.device_model_from_host(shape, host_w)
    hd = Hn.device_head_from_host(shape, head)
    image = W.host_arena(wl)
    # the oracle's own prefixes on both sides
    pre, last = TD.split_last(wl)
    ora = image.copy()
    oracle_lib.rebuild(shape, host_w, pre.tokens, pre.lens, pre.block_tables, ora, wl.block_size, wl.num_blocks)
    arena = Hn.DeviceArena(wl, host_image=ora)
    arena.bind()
    pos = (wl.lens - 1).astype(np.int32)
    nbytes = kvr.kv_decode_workspace_bytes(shape, R, int(pos.max()) + 1)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    nxt = torch.zeros(R, dtype=torch.int32, device="cuda")
    raw = torch.zeros(R * shape.vocab + 4, dtype=torch.float32, device="cuda")
    logits = raw[shift:shift + R * shape.vocab]
    kvr.kv_decode_step(model.weights, hd["final_norm"].data_ptr(), hd["lm_head"].data_ptr(), last, pos,
                       wl.block_tables, arena.handle, ws.data_ptr(), nbytes, nxt.data_ptr(),
                       logits.data_ptr(), Hn.stream_ptr())
    torch.cuda.synchronize()
    before = ora.copy()
    fh = oracle_lib.decode_step(shape, host_w, last, pos, wl.block_tables, ora, wl.block_size, wl.num_blocks)
    want = oracle_lib.logits(shape, head, fh)
    got = logits.view(R, shape.vocab).cpu().numpy()
    errs = [TD.rel(got[r], want[r]) for r in range(R)]
    g = arena.to_host()
    kv = TD.rel(PU.to_float(TD.slot_rows(wl, g, pos), shape.dtype), PU.to_float(TD.slot_rows(wl, ora, pos), shape.dtype))
    TD.say(f"  worst logits {max(errs):.2e}, new rows {kv:.2e}")
    assert max(errs) <= tol and kv <= tol
    TD.assert_valid_argmax(nxt.cpu().numpy(), want, tol)
    # nothing but the new slots changed
    shp = (shape.num_layers, 2, wl.num_blocks, wl.block_size, -1)
    m = np.zeros(shp[:4], bool)
    for r, p in enumerate(pos):
        m[:, :, wl.block_tables[r, p // wl.block_size], p % wl.block_size] = True
    assert np.array_equal(g.reshape(shp)[~m], before.reshape(shp)[~m])
    arena.release()


@pytest.mark.parametrize("R", [1, 20, 64, 65])
def test_decode_v_that_is_not_finite_stays_in_its_dim(oracle_lib, R):
    """V has no rotary partners: an infinite and a NaN bias reach their own dims of
    the new V rows and no others."""
    shape = dataclasses.replace(T2, num_layers=1, vocab=1024, qkv_bias=True)
    wl = TD.resume_workload(shape, [1 + (3 * i) % 20 for i in range(R)], steps=2, seed=811)
    TD.say(f"{R} requests, value biases that are not finite")
    host_w, head = W.host_weights(shape, seed=812), W.host_head_weights(shape, seed=813)
    bv = host_w["layers"][0]["bv"]
    bv[3], bv[128 + 100] = 0x7F80, 0x7FC0
    model = Hn.device_model_from_host(shape, host_w)
    hd = Hn.device_head_from_host(shape, head)
    image = np.zeros_like(W.host_arena(wl))
    arena = Hn.DeviceArena(wl, host_image=image)
    arena.bind()
    pos = (wl.lens - 1).astype(np.int32)
    tok = np.arange(R, dtype=np.int32) % shape.vocab
    GD = TD.GpuDecoder(wl, model, hd, int(pos.max()) + 1)
    GD.step(arena, tok, pos)
    g = PU.to_float(TD.slot_rows(wl, arena.to_host(), pos), W.BF16)
    arena.release()
    oracle_lib.decode_step(shape, host_w, tok, pos, wl.block_tables, image, wl.block_size, wl.num_blocks)
    o = PU.to_float(TD.slot_rows(wl, image, pos), W.BF16)
    assert np.array_equal(np.isfinite(g), np.isfinite(o)) and (~np.isfinite(g)).sum() == 2 * R
    assert (g[0, 1, :, 3] == np.inf).all() and np.isnan(g[0, 1, :, 228]).all()
    ok = np.isfinite(o)
    assert TD.rel(g[ok], o[ok]) <= PU.TOL[W.BF16]


@pytest.mark.parametrize("R", [4, 66])
def test_logits_do_not_depend_on_their_buffers_alignment(R):
    shape = dataclasses.replace(T2, num_layers=1, vocab=1024)
    wl = TD.resume_workload(shape, [1] * R, steps=2, seed=841)
    TD.say(f"{R} requests, logits 0 to 3 floats past a 16-byte boundary")
    model = Hn.device_model_random(shape, seed=842)
    GD = TD.GpuDecoder(wl, model, Hn.device_head_random(shape, seed=843), 1)
    arena = Hn.DeviceArena(wl)
    arena.bind()
    raw = torch.zeros(R * shape.vocab + 4, dtype=torch.float32, device="cuda")
    got = []
    for shift in range(4):
        GD.logits = raw[shift:shift + R * shape.vocab].view(R, shape.vocab)
        got.append(GD.step(arena, np.arange(R, dtype=np.int32), np.zeros(R, np.int32)))
    arena.release()
    for tok, logits in got[1:]:
        assert np.array_equal(tok, got[0][0]) and np.array_equal(logits.view(np.uint32), got[0][1].view(np.uint32))


def test_decode_of_more_requests_than_a_grid_is_wide(oracle_lib):
    """262,148 requests at position 0, 128 tokens over and over: each gets the token
    the first with its own gets, and those are the oracle's."""
    R, n = 262148, 128
    shape = dataclasses.replace(T2, num_layers=1, hidden=256, num_q_heads=2, num_kv_heads=2, ffn_dim=128, vocab=n)
    TD.say(f"{R} requests")
    host_w, head = W.host_weights(shape, seed=821), W.host_head_weights(shape, seed=822)
    model, hd = Hn.device_model_from_host(shape, host_w), Hn.device_head_from_host(shape, head)
    bits = torch.zeros(1, 2, R, 1, 2, 128, dtype=torch.int16, device="cuda")
    handle = kvr.kv_arena_bind(bits.data_ptr(), bits.numel() * 2, shape, 1, R)
    tok, pos = (np.arange(R) % n).astype(np.int32), np.zeros(R, np.int32)
    nbytes = kvr.kv_decode_workspace_bytes(shape, R, 1)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    nxt = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    kvr.kv_decode_step(model.weights, hd["final_norm"].data_ptr(), hd["lm_head"].data_ptr(), tok, pos,
                       np.arange(R, dtype=np.int32)[:, None], handle, ws.data_ptr(), nbytes, nxt.data_ptr(), 0,
                       Hn.stream_ptr())
    torch.cuda.synchronize()
    kvr.kv_arena_release(handle)
    got = nxt.cpu().numpy()
    image = np.zeros(2 * n * 2 * 128, np.uint16)
    fh = oracle_lib.decode_step(shape, host_w, tok[:n], pos[:n], np.arange(n, dtype=np.int32)[:, None], image, 1, n)
    TD.assert_valid_argmax(got[:n], oracle_lib.logits(shape, head, fh), PU.TOL[shape.dtype])
    assert np.array_equal(got, np.resize(got[:n], R))
