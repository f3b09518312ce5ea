// Epilogues of the bf16 split-K products of a decode step through LDS (the tiled
// products finish from their accumulators: gemm_epi.h, gemm_f32.hip).  Head dim
// 128; per-head norms and biases as there.
//
// A tile's fp32 sums are first parked in LDS as sC[rows][ldc]; the routines
// below then read it in row-contiguous chunks so that every global store is a
// full 16-byte vector:
//   QKV    : NeoX RoPE on a q or k head (pairs (i, i + 64), fp32 cos/sin),
//            rounding, Q rows to the workspace, K and V rows to their arena slots;
//   SWIGLU : h = silu(gate) * up from the two column halves of the tile.
#pragma once
#include "common.h"
#include "launch.h"

namespace kvr {

// QKV: the tile is one head, logical columns [n0, n0 + 128) of one region
// (q: [0, nq*128), k: the next nkv*128, v: after that).  Biases are added to the
// sums first; with per-head q/k norms, a first pass writes each row's inverse RMS
// into the spare column 128 of the parked tile (ldc > 128), then the rotary pass
// scales by it and by the gain.
template <int NT>
__device__ __forceinline__ void epi_qkv(float* sC, int ldc, int rows, int m_base, int M, int n0,
                                        const EpiParams& e) {
  constexpr int D = 128, HALF = 64;
  const int tid = threadIdx.x;
  const int qcols = e.nq * D, kcols = e.nkv * D;
  const int region = n0 < qcols ? 0 : (n0 < qcols + kcols ? 1 : 2);
  const int rbase = n0 - (region == 0 ? 0 : region == 1 ? qcols : qcols + kcols);  // head's first column
  const bf16_t* bias = reinterpret_cast<const bf16_t*>(region == 0 ? e.bq : region == 1 ? e.bk : e.bv);
  if (region < 2) {
    const bf16_t* gain = reinterpret_cast<const bf16_t*>(region == 0 ? e.q_norm : e.k_norm);
    if (gain != nullptr) {
      // eight consecutive lanes per row, each summing 16 squares in index order
      for (int it = tid; it < rows * 8; it += NT) {
        const int r = it >> 3, part = it & 7;
        const float* src = sC + (int64_t)r * ldc + part * 16;
        float ss = 0.0f;
        for (int i = 0; i < 16; i += 4) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float v = src[i + k] + (bias ? bf2f(bias[rbase + part * 16 + i + k]) : 0.0f);
            ss += v * v;
          }
        }
        ss += __shfl_xor(ss, 1, 64);
        ss += __shfl_xor(ss, 2, 64);
        ss += __shfl_xor(ss, 4, 64);
        if (part == 0) sC[(int64_t)r * ldc + D] = 1.0f / sqrtf(ss / (float)D + e.eps);
      }
      __syncthreads();
    }
    // items: (row, chunk of 8 rotary pairs)
    for (int it = tid; it < rows * (HALF / 8); it += NT) {
      const int r = it / (HALF / 8), c0 = (it % (HALF / 8)) * 8;
      const int m = m_base + r;
      if (m >= M) continue;
      const float* src = sC + (int64_t)r * ldc;
      const float2* cs = e.rope + (int64_t)e.pos[m] * HALF + c0;
      const float inv = gain != nullptr ? src[D] : 1.0f;
      float lo[8], hi[8], ba[8], bb[8], ga[8], gb[8];
      if (bias) {
        ld8(bias + rbase + c0, ba);
        ld8(bias + rbase + c0 + HALF, bb);
      }
      if (gain != nullptr) {
        ld8(gain + c0, ga);
        ld8(gain + c0 + HALF, gb);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float a = src[c0 + i], b = src[c0 + HALF + i];
        if (bias) {
          a += ba[i];
          b += bb[i];
        }
        if (gain != nullptr) {
          a = a * inv * ga[i];
          b = b * inv * gb[i];
        }
        const float2 t = cs[i];
        lo[i] = a * t.x - b * t.y;
        hi[i] = b * t.x + a * t.y;
      }
      bf16_t* dst = region == 0
                        ? reinterpret_cast<bf16_t*>(e.q_out) + (int64_t)m * qcols + rbase
                        : reinterpret_cast<bf16_t*>(e.arena_k) + e.slot[m] * (int64_t)kcols + rbase;
      store8(dst + c0, lo);
      store8(dst + c0 + HALF, hi);
    }
  } else {
    for (int it = tid; it < rows * (D / 8); it += NT) {
      const int r = it / (D / 8), c0 = (it % (D / 8)) * 8;
      const int m = m_base + r;
      if (m >= M) continue;
      const float* src = sC + (int64_t)r * ldc + c0;
      float v[8], bv[8];
      if (bias) ld8(bias + rbase + c0, bv);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = bias ? src[i] + bv[i] : src[i];
      store8(reinterpret_cast<bf16_t*>(e.arena_v) + e.slot[m] * (int64_t)kcols + rbase + c0, v);
    }
  }
}

// SWIGLU: tile columns [0, BN/2) are gate rows j0.., [BN/2, BN) the same up rows.
template <int BN, int NT>
__device__ __forceinline__ void epi_swiglu(const float* sC, int ldc, int rows, int m_base, int M, int j0,
                                           const EpiParams& e) {
  const int tid = threadIdx.x;
  constexpr int HB = BN / 2;
  const int per_row = HB / 8;
#pragma unroll 4
  for (int it = tid; it < rows * per_row; it += NT) {
    const int r = it / per_row, c0 = (it % per_row) * 8;
    const int m = m_base + r;
    if (m >= M) continue;
    const float* src = sC + (int64_t)r * ldc + c0;
    float h[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = silu(src[i]) * src[HB + i];
    store8(reinterpret_cast<bf16_t*>(e.hf) + (int64_t)m * e.ldh + j0 + c0, h);
  }
}

}  // namespace kvr
