// Epilogues of the bf16 matrix-core products, straight from the accumulators.
//
// The products run v_mfma_f32_16x16x32_bf16 with the weight rows as the first
// operand, so a lane holds four consecutive output columns of one row: frag
// (i, j) of a wave is the 16 x 16 piece at rows row(i) .. +15, columns col(j)
// .. +15, of which lane l has row row(i) + l%16 and columns col(j) + 4*(l/16)
// .. +3.  Every load and store is then 16 bytes (fp32) or 8 bytes (bf16) per
// lane with four lanes per row segment, no LDS round trip and no barrier.
//
// Columns are taken in an order that puts what an epilogue combines into the
// same lane (perm_row): a QKV tile's 32-column groups hold rotary pairs, dims
// 16w .. 16w+15 of a head and dims 64+16w .. +15; a gate/up tile's hold 16
// gate rows and the same 16 up rows.  Frags 2x and 2x+1 are such a pair.
//
// Loads and stores share one wait counter on this GPU, and once a store is
// pending every wait for a load is a wait for all: each routine loads a batch
// of rows, forms the results, and only then stores.
#pragma once
#include "common.h"
#include "launch.h"

namespace kvr {

// Weight row (within its 128-row head, or its gate/up matrix) of a column in
// the order of the pairs above; c counts from the head's (the tile's) start.
__device__ __forceinline__ int qkv_perm_row(int c) {
  const int h = c & 127;
  return (c & ~127) + ((h >> 4) & 1) * 64 + (h >> 5) * 16 + (h & 15);
}
__device__ __forceinline__ int gateup_perm_row(int c) { return (c >> 5) * 16 + (c & 15); }

__device__ __forceinline__ uint2 pack4(const float* v) {
  uint2 u;
  u.x = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
  u.y = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
  return u;
}
__device__ __forceinline__ void unpack4(uint2 u, float* v) {
  v[0] = __uint_as_float(u.x << 16);
  v[1] = __uint_as_float(u.x & 0xffff0000u);
  v[2] = __uint_as_float(u.y << 16);
  v[3] = __uint_as_float(u.y & 0xffff0000u);
}

// Exchange of two registers between lane groups of 16: odd groups of a with even
// groups of b, and the upper two groups of a with the lower two of b.
__device__ __forceinline__ void swap_rows16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// RESID: X += acc (fp32).  GI row frags are loaded, summed and stored at a
// time; X is touched once per product, so it goes past the caches' reuse.
template <int RI, int CJ, int GI, typename Row, typename Col>
__device__ __forceinline__ void acc_resid(const f32x4 (&acc)[RI][CJ], int M, const EpiParams& e, Row row,
                                          Col col) {
#pragma unroll
  for (int i0 = 0; i0 < RI; i0 += GI) {
    f32x4 xv[GI][CJ];
#pragma unroll
    for (int i = 0; i < GI; ++i) {
      const float* xr = e.x + (int64_t)min(row(i0 + i), M - 1) * e.ldx;
#pragma unroll
      for (int j = 0; j < CJ; ++j)
        xv[i][j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(xr + col(j)));
    }
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        xv[i][j].x += acc[i0 + i][j].x;
        xv[i][j].y += acc[i0 + i][j].y;
        xv[i][j].z += acc[i0 + i][j].z;
        xv[i][j].w += acc[i0 + i][j].w;
        asm volatile("" : "+v"(xv[i][j]));  // the sum is formed here, before any store
      }
#pragma unroll
    for (int i = 0; i < GI; ++i)
      if (row(i0 + i) < M) {
        float* xr = e.x + (int64_t)row(i0 + i) * e.ldx;
#pragma unroll
        for (int j = 0; j < CJ; ++j) __builtin_nontemporal_store(xv[i][j], reinterpret_cast<f32x4*>(xr + col(j)));
      }
  }
}

// STORE: out = acc (fp32), out on any 4-byte boundary (a caller's logits).
template <int RI, int CJ, typename Row, typename Col>
__device__ __forceinline__ void acc_store(const f32x4 (&acc)[RI][CJ], int M, float* out, int64_t ld, Row row,
                                          Col col) {
#pragma unroll
  for (int i = 0; i < RI; ++i)
    if (row(i) < M)
#pragma unroll
      for (int j = 0; j < CJ; ++j) *reinterpret_cast<f32x4_a4*>(out + row(i) * ld + col(j)) = acc[i][j];
}

// SWIGLU: hf = silu(gate) * up; col(j) counts gate/up columns in pair order,
// output column = 16 * (col / 32) + col % 16.
template <int RI, int CJ, typename Row, typename Col>
__device__ __forceinline__ void acc_swiglu(const f32x4 (&acc)[RI][CJ], int M, const EpiParams& e, Row row,
                                           Col col) {
#pragma clang fp contract(off)
#pragma unroll
  for (int i = 0; i < RI; ++i)
    if (row(i) < M) {
      bf16_t* hr = reinterpret_cast<bf16_t*>(e.hf) + (int64_t)row(i) * e.ldh;
#pragma unroll
      for (int x = 0; x < CJ / 2; ++x) {
        float h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = silu(acc[i][2 * x][k]) * acc[i][2 * x + 1][k];
        *reinterpret_cast<uint2*>(hr + gateup_perm_row(col(2 * x))) = pack4(h);
      }
    }
}

// QKV: bias, per-head q/k RMSNorm, NeoX RoPE, rounding, then Q rows to the
// workspace, K and V rows to their arena slots, the K copy and V^T.  n0: the
// tile's first column (q columns, then k, then v); the tile lies in one of the
// three regions and starts on a multiple of 32.  smem: the workgroup's LDS
// (free after the product).  WR: rows of a wave that are consecutive (frags
// G*WR/16 .. +WR/16-1 for G = 0, 1, ..).  Head dim 128.  NORM: the model has
// the per-head norms (the tile then holds whole heads); a kernel of its own, as
// one that decides at run time spills a hundred registers in the 256 x 256 tile.
// A head's sum of squares is formed in one fixed order whatever the tile: FMAs
// over 16 dims in index order, then the head's eight such parts pairwise (the
// order of the split-K epilogue, epilogue.h).
template <bool NORM, int RI, int CJ, int BM, int BN, int WAVES, int WR, typename Row, typename Col>
__device__ __forceinline__ void acc_qkv(f32x4 (&acc)[RI][CJ], int m0, int M, int n0, const EpiParams& e,
                                        char* smem, int wave, int lane, Row row, Col col) {
  // every tile's instance has to round alike, so no product is contracted into
  // an FMA but those written as one
#pragma clang fp contract(off)
  constexpr int D = 128, HALF = 64;
  const int qcols = e.nq * D, kcols = e.nkv * D;
  const int region = n0 < qcols ? 0 : (n0 < qcols + kcols ? 1 : 2);
  const int rbase = region == 0 ? 0 : region == 1 ? qcols : qcols + kcols;  // region's first column
  const int fq = lane >> 4;
  // pair x: head hd[x] of the region, dims d0[x] .. +3 and +64 .. +67
  int hd[CJ / 2], d0[CJ / 2];
#pragma unroll
  for (int x = 0; x < CJ / 2; ++x) {
    const int c = n0 + col(2 * x) - 4 * fq - rbase;
    hd[x] = c >> 7;
    d0[x] = ((c & 127) >> 5) * 16 + 4 * fq;
  }
  const bf16_t* bias = reinterpret_cast<const bf16_t*>(region == 0 ? e.bq : region == 1 ? e.bk : e.bv);
  if (bias != nullptr) {
#pragma unroll
    for (int x = 0; x < CJ / 2; ++x)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        float b[4];
        unpack4(*reinterpret_cast<const uint2*>(bias + hd[x] * D + d0[x] + s * HALF), b);
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[i][2 * x + s][k] += b[k];
      }
  }
  // slots and key rows of this lane's rows (padding rows: slot -1)
  int64_t sl[RI];
  int kr[RI];
  if (region != 0) {
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const int m = min(row(i), M - 1);
      sl[i] = row(i) < M ? e.slot[m] : -1;
      kr[i] = e.krow != nullptr ? e.krow[m] : m;
    }
  }
  if (region == 2) {
    __syncthreads();  // every wave is done with the operand ring
    // arena rows first (they need no exchange), then V^T through a per-wave
    // LDS area [dims][rows]: 8 consecutive rows of one dim per 16-byte store
    constexpr int PITCH = WR + 8, DIMS = CJ * 16, GF = WR / 16;
    uint16_t* sv = reinterpret_cast<uint16_t*>(smem) + wave * DIMS * PITCH;
#pragma unroll
    for (int g = 0; g < RI / GF; ++g) {
      if (e.vt != nullptr) {
#pragma unroll
        for (int i = 0; i < GF; ++i)
#pragma unroll
          for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k)
              sv[(j * 16 + 4 * fq + k) * PITCH + i * 16 + (lane & 15)] =
                  sl[g * GF + i] < 0 ? 0 : f2bf(acc[g * GF + i][j][k]);
        // a wave's own area, and its LDS accesses run in order: only the
        // compiler has to keep the writes before the reads
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
#pragma unroll
      for (int i = 0; i < GF; ++i) {
        const int64_t s = sl[g * GF + i];
        if (s >= 0) {
          bf16_t* dst = reinterpret_cast<bf16_t*>(e.arena_v) + s * (int64_t)kcols;
#pragma unroll
          for (int x = 0; x < CJ / 2; ++x)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              float v[4];
#pragma unroll
              for (int k = 0; k < 4; ++k) v[k] = acc[g * GF + i][2 * x + h][k];
              *reinterpret_cast<uint2*>(dst + hd[x] * D + d0[x] + h * HALF) = pack4(v);
            }
        }
      }
      if (e.vt != nullptr) {
        // first row of the group (uniform over the wave)
        const int gm = row(g * GF) - (lane & 15);
        constexpr int OCT = WR / 8;
#pragma unroll
        for (int it = 0; it < DIMS * OCT / 64; ++it) {
          const int idx = it * 64 + lane, o = idx % OCT, c = idx / OCT;
          const int m = gm + o * 8;
          const uint4 v = *reinterpret_cast<const uint4*>(sv + c * PITCH + o * 8);
          if (m < M) {
            const int cc = n0 + col((c >> 4)) - 4 * fq + (c & 15) - rbase;
            const int64_t k0 = e.krow != nullptr ? e.krow[m] : m;
            *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(e.vt) +
                                      vt_offset(qkv_perm_row(cc), k0, e.ldvt, D)) = v;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    return;
  }
  // positions, then the RoPE rows of every frag, before any store
  int pos[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) pos[i] = e.pos[min(row(i), M - 1)];
  if constexpr (NORM) {
    const bf16_t* gain = reinterpret_cast<const bf16_t*>(region == 0 ? e.q_norm : e.k_norm);
    // sum of squares of (row, head): eight 16-dim parts, each one chain of FMAs
    // over its dims in index order, to LDS.  A part's dims lie four to a lane:
    // the four lanes of a row exchange frags, so that each has one part's whole.
    float* red = reinterpret_cast<float*>(smem);  // [row][head of the tile][8 parts]
    constexpr int HT = BN / D < 1 ? 1 : BN / D;
    __syncthreads();
    static_assert(CJ == 4, "four frags for the four lanes of a row");
    const int pc = n0 + col(fq) - 4 * fq - rbase;  // frag fq's first column in the region
    const int part = ((pc >> 7) - ((n0 - rbase) >> 7)) * 8 + ((pc >> 4) & 1) * 4 + ((pc & 127) >> 5);
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      float t[4][4];  // [frag][dim], after the exchanges [lane of the row][dim]
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j][k] = acc[i][j][k];
        swap_rows16(t[0][k], t[1][k]);
        swap_rows16(t[2][k], t[3][k]);
        swap_rows32(t[0][k], t[2][k]);
        swap_rows32(t[1][k], t[3][k]);
      }
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) s = fmaf(t[q][k], t[q][k], s);
      red[(row(i) - m0) * HT * 8 + part] = s;
    }
    __syncthreads();
    // one inverse RMS per (row, head), in place of its first part
    for (int t = wave * 64 + lane; t < BM * HT; t += WAVES * 64) {
      const f32x4 u = *reinterpret_cast<const f32x4*>(red + t * 8), v = *reinterpret_cast<const f32x4*>(red + t * 8 + 4);
      const float ss = ((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w));
      red[t * 8] = 1.0f / sqrtf(ss / (float)D + e.eps);
    }
    __syncthreads();
    float ga[CJ / 2][2][4];
#pragma unroll
    for (int x = 0; x < CJ / 2; ++x) {
      unpack4(*reinterpret_cast<const uint2*>(gain + d0[x]), ga[x][0]);
      unpack4(*reinterpret_cast<const uint2*>(gain + d0[x] + HALF), ga[x][1]);
    }
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int x = 0; x < CJ / 2; ++x) {
        const float inv = red[((row(i) - m0) * HT + (hd[x] - ((n0 - rbase) >> 7))) * 8];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[i][2 * x + h][k] = acc[i][2 * x + h][k] * inv * ga[x][h][k];
      }
  }
  // rotate in place, a few rows' cos/sin at a time (they are all loads, so
  // nothing waits for a store); the pairs of one lane share them where they
  // are the same dims of different heads
  constexpr bool SAME_DIMS = BN == 256;
  constexpr int GR = RI < 4 ? RI : 4;
#pragma unroll
  for (int i0 = 0; i0 < RI; i0 += GR) {
    float4 cs[GR][SAME_DIMS ? 1 : CJ / 2][2];
#pragma unroll
    for (int i = 0; i < GR; ++i)
#pragma unroll
      for (int x = 0; x < (SAME_DIMS ? 1 : CJ / 2); ++x) {
        const float4* src = reinterpret_cast<const float4*>(e.rope + (int64_t)pos[i0 + i] * HALF + d0[x]);
        cs[i][x][0] = src[0];
        cs[i][x][1] = src[1];
      }
#pragma unroll
    for (int i = 0; i < GR; ++i)
#pragma unroll
      for (int x = 0; x < CJ / 2; ++x) {
        const float4 c0 = cs[i][SAME_DIMS ? 0 : x][0], c1 = cs[i][SAME_DIMS ? 0 : x][1];
        const float cc[4] = {c0.x, c0.z, c1.x, c1.z}, ss[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float a = acc[i0 + i][2 * x][k], b = acc[i0 + i][2 * x + 1][k];
          acc[i0 + i][2 * x][k] = fmaf(a, cc[k], -(b * ss[k]));
          acc[i0 + i][2 * x + 1][k] = fmaf(a, ss[k], b * cc[k]);
        }
      }
  }
#pragma unroll
  for (int i = 0; i < RI; ++i)
#pragma unroll
    for (int x = 0; x < CJ / 2; ++x) {
      float lo[4], hi[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lo[k] = acc[i][2 * x][k];
        hi[k] = acc[i][2 * x + 1][k];
      }
      uint2 ul = pack4(lo), uh = pack4(hi);
      if (region == 0) {
        if (row(i) < M) {
          bf16_t* dst = reinterpret_cast<bf16_t*>(e.q_out) + (int64_t)row(i) * qcols + hd[x] * D + d0[x];
          *reinterpret_cast<uint2*>(dst) = ul;
          *reinterpret_cast<uint2*>(dst + HALF) = uh;
        }
      } else {
        if (sl[i] >= 0) {
          bf16_t* dst = reinterpret_cast<bf16_t*>(e.arena_k) + (sl[i] * e.nkv + hd[x]) * (int64_t)D + d0[x];
          *reinterpret_cast<uint2*>(dst) = ul;
          *reinterpret_cast<uint2*>(dst + HALF) = uh;
        } else {
          // padding rows: zeros in the K copy (keys past a request's end are
          // inert), nothing in the arena
          ul = uh = make_uint2(0u, 0u);
        }
        if (e.kc != nullptr && row(i) < M) {
          bf16_t* kd = reinterpret_cast<bf16_t*>(e.kc) + ((int64_t)hd[x] * e.ldvt + kr[i]) * D + d0[x];
          *reinterpret_cast<uint2*>(kd) = ul;
          *reinterpret_cast<uint2*>(kd + HALF) = uh;
        }
      }
    }
}

}  // namespace kvr
