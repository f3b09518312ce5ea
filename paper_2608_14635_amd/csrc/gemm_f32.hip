// fp32 GEMM C[M, N] = A[M, K] . B[N, K]^T for fp32 models on the fp32 matrix
// cores (v_mfma_f32_16x16x4_f32, fp32 products and sums), with the rebuild's
// epilogues taken from the accumulators.  Ragged M, N (FFN widths that are not
// tile multiples, decode batches as columns) and K (a multiple of 8) are handled.
//
// The structure is that of the bf16 tiles (gemm_tile.hip): K tiles of 128 bytes
// a row (32 k) stream with buffer_load_dwordx4 ... lds into a ring of STAGES,
// fragments are read one K tile ahead, one barrier per K tile.  A lane's
// 16-byte fragment holds four consecutive k of one row; MFMA t of four takes
// element t, so a group of 16 k is summed in the order t, 4+t, 8+t, 12+t for
// t = 0..3 whatever the tile.  The last K % 32 values are loaded straight from
// memory.
//
// The tiny fp32 decoder's products (384 rows, K 256) are latency-bound: 32 x 32
// tiles give 96 to 528 workgroups and take 7-10 us each, where 64 x 128 tiles of
// scalar loads and vector FMAs took 50-90 us.  Larger batches are bound by the
// fp32 matrix cores (64 x 64 tiles).
// Every output is produced by one workgroup in one K order: results do not
// depend on the other rows of a call.
// Weights, biases, gains and the arena come from the caller on any 4-byte boundary.
#include "common.h"
#include "dma.h"
#include "launch.h"

namespace kvr {

namespace {

constexpr int BK = 32;  // floats: 128 bytes

// Weight row (within its head) of a column: 32-column groups of 16 dims and
// their rotary partners, so that a lane holds both (head dim 32 and up; at 16
// a 16-column piece is one head and the partner is two lane groups away)
__device__ __forceinline__ int head_row(int c, int d) {
  if (d == 16) return c;
  return ((c >> 4) & 1) * (d >> 1) + (c >> 5) * 16 + (c & 15);
}

// Row of weights behind column c of the tile at columns n0.. (clamped to a
// valid one where the tile overhangs; those results are dropped)
template <int EPI>
__device__ __forceinline__ const float* b_row(const GemmParams& p, int n0, int c) {
  const int64_t ldb = p.ldb ? p.ldb : p.K;
  if (EPI == EPI_SWIGLU) {
    const int n = n0 + c;  // 16 gate columns, then the same 16 up columns
    const int j = min((n >> 5) * 16 + (n & 15), p.epi.ffn - 1);
    return reinterpret_cast<const float*>((n >> 4) & 1 ? p.B1 : p.B0) + j * ldb;
  }
  if (EPI == EPI_QKV) {
    const int n = n0 + c, d = p.epi.d;
    const int reg = n < p.s0 ? 0 : n < p.s1 ? p.s0 : p.s1;
    const void* m = n < p.s0 ? p.B0 : n < p.s1 ? p.B1 : p.B2;
    const int h = (n - reg) / d * d;
    return reinterpret_cast<const float*>(m) + (int64_t)(h + head_row(n - reg - h, d)) * ldb;
  }
  return reinterpret_cast<const float*>(p.B0) + (int64_t)min(n0 + c, p.n_end - 1) * ldb;
}

// Bias, per-head q/k RMSNorm and RoPE of a tile within one region, then Q rows
// to the workspace, K and V rows to their arena slots.  With the norms a wave's
// columns are whole heads (128 columns a wave).
template <int RI, int CJ, typename Row, typename Col>
__device__ __forceinline__ void qkv_f32(f32x4 (&acc)[RI][CJ], int M, int n0, const EpiParams& e, int lane, Row row,
                                        Col col) {
  // every tile's instance has to round alike, so no product is contracted into
  // an FMA but those written as one
#pragma clang fp contract(off)
  const int d = e.d, half = d >> 1, fq = lane >> 4;
  const int qcols = e.nq * d, kcols = e.nkv * d;
  const int region = n0 < qcols ? 0 : (n0 < qcols + kcols ? 1 : 2);
  const int rbase = region == 0 ? 0 : region == 1 ? qcols : qcols + kcols;
  // piece j: this lane's four dims start at dim[j] of head hd[j]
  int hd[CJ], dim[CJ];
#pragma unroll
  for (int j = 0; j < CJ; ++j) {
    const int c = n0 + col(j) - 4 * fq - rbase;
    hd[j] = c / d;
    dim[j] = head_row(c % d, d) + 4 * fq;
  }
  const float* bias = reinterpret_cast<const float*>(region == 0 ? e.bq : region == 1 ? e.bk : e.bv);
  if (bias != nullptr) {
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      const f32x4 b = *reinterpret_cast<const f32x4_a4*>(bias + hd[j] * d + dim[j]);
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[i][j][k] += b[k];
    }
  }
  if (region < 2) {
    const float* gain = reinterpret_cast<const float*>(region == 0 ? e.q_norm : e.k_norm);
    if constexpr (CJ == 8) {
      if (gain != nullptr) {
        const int per = d >> 4;  // pieces of a head
#pragma unroll
        for (int i = 0; i < RI; ++i) {
          float ss[CJ];
#pragma unroll
          for (int j = 0; j < CJ; ++j) {
            const f32x4 a = acc[i][j];
            ss[j] = fmaf(a.x, a.x, a.y * a.y) + fmaf(a.z, a.z, a.w * a.w);
            ss[j] += __shfl_xor(ss[j], 16, 64);
            ss[j] += __shfl_xor(ss[j], 32, 64);
          }
          // the head's pieces pairwise
          if (per >= 2)
#pragma unroll
            for (int j = 0; j < CJ; j += 2) ss[j] = ss[j + 1] = ss[j] + ss[j + 1];
          if (per >= 4)
#pragma unroll
            for (int j = 0; j < CJ; j += 4) ss[j] = ss[j + 1] = ss[j + 2] = ss[j + 3] = ss[j] + ss[j + 2];
          if (per >= 8) {
            const float t = ss[0] + ss[4];
#pragma unroll
            for (int j = 0; j < CJ; ++j) ss[j] = t;
          }
#pragma unroll
          for (int j = 0; j < CJ; ++j) {
            const float inv = 1.0f / sqrtf(ss[j] / (float)d + e.eps);
            const f32x4 g = *reinterpret_cast<const f32x4_a4*>(gain + dim[j]);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[i][j][k] = acc[i][j][k] * inv * g[k];
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const float2* tab = e.rope + (int64_t)e.pos[min(row(i), M - 1)] * half;
      if (d == 16) {
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float2 t = tab[(dim[j] + k) & 7];
            const float own = acc[i][j][k], other = __shfl_xor(own, 32, 64);
            acc[i][j][k] = fq < 2 ? fmaf(own, t.x, -(other * t.y)) : fmaf(own, t.x, other * t.y);
          }
      } else if constexpr (CJ >= 2) {
#pragma unroll
        for (int x = 0; x < CJ; x += 2)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float2 t = tab[dim[x] + k];
            const float a = acc[i][x][k], b = acc[i][x + 1][k];
            acc[i][x][k] = fmaf(a, t.x, -(b * t.y));
            acc[i][x + 1][k] = fmaf(b, t.x, a * t.y);
          }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    if (row(i) >= M) continue;
    float* dst;
    if (region == 0) {
      dst = reinterpret_cast<float*>(e.q_out) + (int64_t)row(i) * qcols;
    } else {
      const int64_t sl = e.slot[row(i)];
      if (sl < 0) continue;  // padding row
      dst = reinterpret_cast<float*>(region == 1 ? e.arena_k : e.arena_v) + sl * kcols;
    }
#pragma unroll
    for (int j = 0; j < CJ; ++j) *reinterpret_cast<f32x4_a4*>(dst + hd[j] * d + dim[j]) = acc[i][j];
  }
}

template <int BM, int BN, int WM, int WN, int STAGES, int EPI>
__global__ __launch_bounds__(64 * WM * WN) void gemm_f32_kernel(GemmParams p, int tiles_n) {
  constexpr int WAVES = WM * WN, WR = BM / WM, WC = BN / WN, RI = WR / 16, CJ = WC / 16;
  constexpr int STAGE = (BM + BN) * BK * 4;
  constexpr int LA = BM / 8 / WAVES, LB = BN / 8 / WAVES, LPW = LA + LB;  // loads per wave and stage
  static_assert(LA >= 1 && LB >= 1, "tile shape");
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE];
  const int tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x % tiles_n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = tile_m * BM, n0 = p.n_begin + tile_n * BN;

  // direct-to-LDS loaders: wave w fills blocks w, w + WAVES, ... of 8 rows.  A
  // block's eight weight rows are consecutive but for the clamp of a tile that
  // overhangs, so each lane keeps its offset from the block's first row.
  const float* A = reinterpret_cast<const float*>(p.A) + (int64_t)m0 * p.lda;
  const int rows_a = min(BM, p.M - m0);
  const int a_bytes = (int)(rows_a * p.lda * 4);
  const int64_t ldb = p.ldb ? p.ldb : p.K;
  const int lrow = lane >> 3, unit = (lane & 7) ^ swz((wave & 1) * 8 + lrow);
  int a_voff[LA], b_voff[LB];
  const float* b_base[LB];
#pragma unroll
  for (int q = 0; q < LA; ++q) {
    // rows past M are clamped to the last one, their results dropped
    const int r = min((wave + WAVES * q) * 8 + lrow, rows_a - 1);
    a_voff[q] = (int)(r * p.lda * 4) + unit * 16;
  }
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const int r = (wave + WAVES * q) * 8;
    b_base[q] = b_row<EPI>(p, n0, r);
    b_voff[q] = (int)((b_row<EPI>(p, n0, r + lrow) - b_base[q]) * 4) + unit * 16;
  }
  const int KT = p.K / BK;
  // past the end the last K tile is fetched again, into a stage nobody reads
  auto issue = [&](int kt) {
    char* st = smem + (kt % STAGES) * STAGE;
    const int kb = min(kt, KT - 1) * BK * 4;
#pragma unroll
    for (int q = 0; q < LA; ++q) load_lds(A, a_bytes, st + (wave + WAVES * q) * 1024, a_voff[q], kb);
#pragma unroll
    for (int q = 0; q < LB; ++q)
      load_lds(b_base[q], (int)(8 * ldb * 4), st + BM * BK * 4 + (wave + WAVES * q) * 1024, b_voff[q], kb);
  };
  if (KT > 0)
#pragma unroll
    for (int s = 0; s < STAGES; ++s) issue(s);

  f32x4 acc[RI][CJ];
#pragma unroll
  for (int i = 0; i < RI; ++i)
#pragma unroll
    for (int j = 0; j < CJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int fr = lane & 15, fq = lane >> 4;
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int u = ((ks * 4 + fq) ^ swz(fr)) << 4;
    a_off[ks] = (wm * WR + fr) * (BK * 4) + u;
    b_off[ks] = BM * BK * 4 + (wn * WC + fr) * (BK * 4) + u;
  }
  f32x4 af[2][2][RI], bf[2][2][CJ];  // [K tile parity][16-k group][piece]
  auto read = [&](int kt, int par) {
    const char* st = smem + (kt % STAGES) * STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int j = 0; j < CJ; ++j) bf[par][ks][j] = *reinterpret_cast<const f32x4*>(st + b_off[ks] + j * 2048);
#pragma unroll
      for (int i = 0; i < RI; ++i) af[par][ks][i] = *reinterpret_cast<const f32x4*>(st + a_off[ks] + i * 2048);
    }
  };
  auto multiply = [&](const f32x4 (&a)[RI], const f32x4 (&b)[CJ]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][t], a[i][t], acc[i][j], 0, 0, 0);
  };
  // as gemm_tile.hip: this wave's fragments of K tile kt are in registers and
  // its loads of K tile kt+1 have landed; the barrier makes both true of all
  auto step = [&](int kt, int par) {
    __builtin_amdgcn_sched_barrier(0);
    KVR_WAIT_LGKM0();
    KVR_WAIT_VMCNT((STAGES - 2) * LPW);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(kt + 1, par ^ 1);
    issue(kt + STAGES);
    multiply(af[par][0], bf[par][0]);
    multiply(af[par][1], bf[par][1]);
  };
  KVR_WAIT_VMCNT((STAGES - 1) * LPW);
  __builtin_amdgcn_s_barrier();
  read(0, 0);
  int kt = 0;
  for (; kt + 1 < KT; kt += 2) {
    step(kt, 0);
    step(kt + 1, 1);
  }
  if (kt < KT) step(kt, 0);
  KVR_WAIT_LGKM0();
  KVR_WAIT_VMCNT(0);  // trailing refetches land before the LDS is given back

  auto row = [&](int i) { return m0 + wm * WR + i * 16 + fr; };
  auto col = [&](int j) { return wn * WC + j * 16 + 4 * fq; };
  // the last K % 32 (a multiple of 8): units of four k, all inside or all outside
  if (KT * BK < p.K) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int k = KT * BK + (ks * 4 + fq) * 4;
      f32x4 a[RI], b[CJ];
#pragma unroll
      for (int i = 0; i < RI; ++i) {
        a[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (k < p.K) a[i] = *reinterpret_cast<const f32x4_a4*>(A + (int64_t)min(row(i) - m0, rows_a - 1) * p.lda + k);
      }
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        b[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (k < p.K) b[j] = *reinterpret_cast<const f32x4_a4*>(b_row<EPI>(p, n0, wn * WC + j * 16 + fr) + k);
      }
      multiply(a, b);
    }
  }

  if constexpr (EPI == EPI_QKV) {
    qkv_f32<RI, CJ>(acc, p.M, n0, p.epi, lane, row, col);
  } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int x = 0; x + 1 < CJ; x += 2) {
        const int n = n0 + col(x), o = (n >> 5) * 16 + (n & 15);
        f32x4 h;
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = silu(acc[i][x][k]) * acc[i][x + 1][k];
        if (row(i) < p.M && o < p.epi.ffn)
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.epi.hf) + (int64_t)row(i) * p.epi.ldh + o) = h;
      }
  } else {
    f32x4 xv[RI][CJ];
    if constexpr (EPI == EPI_RESID) {  // loads before any store: they share one wait counter
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
          xv[i][j] = *reinterpret_cast<const f32x4*>(p.epi.x + (int64_t)min(row(i), p.M - 1) * p.epi.ldx + n0 + col(j));
          xv[i][j] += acc[i][j];
        }
    }
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      if (row(i) >= p.M) continue;
      float* xr = p.epi.x + (int64_t)row(i) * p.epi.ldx;
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        if constexpr (EPI == EPI_RESID) {
          *reinterpret_cast<f32x4*>(xr + n0 + col(j)) = xv[i][j];
        } else {  // STORE: columns may end inside a piece
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (n0 + col(j) + k < p.n_end) xr[n0 + col(j) + k] = acc[i][j][k];
        }
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int STAGES, int EPI>
void launch_tile(const GemmParams& p, int N, hipStream_t s) {
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, WM, WN, STAGES, EPI>), dim3(tiles_m * tiles_n), dim3(64 * WM * WN), 0,
                     s, p, tiles_n);
}

// 32 x 32 tiles of two waves until 64 x 64 ones would give every CU two
// (a K tile of the larger one costs 1024 clocks of matrix core, of the small one 256)
template <int EPI>
void launch_sized(const GemmParams& p, int N, hipStream_t s) {
  const int64_t big = (int64_t)((p.M + 63) / 64) * ((N + 63) / 64);
  if (big >= 512)
    launch_tile<64, 64, 2, 2, 4, EPI>(p, N, s);
  else
    launch_tile<32, 32, 2, 1, 6, EPI>(p, N, s);
}

}  // namespace

void launch_gemm_f32(int epi, const GemmParams& p, hipStream_t s) {
  // gate/up columns: 16 and 16 at a time
  const int N = p.bmap == BMAP_GATEUP ? 2 * ((p.epi.ffn + 15) / 16 * 16) : p.n_end - p.n_begin;
  if (p.M <= 0 || N <= 0) return;
  if (epi == EPI_QKV && p.epi.q_norm != nullptr)
    launch_tile<64, 128, 4, 1, 3, EPI_QKV>(p, N, s);  // a wave's columns hold whole heads
  else if (epi == EPI_QKV)
    launch_sized<EPI_QKV>(p, N, s);
  else if (epi == EPI_RESID)
    launch_sized<EPI_RESID>(p, N, s);
  else if (epi == EPI_STORE)
    launch_sized<EPI_STORE>(p, N, s);
  else
    launch_sized<EPI_SWIGLU>(p, N, s);
}

}  // namespace kvr
