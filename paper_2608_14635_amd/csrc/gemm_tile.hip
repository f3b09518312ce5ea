// bf16 GEMM C[M, N] = A[M, K] . B[N, K]^T on gfx950 matrix cores for products
// whose 256 x 256 tiles would leave most of the 256 CUs idle (short requests,
// wide decode batches), in smaller tiles with the same epilogues (gemm_epi.h),
// and the choice of the tile for every bf16 product.
//
// What bounds these products is each CU's operand stream, not its matrix core:
// however much a workgroup has issued, about 32 KB of loads are outstanding per
// CU, and while weights come from HBM with 0.7 us latency that is at most 47 GB/s
// a CU, A's rows from L2 included, whatever the tile or the depth of the ring
// (twice the stages gave nothing).  (HBM itself gives 256 CUs 25 GB/s each: the
// rest of a CU's stream is A and the weights that its neighbours already fetched.)
// A K tile of (BM + BN) x 64 therefore takes about (BM + BN) * 128 B / 47 GB/s,
// and a product takes that times its K tiles times the rounds of workgroups over
// the CUs (tile_cost below).
//
// One workgroup of WM x WN waves; K tiles stream with buffer_load_dwordx4 ...
// lds into a ring of STAGES; fragments are read one K tile ahead of their
// MFMAs, so one barrier per K tile covers both the hand-over of the next stage
// and the refill of this one.  v_mfma_f32_16x16x32_bf16 with k ascending, as
// the 256 x 256 kernel: a row's result is the same bits whatever the tile.
//
// Measured (weights from HBM, 4096 -> 4096 columns, us): 64 rows 69 -> 12.6
// with 32 x 32 tiles, 192 rows 78 -> 21 (64 x 64), 512 rows 85 -> 30 (128 x 64),
// 1024 rows 88 -> 44 (128 x 128), 2048 rows 90 -> 74 (256 x 128).
#include <algorithm>

#include "common.h"
#include "dma.h"
#include "gemm_epi.h"
#include "launch.h"

namespace kvr {

namespace {

constexpr int BK = 64;

template <int BM, int BN, int WM, int WN, int STAGES, int EPI, bool NORM = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_tile_kernel(GemmParams p, int tiles_m, int tiles_n) {
  constexpr int WAVES = WM * WN, WR = BM / WM, WC = BN / WN;  // rows and columns of a wave
  constexpr int RI = WR / 16, CJ = WC / 16;
  constexpr int STAGE = (BM + BN) * BK * 2;
  constexpr int LA = BM / 8 / WAVES, LB = BN / 8 / WAVES, LPW = LA + LB;  // loads per wave and stage
  static_assert(LA >= 1 && LB >= 1 && CJ >= 2 && CJ % 2 == 0, "tile shape");
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE];

  const int ksplit = EPI == EPI_PARTIAL ? p.ksplit : 1;
  const int split = EPI == EPI_PARTIAL ? (int)(blockIdx.x % ksplit) : 0;
  // ---- tile coordinates: XCD-contiguous ranges, grouped along M ----
  const int num_tiles = tiles_m * tiles_n;
  int t = EPI == EPI_PARTIAL ? (int)(blockIdx.x / ksplit) : (int)blockIdx.x;
  const int full = (num_tiles / 8) * 8;
  if (t < full) t = (t % 8) * (num_tiles / 8) + t / 8;
  const int gm = p.group_m;
  const int group = t / (gm * tiles_n);
  const int first_m = group * gm;
  const int gsz = min(tiles_m - first_m, gm);
  const int tile_m = first_m + (t % (gm * tiles_n)) % gsz;
  const int tile_n = (t % (gm * tiles_n)) / gsz;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = tile_m * BM, n0 = p.n_begin + tile_n * BN;

  // ---- direct-to-LDS loaders: wave w fills blocks w, w + 4, ... of 8 rows ----
  const void *a_base, *b_base[LB];
  int a_bytes, b_bytes, a_voff[LA], b_voff[LB];
  {
    const int lrow = lane >> 3;
    const int unit = (lane & 7) ^ swz((wave & 1) * 8 + lrow);
    const int rows_a = min(BM, p.M - m0);
    a_base = reinterpret_cast<const bf16_t*>(p.A) + (int64_t)m0 * p.lda;
    a_bytes = (int)(rows_a * p.lda * 2);
    const int64_t ldb = p.ldb ? p.ldb : p.K;
    const void* mat = p.B0;
    int64_t brow = n0;
    int c0 = 0;          // tile's first column within its head (QKV)
    int b_rows = BN;
    if (EPI == EPI_QKV) {
      c0 = n0 & 127;
      brow = n0 - c0;
      b_rows = 128;
      if (n0 >= p.s0) {
        mat = n0 < p.s1 ? p.B1 : p.B2;
        brow -= n0 < p.s1 ? p.s0 : p.s1;
      }
    }
    if (EPI == EPI_SWIGLU) {
      brow = (int64_t)tile_n * (BN / 2);
      b_rows = BN / 2;
    }
    if (EPI == EPI_PARTIAL) {
      // plain column order: 256-column groups of 128 gate and 128 up columns, or
      // the q, k and v rows one after the other
      const int n = tile_n * BN;
      if (p.bmap == BMAP_GATEUP) {
        mat = n & 128 ? p.B1 : p.B0;
        brow = (n >> 8) * 128 + (n & 127);
      } else {
        brow = p.n_begin + n;
        if (p.bmap == BMAP_QKV && brow >= p.s0) {
          mat = brow < p.s1 ? p.B1 : p.B2;
          brow -= brow < p.s1 ? p.s0 : p.s1;
        }
      }
    }
    b_bytes = (int)(b_rows * ldb * 2);
    const int k0 = EPI == EPI_PARTIAL ? split * p.kt_per * BK * 2 : 0;  // first byte of the K range
#pragma unroll
    for (int q = 0; q < LA; ++q) {
      const int r = (wave + WAVES * q) * 8 + lrow;
      // rows past M are clamped to the last one, their results dropped
      a_voff[q] = (int)(min(r, rows_a - 1) * p.lda * 2) + unit * 16 + k0;
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
      const int r = (wave + WAVES * q) * 8 + lrow;
      const int br = EPI == EPI_QKV ? qkv_perm_row(c0 + r) : EPI == EPI_SWIGLU ? gateup_perm_row(r) : r;
      // a block of 8 rows is all gate or all up
      const void* m = EPI == EPI_SWIGLU && ((wave + WAVES * q) >> 1) & 1 ? p.B1 : mat;
      b_base[q] = reinterpret_cast<const bf16_t*>(m) + brow * ldb;
      b_voff[q] = (int)(br * ldb * 2) + unit * 16 + k0;
    }
  }
  const int KT = EPI == EPI_PARTIAL ? min(p.kt_per, p.K / BK - split * p.kt_per) : p.K / BK;  // even
  // past the end the last K tile is fetched again, into a stage nobody reads
  auto issue = [&](int kt) {
    char* st = smem + (kt % STAGES) * STAGE;
    const int kb = min(kt, KT - 1) * BK * 2;
#pragma unroll
    for (int q = 0; q < LA; ++q) load_lds(a_base, a_bytes, st + (wave + WAVES * q) * 1024, a_voff[q], kb);
#pragma unroll
    for (int q = 0; q < LB; ++q)
      load_lds(b_base[q], b_bytes, st + BM * BK * 2 + (wave + WAVES * q) * 1024, b_voff[q], kb);
  };
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
    a_off[ks] = (wm * WR + fr) * (BK * 2) + u;
    b_off[ks] = BM * BK * 2 + (wn * WC + fr) * (BK * 2) + u;
  }
  bf16x8 af[2][2][RI], bf[2][2][CJ];  // [K tile parity][k-step][piece]
  auto read = [&](int kt, int par) {
    const char* st = smem + (kt % STAGES) * STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int j = 0; j < CJ; ++j) bf[par][ks][j] = *reinterpret_cast<const bf16x8*>(st + b_off[ks] + j * 2048);
#pragma unroll
      for (int i = 0; i < RI; ++i) af[par][ks][i] = *reinterpret_cast<const bf16x8*>(st + a_off[ks] + i * 2048);
    }
  };
  KVR_WAIT_VMCNT((STAGES - 1) * LPW);
  __builtin_amdgcn_s_barrier();
  read(0, 0);
  // Step kt: this wave's fragments of K tile kt are in registers and its loads
  // of K tile kt+1 have landed; the barrier makes both true of every wave, so
  // stage kt may be refilled and stage kt+1 read, behind the MFMAs of K tile kt.
  auto step = [&](int kt, int par) {
    __builtin_amdgcn_sched_barrier(0);
    KVR_WAIT_LGKM0();
    KVR_WAIT_VMCNT((STAGES - 2) * LPW);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(kt + 1, par ^ 1);
    issue(kt + STAGES);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[par][ks][j], af[par][ks][i], acc[i][j], 0, 0, 0);
    constexpr int MF = 2 * RI * CJ, RD = 2 * (RI + CJ);
    if constexpr (MF >= RD + LPW) {
#pragma unroll
      for (int q = 0; q < RD; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
#pragma unroll
      for (int q = 0; q < LPW; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      if (MF - RD - LPW > 0) __builtin_amdgcn_sched_group_barrier(0x008, MF - RD - LPW, 0);
    }
  };
  for (int kt = 0; kt < KT; kt += 2) {
    step(kt, 0);
    step(kt + 1, 1);
  }
  KVR_WAIT_LGKM0();
  KVR_WAIT_VMCNT(0);  // trailing refetches land before the LDS is reused or given back

  auto row = [&](int i) { return m0 + wm * WR + i * 16 + fr; };
  auto col = [&](int j) { return wn * WC + j * 16 + 4 * fq; };
  auto ocol = [&](int j) { return (EPI == EPI_SWIGLU ? tile_n * BN : n0) + col(j); };
  if constexpr (EPI == EPI_QKV) {
    acc_qkv<NORM, RI, CJ, BM, BN, WAVES, WR>(acc, m0, p.M, n0, p.epi, smem, wave, lane, row, col);
  } else if constexpr (EPI == EPI_RESID) {
    acc_resid<RI, CJ, RI>(acc, p.M, p.epi, row, ocol);
  } else if constexpr (EPI == EPI_SWIGLU) {
    acc_swiglu<RI, CJ>(acc, p.M, p.epi, row, ocol);
  } else {
    // STORE: the product itself; PARTIAL: one K range's share of it
    float* out = EPI == EPI_STORE ? p.epi.x : p.part + split * p.part_stride;
    const int64_t ld = EPI == EPI_STORE ? p.epi.ldx : p.part_ld;
    const int nb = EPI == EPI_STORE ? n0 : tile_n * BN;
    acc_store<RI, CJ>(acc, p.M, out + nb, ld, row, col);
  }
}

template <int BM, int BN, int WM, int WN, int STAGES, int EPI, bool NORM = false>
void launch_tile(const GemmParams& p_in, hipStream_t s) {
  GemmParams p = p_in;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tiles_n = (p.bmap == BMAP_GATEUP ? 2 * p.epi.ffn : p.n_end - p.n_begin) / BN;
  if (tiles_m <= 0 || tiles_n <= 0) return;
  p.group_m = 8;
  const dim3 grid(tiles_m * tiles_n * (EPI == EPI_PARTIAL ? p.ksplit : 1)), block(64 * WM * WN);
  hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WM, WN, STAGES, EPI, NORM>), grid, block, 0, s, p, tiles_m, tiles_n);
}

// The tiles, and the time of one K tile with one workgroup on each CU (ns,
// measured on products of 64 to 2048 rows with weights from HBM).
enum Tile : int { T32x32, T64x32, T64x64, T64x128, T128x64, T128x128, T256x128, T_WIDE, TILES };
struct TileShape {
  int bm, bn, ns;
};
constexpr TileShape TILE[TILES] = {{32, 32, 170},  {64, 32, 235},   {64, 64, 310},   {64, 128, 480},
                                   {128, 64, 400}, {128, 128, 620}, {256, 128, 810}, {256, 256, 1210}};
constexpr int CUS = 256;

int cdiv(int a, int b) { return (a + b - 1) / b; }
int64_t tiles_of(int t, int M, int N) { return (int64_t)cdiv(M, TILE[t].bm) * (N / TILE[t].bn); }

// Rounds of workgroups over the CUs times the time of a K tile.  Measured over
// 64 to 3072 rows of the 1.5B, 8B and 14B products, the tile of least cost is
// the fastest one or within 7 % of it.
int64_t tile_cost(int t, int64_t workgroups) { return (workgroups + CUS - 1) / CUS * TILE[t].ns; }

// The tile of least cost, the larger one on a tie (fewer bytes moved).
// head_tiles: columns in whole heads (the per-head norm sums one).  64 x 128
// loses to 128 x 64 wherever both may be used.
// A plain store of at most 128 rows keeps to 128-row tiles, whatever near ties say
// (LM head of 128256 columns, K 4096, whole steps: 65 rows 398 us with 128 x 128
// tiles, 412 with 256 x 256 ones; from 129 rows on 519 and 485).
int pick_tile(int M, int N, bool head_tiles, bool wide_ok) {
  int best = T128x128;
  int64_t cost = tile_cost(best, tiles_of(best, M, N));
  for (int t = TILES - 1; t >= 0; --t) {
    if (N % TILE[t].bn != 0 || (t == T_WIDE && !wide_ok)) continue;
    if (head_tiles ? TILE[t].bn < 128 : t == T64x128) continue;
    const int64_t c = tile_cost(t, tiles_of(t, M, N));
    if (c < cost) {
      cost = c;
      best = t;
    }
  }
  return best;
}

template <int EPI>
void launch_picked(int t, const GemmParams& p, hipStream_t s) {
  switch (t) {
    case T32x32: launch_tile<32, 32, 2, 1, 8, EPI>(p, s); break;
    case T64x32: launch_tile<64, 32, 4, 1, 6, EPI>(p, s); break;
    case T64x64: launch_tile<64, 64, 2, 2, 5, EPI>(p, s); break;
    case T128x64: launch_tile<128, 64, 2, 2, 6, EPI>(p, s); break;
    case T256x128: launch_tile<256, 128, 2, 2, 3, EPI>(p, s); break;
    default: launch_tile<128, 128, 2, 2, 4, EPI>(p, s); break;
  }
}

int columns_of(const GemmParams& p) { return p.bmap == BMAP_GATEUP ? 2 * p.epi.ffn : p.n_end - p.n_begin; }

void launch_one(int t, int epi, const GemmParams& p, hipStream_t s) {
  if (t == T_WIDE) {
    launch_gemm_wide(epi, p, s);
  } else if (epi == EPI_QKV && p.epi.q_norm != nullptr) {  // tiles of whole heads
    switch (t) {
      case T64x128: launch_tile<64, 128, 2, 2, 6, EPI_QKV, true>(p, s); break;
      case T256x128: launch_tile<256, 128, 2, 2, 3, EPI_QKV, true>(p, s); break;
      default: launch_tile<128, 128, 2, 2, 4, EPI_QKV, true>(p, s); break;
    }
  } else if (epi == EPI_QKV) {
    launch_picked<EPI_QKV>(t, p, s);
  } else if (epi == EPI_RESID) {
    launch_picked<EPI_RESID>(t, p, s);
  } else if (epi == EPI_SWIGLU) {
    launch_picked<EPI_SWIGLU>(t, p, s);
  } else {
    launch_picked<EPI_STORE>(t, p, s);
  }
}

// Columns [c0, c1) of a product (multiples of 256), as a product of its own
GemmParams columns(int epi, const GemmParams& p, int c0, int c1) {
  GemmParams q = p;
  if (epi == EPI_SWIGLU) {  // half of the columns are outputs
    q.B0 = reinterpret_cast<const bf16_t*>(p.B0) + (int64_t)(c0 / 2) * p.K;
    q.B1 = reinterpret_cast<const bf16_t*>(p.B1) + (int64_t)(c0 / 2) * p.K;
    q.epi.hf = reinterpret_cast<bf16_t*>(p.epi.hf) + c0 / 2;
    q.epi.ffn = (c1 - c0) / 2;
  } else {
    q.n_begin = p.n_begin + c0;
    q.n_end = p.n_begin + c1;
  }
  return q;
}

}  // namespace

void launch_gemm_bf16(int epi, const GemmParams& p, hipStream_t s) {
  const int N = columns_of(p);
  if (p.M <= 0 || N <= 0) return;
  const bool heads = epi == EPI_QKV && p.epi.q_norm != nullptr, wide_ok = epi != EPI_STORE || p.M > 128;
  const int t = pick_tile(p.M, N, heads, wide_ok);
  // A last round of workgroups that is mostly empty costs as much as a full
  // one: where it pays for another launch, whole rounds of one tile take the
  // first columns and a smaller tile the rest.  Gate/up at 1003 rows, K 4096,
  // 384 tiles of 256 x 256: 184 us in two rounds, 102 + 71 as one round and one
  // of 256 x 128 tiles.  Layers of the 8B shape: 520 rows -3.5 %, 3000 -3.2 %,
  // 4200 -10 %, 9000 -1 %; beyond four rounds there is too little to gain.
  constexpr int64_t LAUNCH_NS = 8000;
  const int KT = p.K / BK;
  const int64_t tiles = tiles_of(t, p.M, N);
  int64_t cost = tile_cost(t, tiles) * KT * 15 / 16;  // what the costs are good for
  int best1 = -1, cut = 0;
  if (epi != EPI_STORE && tiles > CUS && tiles <= 4 * CUS)
    for (int t1 = T128x128; t1 < TILES; ++t1) {
      const int tiles_m = cdiv(p.M, TILE[t1].bm);
      for (int r = 1; r <= 3; ++r) {
        const int c = r * CUS / tiles_m * TILE[t1].bn / 256 * 256;  // columns of r whole rounds
        if (c <= 0 || c >= N) continue;
        const int t2 = pick_tile(p.M, N - c, heads, wide_ok);
        const int64_t both = (tile_cost(t1, tiles_of(t1, p.M, c)) + tile_cost(t2, tiles_of(t2, p.M, N - c))) * KT +
                             LAUNCH_NS;
        if (both < cost) {
          cost = both;
          best1 = t1;
          cut = c;
        }
      }
    }
  if (best1 < 0) {
    launch_one(t, epi, p, s);
    return;
  }
  launch_one(best1, epi, columns(epi, p, 0, cut), s);
  launch_one(pick_tile(p.M, N - cut, heads, wide_ok), epi, columns(epi, p, cut, N), s);
}

// Split-K pays where the tiles of a product leave CUs idle: the K tiles per
// workgroup shrink, for one more launch and the partial sums' round trip
// (about SPLIT_NS).  A range is a whole number of K tile pairs.
TilePlan gemm_tile_split_plan(int M, int N, int K, int64_t part_cap) {
  constexpr int64_t SPLIT_NS = 8000;
  const int KT = K / BK;
  TilePlan best{T128x128, 1, KT};
  int64_t cost = INT64_MAX;
  for (int t = T_WIDE - 1; t >= 0; --t) {
    if (t == T64x128 || N % TILE[t].bn != 0) continue;
    const int64_t tiles = tiles_of(t, M, N);
    const int most = (int)std::max<int64_t>(1, std::min<int64_t>(CUS / std::max<int64_t>(1, tiles), 16));
    for (int want = 1; want <= most; ++want) {
      const int per = 2 * cdiv(KT, 2 * want), split = cdiv(KT, per);
      if (split > 1 && (int64_t)split * M * N > part_cap) break;
      const int64_t c = tile_cost(t, tiles * split) * per + (split > 1 ? SPLIT_NS : 0);
      if (c < cost) {
        cost = c;
        best = TilePlan{t, split, per};
      }
    }
  }
  return best;
}

void launch_gemm_tile_partial(const GemmParams& p, const TilePlan& plan, hipStream_t s) {
  GemmParams q = p;
  q.ksplit = plan.ksplit;
  q.kt_per = plan.kt_per;
  launch_picked<EPI_PARTIAL>(plan.tile, q, s);
}

}  // namespace kvr
