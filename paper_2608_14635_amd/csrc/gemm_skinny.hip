// bf16 products of few rows (the resumed decode) on gfx950: a weight-stationary
// kernel for at most 64 rows, and the split-K partial sums of that kernel and
// of the tiled one (gemm_tile.hip), finished by kernels that sum the K ranges
// in a fixed order and apply the decode step's epilogues.  Results are
// deterministic.
#include <algorithm>

#include "common.h"
#include "epilogue.h"
#include "launch.h"

namespace kvr {

namespace {

constexpr int BN = 256;      // columns of an epilogue tile
constexpr int LDC = BN + 4;  // its fp32 row in LDS, elements

// Weight row of column r of epilogue tile tile_n (gate/up: 128 gate columns,
// then the same 128 up columns)
__device__ __forceinline__ const bf16_t* b_row_ptr(const GemmParams& p, int tile_n, int r) {
  const int64_t K = p.ldb ? p.ldb : p.K;
  if (p.bmap == BMAP_GATEUP) {
    const int j = tile_n * (BN / 2) + (r & (BN / 2 - 1));
    const bf16_t* base = reinterpret_cast<const bf16_t*>(r < BN / 2 ? p.B0 : p.B1);
    return base + (int64_t)j * K;
  }
  const int n = p.n_begin + tile_n * BN + r;
  if (p.bmap == BMAP_QKV) {
    if (n < p.s0) return reinterpret_cast<const bf16_t*>(p.B0) + (int64_t)n * K;
    if (n < p.s1) return reinterpret_cast<const bf16_t*>(p.B1) + (int64_t)(n - p.s0) * K;
    return reinterpret_cast<const bf16_t*>(p.B2) + (int64_t)(n - p.s1) * K;
  }
  return reinterpret_cast<const bf16_t*>(p.B0) + (int64_t)n * K;
}

// Split-K partials summed in split order (slice 0, then += slice 1, ...),
// then the fused epilogue, in 32-row x 256-column pieces, exactly as the
// one-pass GEMM would apply it.
constexpr int SK_ROWS = 32;

// Sums the ksplit partials of IPT float4 items (item i at src[i], splits
// stride apart) in split order, with SPB splits of every item loaded before
// any is added, so the loads of a thread overlap instead of waiting one by one.
template <int IPT, int SPB>
__device__ __forceinline__ void sum_splits(const float* const (&src)[IPT], const bool (&valid)[IPT],
                                           int ksplit, int64_t stride, float4 (&a)[IPT]) {
  for (int sp0 = 0; sp0 < ksplit; sp0 += SPB) {
    float4 v[IPT][SPB];
#pragma unroll
    for (int i = 0; i < IPT; ++i)
#pragma unroll
      for (int j = 0; j < SPB; ++j)
        if (valid[i] && sp0 + j < ksplit) v[i][j] = *reinterpret_cast<const float4*>(src[i] + (sp0 + j) * stride);
#pragma unroll
    for (int i = 0; i < IPT; ++i)
#pragma unroll
      for (int j = 0; j < SPB; ++j) {
        if (!valid[i] || sp0 + j >= ksplit) continue;
        if (sp0 + j == 0) {
          a[i] = v[i][j];
        } else {
          a[i].x += v[i][j].x;
          a[i].y += v[i][j].y;
          a[i].z += v[i][j].z;
          a[i].w += v[i][j].w;
        }
      }
  }
}

// TW: the epilogue's tile width, BN or (QKV, head dim dividing 128) 128 for
// twice the workgroups
template <int EPI, int TW>
__global__ __launch_bounds__(256) void splitk_epi_kernel(GemmParams p, int tiles_n) {
  __shared__ __attribute__((aligned(16))) float sC[SK_ROWS * LDC];
  const int tile_n = blockIdx.x % tiles_n, m0 = (blockIdx.x / tiles_n) * SK_ROWS;
  const int tid = threadIdx.x;
  constexpr int IPT = SK_ROWS * (TW / 4) / 256;
  const float* src[IPT];
  bool valid[IPT];
  float4 a[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int it = tid + i * 256, r = it / (TW / 4), c = (it % (TW / 4)) * 4;
    valid[i] = m0 + r < p.M;
    src[i] = p.part + (int64_t)min(m0 + r, p.M - 1) * p.part_ld + tile_n * TW + c;
    a[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  sum_splits<IPT, 4>(src, valid, p.ksplit, p.part_stride, a);
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int it = tid + i * 256, r = it / (TW / 4), c = (it % (TW / 4)) * 4;
    *reinterpret_cast<float4*>(sC + r * LDC + c) = a[i];
  }
  __syncthreads();
  if (EPI == EPI_QKV) {
    epi_qkv<bf16_t, TW, 256>(sC, LDC, SK_ROWS, m0, p.M, p.n_begin + tile_n * TW, p.epi);
  } else {
    epi_swiglu<bf16_t, BN, 256>(sC, LDC, SK_ROWS, m0, p.M, tile_n * (BN / 2), p.epi);
  }
}

// ---- products of few rows (resumed decode) ----
// C[M <= 64, N] = A . B^T, weight-stationary: a wave owns NBW blocks of 16
// output columns (16 weight rows each) and one K range.  It streams those rows
// once with 16-byte loads (per 128-k chunk a lane takes 64 contiguous bytes of
// its row) and multiplies them with every row of A on
// v_mfma_f32_16x16x32_bf16 (16-row tiles of A; rows past M are clamped and
// their results dropped).  The A fragments of a chunk are loaded once for all
// NBW blocks: with one block per wave, the A loads (from L2) equal the weight
// bytes and bound the kernel.  In a chunk of 128 k, MFMA t takes the k values
// 32t+8q..+7 from lane group q = lane/16 (the matrix core's own operand
// layout), so each load instruction reads 64 contiguous bytes of each of 16
// rows and the next one the rest of those lines; the loads are plain (cached),
// as nontemporal ones would fetch the lines again.  The waves of one K range
// are consecutive, so a workgroup's waves read the same A lines.  No LDS and
// no padding work: HBM-bound on the weights.  Output: the fp32 partial sums of
// the K range, in the split-K partial layout.
constexpr int SK_CHUNK = 128;   // k per chunk
constexpr int SK_UNROLL = 2;    // chunks in flight per wave
constexpr int SK_MAX_M = 64;
// K is split into ranges for about SK_WAVES waves, at most 16 where the
// epilogue is elementwise (it sums the splits of every output in parallel)
// and 8 where it works on whole tiles, whose few workgroups read every split
// (measured best on the 8B shapes with weights not in the last-level cache)
constexpr int SK_WAVES = 2048, SK_MAX_SPLIT_ELEM = 16, SK_MAX_SPLIT_TILE = 8;

template <int MT, int NBW>
__global__ __launch_bounds__(256) void gemm_bf16_skinny_kernel(GemmParams p, int ngroups, int kc_per) {
  const int lane = threadIdx.x & 63;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= ngroups * p.ksplit) return;  // whole waves
  const int grp = item % ngroups, split = item / ngroups;
  const int r16 = lane & 15, q = lane >> 4;
  const bf16_t* brow[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const int nb = grp * NBW + b;
    brow[b] = b_row_ptr(p, nb / (BN / 16), (nb % (BN / 16)) * 16 + r16) + 8 * q;
  }
  const bf16_t* arow[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    arow[mt] = reinterpret_cast<const bf16_t*>(p.A) + (int64_t)min(mt * 16 + r16, p.M - 1) * p.lda + 8 * q;
  const int KC = p.K / SK_CHUNK;
  const int kc0 = split * kc_per, kc1 = min(KC, kc0 + kc_per);
  f32x4 acc[NBW][MT];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[b][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // SK_UNROLL chunks of loads in flight (weights first), then their MFMAs
  for (int kc = kc0; kc < kc1; kc += SK_UNROLL) {
    bf16x8 bv[SK_UNROLL][NBW][4], av[SK_UNROLL][MT][4];
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u) {
      if (kc + u < kc1) {
        const int ko = (kc + u) * SK_CHUNK;
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
          for (int t = 0; t < 4; ++t) bv[u][b][t] = *reinterpret_cast<const bf16x8*>(brow[b] + ko + 32 * t);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int t = 0; t < 4; ++t) av[u][mt][t] = *reinterpret_cast<const bf16x8*>(arow[mt] + ko + 32 * t);
      }
    }
#pragma unroll
    for (int u = 0; u < SK_UNROLL; ++u) {
      if (kc + u < kc1) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u][mt][t], bv[u][b][t], acc[b][mt], 0, 0, 0);
      }
    }
  }
  // a lane holds rows 4q .. 4q+3 of each 16-row tile, at column r16 of a block
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const int nb = grp * NBW + b;
    float* out = p.part + split * p.part_stride + nb * 16 + r16;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = mt * 16 + 4 * q + j;
        if (m < p.M) out[(int64_t)m * p.part_ld] = acc[b][mt][j];
      }
  }
}

// Residual sum and RMSNorm after a few-row product: workgroup m sums row m's
// split-K partials in split order into the residual row X (the values
// splitk_elem_kernel writes), then writes round(g * x / rms(x)) as the next
// product's A row.  Every load (X, partials, gain) comes before any store.
constexpr int RN_THREADS = 1024, RN_MAXI = 2;  // rows up to RN_THREADS * 4 * RN_MAXI wide
__global__ __launch_bounds__(RN_THREADS) void splitk_resid_norm_kernel(GemmParams p, const bf16_t* gain,
                                                                       bf16_t* a_out, float eps) {
  __shared__ float red[RN_THREADS / 64];
  const int m = blockIdx.x, tid = threadIdx.x;
  const int N = p.n_end - p.n_begin;
  float* xrow = p.epi.x + (int64_t)m * p.epi.ldx + p.n_begin;
  const float* src[RN_MAXI];
  bool valid[RN_MAXI];
  float4 acc[RN_MAXI], xv[RN_MAXI];
  uint2 gv[RN_MAXI];
#pragma unroll
  for (int i = 0; i < RN_MAXI; ++i) {
    const int col = (tid + i * RN_THREADS) * 4;
    valid[i] = col < N;
    const int cc = valid[i] ? col : 0;
    src[i] = p.part + (int64_t)m * p.part_ld + cc;
    xv[i] = valid[i] ? *reinterpret_cast<const float4*>(xrow + cc) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    gv[i] = valid[i] ? *reinterpret_cast<const uint2*>(gain + cc) : make_uint2(0u, 0u);
    acc[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  sum_splits<RN_MAXI, 8>(src, valid, p.ksplit, p.part_stride, acc);
  float ss = 0.0f;
#pragma unroll
  for (int i = 0; i < RN_MAXI; ++i) {
    if (!valid[i]) continue;
    xv[i].x += acc[i].x;
    xv[i].y += acc[i].y;
    xv[i].z += acc[i].z;
    xv[i].w += acc[i].w;
    ss += xv[i].x * xv[i].x + xv[i].y * xv[i].y + xv[i].z * xv[i].z + xv[i].w * xv[i].w;
  }
#pragma unroll
  for (int i = 0; i < RN_MAXI; ++i)
    if (valid[i]) *reinterpret_cast<float4*>(xrow + (tid + i * RN_THREADS) * 4) = xv[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.0f;
#pragma unroll
  for (int w = 0; w < RN_THREADS / 64; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)N + eps);
#pragma unroll
  for (int i = 0; i < RN_MAXI; ++i) {
    if (!valid[i]) continue;
    const float g0 = __uint_as_float(gv[i].x << 16), g1 = __uint_as_float(gv[i].x & 0xffff0000u);
    const float g2 = __uint_as_float(gv[i].y << 16), g3 = __uint_as_float(gv[i].y & 0xffff0000u);
    uint2 o;
    o.x = (uint32_t)f2bf(g0 * xv[i].x * inv) | ((uint32_t)f2bf(g1 * xv[i].y * inv) << 16);
    o.y = (uint32_t)f2bf(g2 * xv[i].z * inv) | ((uint32_t)f2bf(g3 * xv[i].w * inv) << 16);
    *reinterpret_cast<uint2*>(a_out + (int64_t)m * N + (tid + i * RN_THREADS) * 4) = o;
  }
}

struct SkinnyPlan {
  int nbw, ngroups, ksplit, kc_per;
};

bool skinny_ok(int M, int K) { return M > 0 && M <= SK_MAX_M && K % SK_CHUNK == 0; }

// 16-row blocks per wave: as many as keep the A tiles and the blocks' loads
// in registers (MT tiles of A cost as much as MT blocks)
int skinny_nbw(int M) {
  const int mt = (M + 15) / 16;
  return mt == 1 ? 4 : mt == 2 ? 2 : 1;
}

SkinnyPlan skinny_plan(int M, int tiles_n, int K, int max_split) {
  SkinnyPlan sp;
  sp.nbw = skinny_nbw(M);
  sp.ngroups = tiles_n * (BN / 16) / sp.nbw;
  const int KC = K / SK_CHUNK;
  const int want = std::max(1, std::min({KC, max_split, SK_WAVES / std::max(1, sp.ngroups)}));
  sp.kc_per = (KC + want - 1) / want;
  sp.ksplit = (KC + sp.kc_per - 1) / sp.kc_per;
  return sp;
}

// q.ksplit K ranges of kc_per chunks over ngroups groups of 16-row blocks
void launch_skinny(const GemmParams& q, int ngroups, int kc_per, hipStream_t s) {
  const dim3 grid((unsigned)((ngroups * q.ksplit + 3) / 4)), block(256);
  switch ((q.M + 15) / 16) {
    case 1: hipLaunchKernelGGL((gemm_bf16_skinny_kernel<1, 4>), grid, block, 0, s, q, ngroups, kc_per); break;
    case 2: hipLaunchKernelGGL((gemm_bf16_skinny_kernel<2, 2>), grid, block, 0, s, q, ngroups, kc_per); break;
    case 3: hipLaunchKernelGGL((gemm_bf16_skinny_kernel<3, 1>), grid, block, 0, s, q, ngroups, kc_per); break;
    default: hipLaunchKernelGGL((gemm_bf16_skinny_kernel<4, 1>), grid, block, 0, s, q, ngroups, kc_per); break;
  }
}

int n_tiles_of(const GemmParams& p) {
  return p.bmap == BMAP_GATEUP ? p.epi.ffn / (BN / 2) : (p.n_end - p.n_begin) / BN;
}

}  // namespace

int64_t gemm_bf16_splitk_part_elems(int M, int N, int K) {
  if (skinny_ok(M, K))  // the larger of the two caps: enough for either epilogue
    return (int64_t)skinny_plan(M, N / BN, K, SK_MAX_SPLIT_ELEM).ksplit * M * (N / BN) * BN;
  // K ranges that give every CU a 256 x 256 tile; smaller tiles need no more
  const int KT = K / 64, tiles = std::max(1, (M + 255) / 256 * (N / BN));
  const int want = std::max(1, std::min(KT, (256 + tiles - 1) / tiles));
  const int per = (KT + want - 1) / want;
  return (int64_t)((KT + per - 1) / per) * M * (N / BN) * BN;
}

namespace {

// The K ranges' partial sums of a product of any row count, by the few-row
// kernel or the tiled one; q.ksplit is set.  one_pass: a plan of one range is
// not run (returns false).
bool launch_partials(GemmParams& q, int tiles_n, int max_split, float* part, int64_t part_cap, bool one_pass,
                     hipStream_t s) {
  const int64_t ld = (int64_t)tiles_n * BN;
  q.part = part;
  q.part_ld = (int)ld;
  q.part_stride = (int64_t)q.M * ld;
  if (skinny_ok(q.M, q.K)) {
    const SkinnyPlan kp = skinny_plan(q.M, tiles_n, q.K, max_split);
    if ((int64_t)kp.ksplit * q.M * ld <= part_cap) {
      q.ksplit = kp.ksplit;
      launch_skinny(q, kp.ngroups, kp.kc_per, s);
      return true;
    }
  }
  const TilePlan tp = gemm_tile_split_plan(q.M, (int)ld, q.K, part_cap);
  if (one_pass && tp.ksplit == 1) return false;
  q.ksplit = tp.ksplit;
  launch_gemm_tile_partial(q, tp, s);
  return true;
}

}  // namespace

void launch_gemm_bf16_splitk(int epi, const GemmParams& p, float* part, int64_t part_cap,
                             hipStream_t s) {
  if (p.M <= 0) return;
  const int tiles_n = n_tiles_of(p);
  GemmParams q = p;
  if (!launch_partials(q, tiles_n, SK_MAX_SPLIT_TILE, part, part_cap, true, s)) {
    launch_gemm_bf16(epi, p, s);
    return;
  }
  const dim3 egrid((unsigned)(((p.M + SK_ROWS - 1) / SK_ROWS) * tiles_n));
  if (epi == EPI_QKV) {  // head dim 128: tiles of one head
    const int tiles_h = tiles_n * (BN / 128);
    const dim3 hgrid((unsigned)(((p.M + SK_ROWS - 1) / SK_ROWS) * tiles_h));
    hipLaunchKernelGGL((splitk_epi_kernel<EPI_QKV, 128>), hgrid, dim3(256), 0, s, q, tiles_h);
  } else {
    hipLaunchKernelGGL((splitk_epi_kernel<EPI_SWIGLU, BN>), egrid, dim3(256), 0, s, q, tiles_n);
  }
}

void launch_gemm_bf16_splitk_resid_norm(const GemmParams& p, float* part, int64_t part_cap,
                                        const void* gain, void* a_out, float eps, hipStream_t s) {
  const int N = p.n_end - p.n_begin;
  GemmParams q = p;
  launch_partials(q, N / BN, SK_MAX_SPLIT_ELEM, part, part_cap, false, s);
  hipLaunchKernelGGL(splitk_resid_norm_kernel, dim3((unsigned)p.M), dim3(RN_THREADS), 0, s, q,
                     (const bf16_t*)gain, (bf16_t*)a_out, eps);
}

bool launch_gemm_bf16_rows(const GemmParams& p, float* out, int64_t ldo, hipStream_t s) {
  const int N = p.n_end - p.n_begin;
  if (N <= 0 || ldo < N) return false;
  if (!skinny_ok(p.M, p.K)) {
    if (N % 128 != 0 || ldo % 4 != 0) return false;
    GemmParams q = p;
    q.epi.x = out;
    q.epi.ldx = (int)ldo;
    launch_gemm_bf16(EPI_STORE, q, s);
    return true;
  }
  const int nbw = skinny_nbw(p.M);
  if (N % (16 * nbw) != 0) return false;
  GemmParams q = p;
  q.part = out;
  q.part_ld = (int)ldo;
  q.part_stride = 0;
  q.ksplit = 1;
  const int ngroups = N / 16 / nbw, kc_per = p.K / SK_CHUNK;
  launch_skinny(q, ngroups, kc_per, s);
  return true;
}

}  // namespace kvr
