// bf16 products of the resumed decode on gfx950: a one-pass kernel for at most
// 64 rows, and, above, the tiled product (gemm_tile.hip) with its split-K
// partials finished by kernels that sum the K ranges in a fixed order and apply
// the decode step's epilogues.  Results are deterministic.
#include <algorithm>

#include "common.h"
#include "epilogue.h"
#include "gemm_epi.h"
#include "launch.h"

namespace kvr {

namespace {

constexpr int BN = 256;      // columns of an epilogue tile
constexpr int LDC = BN + 4;  // its fp32 row in LDS, elements

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

// TW: the epilogue's tile width, a head for QKV and BN for SWIGLU
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
    epi_qkv<256>(sC, LDC, SK_ROWS, m0, p.M, p.n_begin + tile_n * TW, p.epi);
  } else {
    epi_swiglu<BN, 256>(sC, LDC, SK_ROWS, m0, p.M, tile_n * (BN / 2), p.epi);
  }
}

// ---- products of few rows (resumed decode) ----
// C[M <= 64, N] = A . B^T in one pass: a workgroup of 8 waves owns CB blocks of
// 16 output columns (16 weight rows each) and each wave an eighth of K.  A wave
// streams its part of those rows once with 16-byte loads, in the matrix core's
// own operand layout, SK_UNROLL chunks of 128 k at a time, and multiplies them
// with every row of A on v_mfma_f32_16x16x32_bf16 (16-row tiles of A; rows past
// M are clamped and their results dropped).  The waves' sums meet in LDS and are
// added in wave order, and the epilogue follows in the same kernel: no partial
// sums in memory, no second launch.
//
// HBM-bound on the weights.  A CU has about 32 KB of loads outstanding, shared by
// the weights and by A's rows from L2 (gemm_tile.hip), so CB is the smallest that
// the epilogue allows where that gives every CU a workgroup.
// The eight K ranges also spread the accesses: all workgroups walking K in step
// through rows 8 KB apart (hidden size 4096) reach 4.6-4.9 TB/s where other
// row lengths reach 6.
constexpr int SK_CHUNK = 128;  // k per chunk
constexpr int SK_MAX_M = 64;
constexpr int SK_W = 8;        // waves, K ranges
constexpr int CUS = 256;

// Weight row behind column n of the product, in the order of the epilogue's
// pairs (QKV: 16 dims and their rotary partners; gate/up: 16 gate and 16 up rows)
template <int EPI>
__device__ __forceinline__ const bf16_t* rows_b_ptr(const GemmParams& p, int n) {
  if (EPI == EPI_SWIGLU)
    return reinterpret_cast<const bf16_t*>((n >> 4) & 1 ? p.B1 : p.B0) + (int64_t)gateup_perm_row(n) * p.K;
  if (EPI == EPI_QKV) {
    const int reg = n < p.s0 ? 0 : n < p.s1 ? p.s0 : p.s1;
    const void* m = n < p.s0 ? p.B0 : n < p.s1 ? p.B1 : p.B2;
    return reinterpret_cast<const bf16_t*>(m) + (int64_t)qkv_perm_row(n - reg) * p.K;
  }
  if (p.bmap == BMAP_QKV) {  // raw columns (a separate pass norms and rotates)
    if (n < p.s0) return reinterpret_cast<const bf16_t*>(p.B0) + (int64_t)n * p.K;
    if (n < p.s1) return reinterpret_cast<const bf16_t*>(p.B1) + (int64_t)(n - p.s0) * p.K;
    return reinterpret_cast<const bf16_t*>(p.B2) + (int64_t)(n - p.s1) * p.K;
  }
  return reinterpret_cast<const bf16_t*>(p.B0) + (int64_t)n * p.K;
}

template <int MT, int CB, int EPI>
__global__ __launch_bounds__(64 * SK_W) void gemm_rows_kernel(GemmParams p) {
  // chunks of loads in flight per wave: as many as 256 registers hold
  constexpr int U = CB * 2 + MT * 2 <= 4 ? 4 : CB + MT <= 3 ? 3 : CB + MT <= 5 ? 2 : 1;
  constexpr int NP = EPI == EPI_QKV || EPI == EPI_SWIGLU ? CB / 2 : CB;  // column items (pairs or blocks)
  constexpr int ITEMS = NP * MT * 64;
  __shared__ __attribute__((aligned(16))) f32x4 red[SK_W][CB * MT * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, q = lane >> 4;
  // PARTIAL: consecutive workgroups take one K range each of the same columns
  const int ksplit = EPI == EPI_PARTIAL ? p.ksplit : 1;
  const int split = EPI == EPI_PARTIAL ? (int)(blockIdx.x % ksplit) : 0;
  const int n0 = p.n_begin + (EPI == EPI_PARTIAL ? (int)(blockIdx.x / ksplit) : (int)blockIdx.x) * (CB * 16);
  const bf16_t* brow[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) brow[b] = rows_b_ptr<EPI>(p, n0 + b * 16 + r16) + 8 * q;
  const bf16_t* arow[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    arow[mt] = reinterpret_cast<const bf16_t*>(p.A) + (int64_t)min(mt * 16 + r16, p.M - 1) * p.lda + 8 * q;
  const int KC = p.K / SK_CHUNK;
  const int range = split * SK_W + wave, ranges = ksplit * SK_W;
  const int kc0 = range * KC / ranges, kc1 = (range + 1) * KC / ranges;
  f32x4 acc[CB][MT];
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[b][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int kc = kc0; kc < kc1; kc += U) {
    bf16x8 bv[U][CB][4], av[U][MT][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kc + u < kc1) {
        const int ko = (kc + u) * SK_CHUNK;
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
          for (int t = 0; t < 4; ++t) bv[u][b][t] = *reinterpret_cast<const bf16x8*>(brow[b] + ko + 32 * t);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int t = 0; t < 4; ++t) av[u][mt][t] = *reinterpret_cast<const bf16x8*>(arow[mt] + ko + 32 * t);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kc + u < kc1) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[b][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[u][b][t], av[u][mt][t], acc[b][mt], 0, 0, 0);
      }
    }
  }
  // lane: columns 4q .. 4q+3 of each block, row r16 of each tile
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[wave][(b * MT + mt) * 64 + lane] = acc[b][mt];
  __syncthreads();
  const EpiParams& e = p.epi;
  for (int it = threadIdx.x; it < ITEMS; it += 64 * SK_W) {
    const int l = it & 63, mt = (it >> 6) % MT, x = (it >> 6) / MT;
    const int m = mt * 16 + (l & 15), c4 = 4 * (l >> 4);
    if (m >= p.M) continue;
    auto sum = [&](int b) {
      f32x4 s = red[0][(b * MT + mt) * 64 + l];
#pragma unroll
      for (int w = 1; w < SK_W; ++w) s += red[w][(b * MT + mt) * 64 + l];
      return s;
    };
    if constexpr (EPI == EPI_SWIGLU) {
      const f32x4 g = sum(2 * x), u = sum(2 * x + 1);
      float h[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) h[k] = silu(g[k]) * u[k];
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(e.hf) + (int64_t)m * e.ldh + gateup_perm_row(n0 + 32 * x) +
                                c4) = pack4(h);
    } else if constexpr (EPI == EPI_QKV) {
      const f32x4 a = sum(2 * x), b = sum(2 * x + 1);
      const int n = n0 + 32 * x;
      const int region = n < p.s0 ? 0 : n < p.s1 ? 1 : 2, c = n - (region == 0 ? 0 : region == 1 ? p.s0 : p.s1);
      const int hd = c >> 7, d0 = ((c & 127) >> 5) * 16 + c4;
      float lo[4], hi[4], ba[4] = {0.0f, 0.0f, 0.0f, 0.0f}, bb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      const bf16_t* bias = reinterpret_cast<const bf16_t*>(region == 0 ? e.bq : region == 1 ? e.bk : e.bv);
      if (bias != nullptr) {
        unpack4(*reinterpret_cast<const uint2*>(bias + hd * 128 + d0), ba);
        unpack4(*reinterpret_cast<const uint2*>(bias + hd * 128 + d0 + 64), bb);
      }
      const float2* cs = e.rope + (int64_t)e.pos[m] * 64 + d0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float va = a[k] + ba[k], vb = b[k] + bb[k];
        const float2 t = region < 2 ? cs[k] : make_float2(1.0f, 0.0f);
        // a v dim has no partner (and 0 times one that is not finite is not 0)
        lo[k] = region < 2 ? va * t.x - vb * t.y : va;
        hi[k] = region < 2 ? vb * t.x + va * t.y : vb;
      }
      bf16_t* dst;
      if (region == 0)
        dst = reinterpret_cast<bf16_t*>(e.q_out) + (int64_t)m * e.nq * 128;
      else
        dst = reinterpret_cast<bf16_t*>(region == 1 ? e.arena_k : e.arena_v) + e.slot[m] * (int64_t)(e.nkv * 128);
      dst += hd * 128 + d0;
      *reinterpret_cast<uint2*>(dst) = pack4(lo);
      *reinterpret_cast<uint2*>(dst + 64) = pack4(hi);
    } else if constexpr (EPI == EPI_PARTIAL) {
      *reinterpret_cast<f32x4*>(p.part + split * p.part_stride + (int64_t)m * p.part_ld + n0 + x * 16 + c4) = sum(x);
    } else {
      *reinterpret_cast<f32x4_a4*>(e.x + (int64_t)m * e.ldx + n0 + x * 16 + c4) = sum(x);
    }
  }
}

// Residual sum and RMSNorm after a few-row product: workgroup m sums row m's
// split-K partials in split order into the residual row X, then writes
// round(g * x / rms(x)) as the next product's A row.  Every load (X, partials,
// gain) comes before any store.
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

bool few_rows(int M) { return M > 0 && M <= SK_MAX_M; }

template <int CB, int EPI>
void launch_rows(const GemmParams& p, int N, hipStream_t s) {
  const dim3 grid((unsigned)(N / (16 * CB) * (EPI == EPI_PARTIAL ? p.ksplit : 1))), block(64 * SK_W);
  switch ((p.M + 15) / 16) {
    case 1: hipLaunchKernelGGL((gemm_rows_kernel<1, CB, EPI>), grid, block, 0, s, p); break;
    case 2: hipLaunchKernelGGL((gemm_rows_kernel<2, CB, EPI>), grid, block, 0, s, p); break;
    case 3: hipLaunchKernelGGL((gemm_rows_kernel<3, CB, EPI>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((gemm_rows_kernel<4, CB, EPI>), grid, block, 0, s, p); break;
  }
}

int n_tiles_of(const GemmParams& p) {
  return p.bmap == BMAP_GATEUP ? p.epi.ffn / (BN / 2) : (p.n_end - p.n_begin) / BN;
}

}  // namespace

int64_t gemm_bf16_splitk_part_elems(int M, int N, int K) {
  // few rows: the raw columns of a product whose epilogue is a second pass, in
  // as many copies as K ranges of 512 up to 16 (the size this has always had)
  if (few_rows(M)) {
    const int KC = K / SK_CHUNK, mt = (M + 15) / 16, nbw = mt == 1 ? 4 : mt == 2 ? 2 : 1;
    const int ngroups = N / 16 / nbw;
    const int want = std::max(1, std::min({KC, 16, 2048 / std::max(1, ngroups)}));
    const int per = (KC + want - 1) / want;
    return (int64_t)((KC + per - 1) / per) * M * (N / BN) * BN;
  }
  // K ranges that give every CU a 256 x 256 tile; smaller tiles need no more
  const int KT = K / 64, tiles = std::max(1, (M + 255) / 256 * (N / BN));
  const int want = std::max(1, std::min(KT, (256 + tiles - 1) / tiles));
  const int per = (KT + want - 1) / want;
  return (int64_t)((KT + per - 1) / per) * M * (N / BN) * BN;
}

void launch_gemm_bf16_splitk(int epi, const GemmParams& p, float* part, int64_t part_cap,
                             hipStream_t s) {
  if (p.M <= 0) return;
  const int tiles_n = n_tiles_of(p), N = tiles_n * BN;
  const bool head_norm = epi == EPI_QKV && p.epi.q_norm != nullptr;
  GemmParams q = p;
  q.part = part;
  q.part_ld = N;
  q.part_stride = (int64_t)p.M * N;
  q.ksplit = 1;
  if (few_rows(p.M)) {
    if (epi == EPI_SWIGLU) {
      // beyond a few rows A's share of the operand stream outweighs the finer
      // split (8B, us: 1 row 45.3 / 45.8, 16 rows 55.3 / 50.7, 64 rows 97 / 73)
      if (p.M <= 4)
        launch_rows<2, EPI_SWIGLU>(p, N, s);
      else
        launch_rows<4, EPI_SWIGLU>(p, N, s);
      return;
    }
    if (!head_norm) {
      launch_rows<2, EPI_QKV>(p, N, s);
      return;
    }
    // per-head norms sum whole heads: the raw columns first
    q.epi.x = part - p.n_begin;
    q.epi.ldx = N;
    launch_rows<1, EPI_STORE>(q, N, s);
  } else {
    const TilePlan tp = gemm_tile_split_plan(p.M, N, p.K, part_cap);
    if (tp.ksplit == 1) {
      launch_gemm_bf16(epi, p, s);
      return;
    }
    q.ksplit = tp.ksplit;
    launch_gemm_tile_partial(q, tp, s);
  }
  const unsigned mblocks = (unsigned)((p.M + SK_ROWS - 1) / SK_ROWS);
  if (epi == EPI_QKV) {  // head dim 128: tiles of one head
    const int tiles_h = tiles_n * (BN / 128);
    hipLaunchKernelGGL((splitk_epi_kernel<EPI_QKV, 128>), dim3(mblocks * tiles_h), dim3(256), 0, s, q, tiles_h);
  } else {
    hipLaunchKernelGGL((splitk_epi_kernel<EPI_SWIGLU, BN>), dim3(mblocks * tiles_n), dim3(256), 0, s, q, tiles_n);
  }
}

void launch_gemm_bf16_resid_norm(const GemmParams& p, float* part, int64_t part_cap, const void* gain,
                                 void* a_out, float eps, hipStream_t s) {
  const int N = p.n_end - p.n_begin;
  GemmParams q = p;
  q.part = part;
  q.part_ld = N;
  q.part_stride = (int64_t)p.M * N;
  if (few_rows(p.M)) {
    // 64 columns a workgroup, so that A is a quarter of the stream (at 16 rows),
    // and enough K ranges to give every CU one; the norm's kernel adds them up.
    // (16 columns and all of K in a workgroup, then the norm: 12 us a step more
    // for one request through 8 layers, 48 for 16 requests through 4.)
    const int64_t fit = std::max<int64_t>(1, part_cap / q.part_stride);
    q.ksplit = (int)std::min<int64_t>({(int64_t)std::max(1, CUS / (N / 64)), fit, std::max(1, p.K / SK_CHUNK / SK_W)});
    launch_rows<4, EPI_PARTIAL>(q, N, s);
  } else {
    const TilePlan tp = gemm_tile_split_plan(p.M, N, p.K, part_cap);
    q.ksplit = tp.ksplit;
    launch_gemm_tile_partial(q, tp, s);
  }
  hipLaunchKernelGGL(splitk_resid_norm_kernel, dim3((unsigned)p.M), dim3(RN_THREADS), 0, s, q,
                     (const bf16_t*)gain, (bf16_t*)a_out, eps);
}

bool launch_gemm_bf16_rows(const GemmParams& p, float* out, int64_t ldo, hipStream_t s) {
  const int N = p.n_end - p.n_begin;
  if (N <= 0 || ldo < N) return false;
  GemmParams q = p;
  q.epi.x = out;
  q.epi.ldx = (int)ldo;
  if (!few_rows(p.M)) {
    if (N % 128 != 0) return false;
    launch_gemm_bf16(EPI_STORE, q, s);
  } else if (N % 64 == 0) {
    launch_rows<4, EPI_STORE>(q, N, s);
  } else if (N % 32 == 0) {
    launch_rows<2, EPI_STORE>(q, N, s);
  } else if (N % 16 == 0) {
    launch_rows<1, EPI_STORE>(q, N, s);
  } else {
    return false;
  }
  return true;
}

}  // namespace kvr
