// bf16 GEMM C[M, N] = A[M, K] . B[N, K]^T on gfx950 matrix cores for products
// of many rows, with the rebuild's epilogues taken from the accumulators
// (gemm_epi.h).
//
// Tile 256 x 256 x 64 per workgroup of 8 wave64s, two per SIMD in two groups
// (waves 0-3 and 4-7) that run half a phase apart: while one group issues its
// 16 MFMAs the other reads its next fragments from LDS and issues its share of
// the loads, so the matrix core of each SIMD always has one wave to serve.
// Each wave owns a 128 x 64 part of the tile as four 64 x 32 quadrants (row
// half a, column half b); a K tile is four phases, one quadrant each.
//
// v_mfma_f32_16x16x32_bf16 throughout: under the card's power limit a loop of
// nothing but these sustains 2.05 PFLOP/s on random data, one of the 32x32x16
// form 1.80 (both 2.4 on zeros), and the two give the same bits.
//
// Operands stream with buffer_load_dwordx4 ... lds into a ring of eight 16 KB
// half tiles (128 rows x 64 k).  Half tile n of the stream is read in phase n
// and its slot refilled in phase n+1, when every wave has read it, with half
// tile n+8: six half tiles (96 KB) are issued ahead per CU, of which the memory
// system has about 32 KB outstanding at a time (gemm_tile.hip).  Even K tiles are
// taken B0 A0 B1 A1, odd ones B1 A0 B0 A1, so each phase needs one new half
// tile (8 or 4 LDS reads per wave) and the other operand is already in
// registers.  A ring of ten half tiles was 2 % slower.
//
// Measured on 131072 rows (against a 4-wave kernel of the same tile with
// 32x32x16 MFMAs, LDS reads interleaved one by one with them and an epilogue
// through LDS): 4096 columns, K 14336: 11.40 -> 10.19 ms; K 4096: 3.60 -> 3.38.
// What bounds it is power: the matrix cores are busy 76-86 % of the time at
// 1.7-1.8 GHz (8B and 32B rebuilds); with every load served by L2 the K 14336
// product takes 9.7 ms.
//
// Workgroups are remapped so that each XCD (dispatch round-robins workgroups
// over the 8 XCDs) works on a contiguous range of tiles, walked in groups of
// group_m M-tiles so that the 32 CUs of an XCD share A rows and B columns in
// their L2.  Every output element is produced by one workgroup with its K
// products added in index order: results are deterministic and do not depend
// on the tile size or on the other rows of the call.
#include "common.h"
#include "dma.h"
#include "gemm_epi.h"
#include "launch.h"

namespace kvr {

namespace {

constexpr int BM = 256, BN = 256, BK = 64, WAVES = 8, NT = 64 * WAVES;
constexpr int SLOTS = 8;
constexpr int HALF_BYTES = 128 * BK * 2;  // one half tile
constexpr int LDS_BYTES = SLOTS * HALF_BYTES;

// Half tiles by kind, in stream order over two K tiles.
enum Kind { A0 = 0, A1 = 1, B0 = 2, B1 = 3 };
constexpr int KIND[8] = {B0, A0, B1, A1, B1, A0, B0, A1};

struct Operand {
  const void* base;  // wave-uniform
  int bytes;         // extent of the resource
  int voff[2][2];    // [half][q]: this lane's byte offset for blocks wave + 8q
};

template <int EPI, bool NORM = false>
__global__ __launch_bounds__(NT, 2) void gemm_wide_kernel(GemmParams p, int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];

  // ---- tile coordinates: XCD-contiguous ranges, grouped along M ----
  const int num_tiles = tiles_m * tiles_n;
  int t = (int)blockIdx.x;
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
  const int wm = wave >> 2, wn = wave & 3;
  const int m0 = tile_m * BM, n0 = p.n_begin + tile_n * BN;

  // ---- direct-to-LDS loaders: wave w fills blocks w and w + 8 of a half tile ----
  Operand oa, ob;
  {
    const int lrow = lane >> 3;
    const int unit = (lane & 7) ^ swz((wave & 1) * 8 + lrow);
    const int rows_a = min(BM, p.M - m0);
    oa.base = reinterpret_cast<const bf16_t*>(p.A) + (int64_t)m0 * p.lda;
    oa.bytes = (int)(rows_a * p.lda * 2);
    // B: a tile lies in one matrix (the QKV split points are multiples of
    // 256), or, for gate/up, each wave's blocks in one of the two
    const void* mat = p.B0;
    int64_t brow = n0;
    if (EPI == EPI_QKV && n0 >= p.s0) {
      mat = n0 < p.s1 ? p.B1 : p.B2;
      brow = n0 - (n0 < p.s1 ? p.s0 : p.s1);
    }
    if (EPI == EPI_SWIGLU) {
      mat = (wave >> 1) & 1 ? p.B1 : p.B0;
      brow = tile_n * (BN / 2);
    }
    ob.base = reinterpret_cast<const bf16_t*>(mat) + brow * p.K;
    ob.bytes = (int)((EPI == EPI_SWIGLU ? BN / 2 : BN) * (int64_t)p.K * 2);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int r = h * 128 + (wave + 8 * q) * 8 + lrow;
        const int br = EPI == EPI_QKV ? qkv_perm_row(r) : EPI == EPI_SWIGLU ? gateup_perm_row(r) : r;
        // rows past M are clamped to the last one, their results dropped
        oa.voff[h][q] = (int)(min(r, rows_a - 1) * p.lda * 2) + unit * 16;
        ob.voff[h][q] = br * p.K * 2 + unit * 16;
      }
  }
  const int KT = p.K / BK;  // even
  // past the end the last K tile is fetched again, into slots no phase reads
  auto issue = [&](int kind, int kt, int slot) {
    char* dst = smem + slot * HALF_BYTES + wave * 1024;
    const Operand& o = kind < 2 ? oa : ob;
    const int kb = min(kt, KT - 1) * BK * 2;
#pragma unroll
    for (int q = 0; q < 2; ++q) load_lds(o.base, o.bytes, dst + q * 8192, o.voff[kind & 1][q], kb);
  };
#pragma unroll
  for (int n = 0; n < SLOTS; ++n) issue(KIND[n], n >> 2, n);

  f32x4 acc[8][4];  // [4a + i][2b + j]: quadrant (a, b), 16 x 16 piece (i, j)
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // fragment reads: lane%16 picks the row, lane/16 the 8-wide part of a 32-k step
  const int fr = lane & 15, fq = lane >> 4;
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int u = ((ks * 4 + fq) ^ swz(fr)) << 4;
    a_off[ks] = (wm * 64 + fr) * (BK * 2) + u;
    b_off[ks] = (wn * 32 + fr) * (BK * 2) + u;
  }
  bf16x8 af[2][4], bf0[2][2], bf1[2][2];
  auto read_a = [&](int slot) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        af[ks][i] = *reinterpret_cast<const bf16x8*>(smem + slot * HALF_BYTES + a_off[ks] + i * 2048);
  };
  auto read_b = [&](int slot, bf16x8 (&bf)[2][2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bf[ks][j] = *reinterpret_cast<const bf16x8*>(smem + slot * HALF_BYTES + b_off[ks] + j * 2048);
  };
  // the 16 MFMAs of quadrant (a, b), k ascending per accumulator
  auto quadrant = [&](int a, int b, const bf16x8 (&bf)[2][2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[4 * a + i][2 * b + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              bf[ks][j], af[ks][i], acc[4 * a + i][2 * b + j], 0, 0, 0);
  };
  // Between a phase's reads and its MFMAs: this wave's loads of the next
  // phase's half tile have landed (all but the newest six half tiles), its
  // fragments are in registers, and the barrier makes both true of the other
  // group's half phase as well.
  auto turn = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    KVR_WAIT_VMCNT(2 * (SLOTS - 2));
    KVR_WAIT_LGKM0();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
  };
  auto done = [&]() {
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  // phase 0: half tiles 0 and 1 have landed, B0 of K tile 0 is read
  KVR_WAIT_VMCNT(2 * (SLOTS - 2));
  __builtin_amdgcn_s_barrier();
  read_b(0, bf0);
  KVR_WAIT_LGKM0();
  __builtin_amdgcn_s_barrier();
  if (wave >= 4) __builtin_amdgcn_s_barrier();  // the second group runs half a phase behind
  __builtin_amdgcn_sched_barrier(0);
  for (int kt = 0; kt < KT; kt += 2) {
    // phase n of the pair of K tiles reads slot n and refills slot n-1
    read_a(1);       issue(B0, kt + 2, 0); turn(); quadrant(0, 0, bf0); done();
    read_b(2, bf1);  issue(A0, kt + 2, 1); turn(); quadrant(0, 1, bf1); done();
    read_a(3);       issue(B1, kt + 2, 2); turn(); quadrant(1, 1, bf1); done();
    read_b(4, bf1);  issue(A1, kt + 2, 3); turn(); quadrant(1, 0, bf0); done();
    read_a(5);       issue(B1, kt + 3, 4); turn(); quadrant(0, 1, bf1); done();
    read_b(6, bf0);  issue(A0, kt + 3, 5); turn(); quadrant(0, 0, bf0); done();
    read_a(7);       issue(B0, kt + 3, 6); turn(); quadrant(1, 0, bf0); done();
    read_b(0, bf0);  issue(A1, kt + 3, 7); turn(); quadrant(1, 1, bf1); done();
  }
  if (wave < 4) __builtin_amdgcn_s_barrier();
  KVR_WAIT_VMCNT(0);  // the trailing refetches land before the ring is reused or given back

  auto row = [&](int i) { return m0 + (i >> 2) * 128 + wm * 64 + (i & 3) * 16 + fr; };
  auto col = [&](int j) { return (j >> 1) * 128 + wn * 32 + (j & 1) * 16 + 4 * fq; };
  auto ocol = [&](int j) { return (EPI == EPI_SWIGLU ? tile_n * BN : n0) + col(j); };
  if constexpr (EPI == EPI_QKV) {
    acc_qkv<NORM, 8, 4, BM, BN, WAVES, 64>(acc, m0, p.M, n0, p.epi, smem, wave, lane, row, col);
  } else if constexpr (EPI == EPI_RESID) {
    acc_resid<8, 4, 4>(acc, p.M, p.epi, row, ocol);
  } else if constexpr (EPI == EPI_STORE) {
    acc_store<8, 4>(acc, p.M, p.epi.x, p.epi.ldx, row, ocol);
  } else {
    acc_swiglu<8, 4>(acc, p.M, p.epi, row, ocol);
  }
}

}  // namespace

void launch_gemm_wide(int epi, const GemmParams& p_in, hipStream_t s) {
  GemmParams p = p_in;
  const int tiles_m = (p.M + BM - 1) / BM;
  const int tiles_n = epi == EPI_SWIGLU ? p.epi.ffn / (BN / 2) : (p.n_end - p.n_begin) / BN;
  if (tiles_m <= 0 || tiles_n <= 0) return;
  // 4 M-tiles x 8 N-tiles at a time where there are at most 24 N-tiles (the
  // long A panels then stay in the last-level cache), 8 x 4 otherwise
  p.group_m = tiles_n <= 24 ? 4 : 8;
  const dim3 grid(tiles_m * tiles_n), block(NT);
  if (epi == EPI_QKV && p.epi.q_norm != nullptr)
    hipLaunchKernelGGL((gemm_wide_kernel<EPI_QKV, true>), grid, block, 0, s, p, tiles_m, tiles_n);
  else if (epi == EPI_QKV)
    hipLaunchKernelGGL(gemm_wide_kernel<EPI_QKV>, grid, block, 0, s, p, tiles_m, tiles_n);
  else if (epi == EPI_RESID)
    hipLaunchKernelGGL(gemm_wide_kernel<EPI_RESID>, grid, block, 0, s, p, tiles_m, tiles_n);
  else if (epi == EPI_STORE)
    hipLaunchKernelGGL(gemm_wide_kernel<EPI_STORE>, grid, block, 0, s, p, tiles_m, tiles_n);
  else
    hipLaunchKernelGGL(gemm_wide_kernel<EPI_SWIGLU>, grid, block, 0, s, p, tiles_m, tiles_n);
}

}  // namespace kvr
