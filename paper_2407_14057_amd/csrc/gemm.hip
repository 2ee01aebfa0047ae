// bf16 GEMM on the gfx950 matrix cores: C[M,N] = A[M,K] W[N,K]^T, fp32 accumulation.
// Both operands are K-contiguous, which is the layout the MFMA instructions want: lane l of
// v_mfma_f32_32x32x16_bf16 supplies row (l & 31), k elements 8*(l >> 5) .. +8 of a 32x16 operand block.
// This file: the 128-row tiles for small shapes, 128x128 stream-K, and the choice among all kernels (the
// four-wave tiles of gemm_w4.h, the streaming kernel of gemm_stream.hip).
//
// Workgroup = WM x WN waves, each wave owns TM x TN blocks of 32x32 (fp32 accumulators stay
// in registers for the whole K loop).  K advances 64 elements per step; the A and W slabs of
// a step are copied global -> LDS by global_load_lds (no register staging) into one of two
// LDS stages while the other stage feeds the MFMAs.
//
// W may be row-major [N][K] (row stride ldw) or K-step-major [K/64][N][64] (EpiArgs::w_blocked, the
// order the model keeps its weights in): the kernels only differ in two byte strides, row to row
// (ldw * 2 or 128) and K step to K step (128 or N * 128).  K-step-major, the slab of one step is
// one contiguous run, which the memory system serves better than one line from each of 256 rows.
#include <stdlib.h>

#include "common.h"
#include "gemm_shared.h"

namespace lz {

// Workspace of the forms that exchange partial sums between workgroups.  Layout: fp32 partial tiles
// (64 MB) | 4 KB of tickets of the weight-streaming kernel (gemm_stream.hip) | 4 KB of flags of the
// four-wave kernel's stream-K schedule (gemm_w4.h; word 1023 counts its give-ups).  Tickets and
// flags must be zero before the first launch that uses them; every launch leaves them zero again.
constexpr int SK_GRID = 512;
constexpr size_t SK_PART_BYTES = (size_t)SK_GRID * 2 * 128 * 128 * sizeof(float);
constexpr size_t SK_TICKET_BYTES = 4096, PSK_FLAG_BYTES = 4096;

template <int WM, int WN, int TM, int TN, int EPI, int NS = 2>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
            uint16_t* __restrict__ C, const uint16_t* __restrict__ R, int M, int N, int K, int lda,
            int ldw, int ldc, int tiles_m, int tiles_n, int group_m, EpiArgs ra) {
  constexpr int NWAVES = WM * WN;
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  constexpr int A_INSTR = BM / 8 / NWAVES;      // wave-wide 1 KB copies per wave per step
  constexpr int W_INSTR = BN / 8 / NWAVES;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  static_assert(BM % (8 * NWAVES) == 0 && BN % (8 * NWAVES) == 0, "tile/wave mismatch");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if ((int)blockIdx.x >= tiles_m * tiles_n) {     // side job (see EpiArgs): Eq. 1 scores
    const int sb = (int)blockIdx.x - tiles_m * tiles_n;
    score_finish_block<true>(ra.sf_z, ra.sf_stat, ra.sf_s, ra.sf_cu, ra.sf_n_single, ra.sf_heads,
                             ra.sf_z_ld, ra.sf_cu_z, true, sb / ra.sf_blocks_per_seq,
                             (sb % ra.sf_blocks_per_seq) * (int)blockDim.x, (float2*)lds);
    return;
  }

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- workgroup -> tile.  Consecutive workgroup ids land on different XCDs (8 of them,
  // each with its own L2), so ids are first regrouped per XCD, then walked in bands of
  // GROUP_M tile rows so that concurrently running tiles share A and W slabs in L2.
  int tile_m, tile_n;
  workgroup_tile((int)blockIdx.x, tiles_m, tiles_n, group_m, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  // ---- global -> LDS copy plan.  Lane p of a wave instruction fills LDS bytes
  // [16p, 16p+16) of an 8-row slab: row p/8, stored chunk p%8, which holds logical
  // chunk (p%8) ^ swz64(row).
  const int crow = lane >> 3;
  uint32_t a_off[A_INSTR], w_off[W_INSTR];
#pragma unroll
  for (int q = 0; q < A_INSTR; ++q) {
    const int tr = (wave * A_INSTR + q) * 8 + crow;          // row inside the tile
    const int cchunk = (lane & 7) ^ swz64(tr);
    int r = m0 + tr;
    r = r < M ? r : M - 1;                       // rows past the edge: re-read the last row
    if (ra.a_rows != nullptr) r = ra.a_rows[r];
    a_off[q] = (uint32_t)(((size_t)r * lda + cchunk * 8) * 2);
  }
#pragma unroll
  for (int q = 0; q < W_INSTR; ++q) {
    const int tr = (wave * W_INSTR + q) * 8 + crow;
    const int cchunk = (lane & 7) ^ swz64(tr);
    int r = n0 + tr;
    r = r < N ? r : N - 1;
    w_off[q] = (uint32_t)(((size_t)r * ldw + cchunk * 8) * 2);
  }

  const size_t wstep = (size_t)ra.w_step_bytes;     // 128, or N * 128 for the K-step-major weight
  auto issue = [&](int stage, int k0) {
    char* sa = lds + stage * STAGE_BYTES + (wave * A_INSTR) * 1024;
    char* sw = lds + stage * STAGE_BYTES + BM * ROW_BYTES + (wave * W_INSTR) * 1024;
    const char* ga = (const char*)A + (size_t)k0 * 2;
    const char* gw = (const char*)W + (size_t)(k0 / BK) * wstep;
#pragma unroll
    for (int q = 0; q < A_INSTR; ++q) g2l16(ga + a_off[q], sa + q * 1024);
#pragma unroll
    for (int q = 0; q < W_INSTR; ++q) g2l16(gw + w_off[q], sw + q * 1024);
  };

  // ---- MFMA operand addresses: row (l & 31) of a 32-row block, chunk 2*ks + (l >> 5)
  uint32_t koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    koff[ks] = (uint32_t)(((ks * 2 + (lane >> 5)) ^ swz64(lane & 31)) * 16);
  const uint32_t a_row = (uint32_t)((wm * TM * 32 + (lane & 31)) * ROW_BYTES);
  const uint32_t w_row = (uint32_t)(BM * ROW_BYTES + (wn * TN * 32 + (lane & 31)) * ROW_BYTES);

  floatx16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // ---- main loop.  Operand fragments are double-buffered in registers: the reads for k-step
  // s+1 are issued before the MFMAs of k-step s.  The single barrier of an iteration sits
  // before the last k-step, when every wave has pulled its last fragments of the current
  // stage into registers; the stage is then free to receive the tile two steps ahead, and the
  // first fragments of the next stage are fetched under the last 16 MFMAs.
  bf16x8_t af[2][TM], wf[2][TN];
#define LZ_LOAD_FRAGS(buf, st, ks)                                                            \
  do {                                                                                        \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                            \
        af[buf][i] = *(const bf16x8_t*)((st) + a_row + i * 32 * ROW_BYTES + koff[ks]);        \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
        wf[buf][j] = *(const bf16x8_t*)((st) + w_row + j * 32 * ROW_BYTES + koff[ks]);        \
  } while (0)
#define LZ_MFMAS(buf)                                                                         \
  do {                                                                                        \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                            \
      _Pragma("unroll") for (int j = 0; j < TN; ++j)                                          \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[buf][j], af[buf][i],           \
                                                            acc[i][j], 0, 0, 0);              \
  } while (0)
  // Order inside a k-step: the LDS reads of the NEXT k-step go out first, one or two per MFMA,
  // so that the last of them still has at least half a k-step of MFMAs to land under.
#define LZ_SCHED()                                                                            \
  do {                                                                                        \
    constexpr int NR = TM + TN, NM = TM * TN;                                                 \
    constexpr int RPG = (NR * 2 > NM) ? 2 : 1;          /* reads per group */                 \
    constexpr int NG = NR / RPG;                                                              \
    _Pragma("unroll") for (int n = 0; n < NG; ++n) {                                          \
      __builtin_amdgcn_sched_group_barrier(0x100, RPG, 0);                                    \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                      \
    }                                                                                         \
    __builtin_amdgcn_sched_group_barrier(0x008, NM - NG, 0);                                  \
  } while (0)

  // NS stages: K step kt lives in stage kt mod NS; steps 0 .. NS-1 are copied up front, step
  // kt + NS in iteration kt, right after the barrier that frees step kt's stage.  With more than
  // two stages the barrier waits only for the copies of step kt + 1 (everything but the newest
  // NS - 2 steps' worth): a copy then has NS - 3/4 iterations to arrive instead of 1 1/4.
  static_assert(NS == 2 || NS == 3, "two or three stages");
  const int KT = K / BK;
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < KT) issue(t, t * BK);
  float rs[TM];
  load_row_scales<TM>(rs, ra, M, m0, wm, lane);
  // (three steps in flight: only the first has to be there; the row scales fetched last are needed in the epilogue)
  if (NS == 3 && KT >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * (A_INSTR + W_INSTR)) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  LZ_LOAD_FRAGS(0, lds, 0);
  int st_cur = 0;                                   // kt mod NS
  for (int kt = 0; kt < KT; ++kt) {
    const int st_nxt = st_cur + 1 == NS ? 0 : st_cur + 1;
    const char* cur = lds + st_cur * STAGE_BYTES;
    const char* nxt = lds + st_nxt * STAGE_BYTES;
    LZ_LOAD_FRAGS(1, cur, 1);
    LZ_MFMAS(0);
    LZ_SCHED();
    LZ_LOAD_FRAGS(0, cur, 2);
    LZ_MFMAS(1);
    LZ_SCHED();
    LZ_LOAD_FRAGS(1, cur, 3);
    LZ_MFMAS(0);
    LZ_SCHED();
    // step kt + 1 must have landed; with three stages step kt + 2 (issued an iteration ago) may
    // still be on its way, unless it does not exist
    if (NS == 3 && kt + 2 < KT) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(A_INSTR + W_INSTR) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (kt + NS < KT) issue(st_cur, (kt + NS) * BK);
    if (kt + 1 < KT) LZ_LOAD_FRAGS(0, nxt, 0);
    LZ_MFMAS(1);
    LZ_SCHED();
    st_cur = st_nxt;
  }
#undef LZ_LOAD_FRAGS
#undef LZ_MFMAS
#undef LZ_SCHED

  gemm_epilogue<TM, TN, EPI>(acc, C, R, M, ldc, m0, n0, wm, wn, lane, ra, rs);
}

template <int WM, int WN, int TM, int TN, int NS = 2>
static hipError_t launch_cfg(const void* A, const void* W, void* C, const void* R, int M, int N,
                             int K, int lda, int ldw, int ldc, int epi, int group_m,
                             const EpiArgs& ra, hipStream_t st) {
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  constexpr int LDS_BYTES = NS * (BM + BN) * ROW_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  if (N % BN != 0) return hipErrorInvalidValue;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
  const int threads = WM * WN * 64;
  EpiArgs ea = ra;
  ea.w_step_bytes = ra.w_blocked ? (unsigned long long)N * ROW_BYTES : (unsigned long long)ROW_BYTES;
  if (ra.w_blocked) ldw = BK;                       // rows of one K step are 128 bytes apart
  ea.sf_blocks_per_seq = (ea.sf_max_rows + threads - 1) / threads;
  const int side = ea.sf_z != nullptr ? ea.sf_blocks_per_seq * ea.sf_batch : 0;
  dim3 grid(tiles_m * tiles_n + side), block(threads);
#define LZ_GEMM(E)                                                                               \
  do {                                                                                           \
    auto kern = gemm_kernel<WM, WN, TM, TN, E, NS>;                                              \
    static bool attr_set = false;                                                                \
    if (!attr_set) {                                                                             \
      hipError_t e = hipFuncSetAttribute((const void*)kern,                                      \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES); \
      if (e != hipSuccess) return e;                                                             \
      attr_set = true;                                                                           \
    }                                                                                            \
    hipLaunchKernelGGL(kern, grid, block, LDS_BYTES, st, (const uint16_t*)A, (const uint16_t*)W, \
                       (uint16_t*)C, (const uint16_t*)R, M, N, K, lda, ldw, ldc, tiles_m,        \
                       tiles_n, group_m, ea);                                                    \
  } while (0)
  if (epi == EPI_STORE) LZ_GEMM(EPI_STORE);
  else if (epi == EPI_RESIDUAL) LZ_GEMM(EPI_RESIDUAL);
  else if (epi == EPI_SWIGLU) LZ_GEMM(EPI_SWIGLU);
  else if (epi == EPI_QKV_ROPE) {
    if ((TN * 32) % ra.head_dim != 0) return hipErrorInvalidValue;
    if (ra.head_dim == 64) LZ_GEMM(EPI_QKV_ROPE64);
    else if constexpr (TN >= 4) LZ_GEMM(EPI_QKV_ROPE128);
    else return hipErrorInvalidValue;
  }
  else return hipErrorInvalidValue;
#undef LZ_GEMM
  return hipGetLastError();
}

// The four-wave kernel addresses both operands with 32-bit byte offsets from a uniform base.
static bool operands_fit_32bit(int M, int N, int K, int lda, int ldw, bool w_blocked) {
  return (unsigned long long)M * lda * 2 < (1ull << 32) &&
         (unsigned long long)N * (w_blocked ? K : ldw) * 2 < (1ull << 32);
}

// Fewer tiles than workgroups, the same number on every XCD: a whole number S of workgroups per
// tile makes every range an exact 1/S of ONE tile, so that a workgroup has one piece, S - 1 of S
// leave a partial tile and the owner reads S - 1 (80 tiles: 240 workgroups, three per tile,
// instead of 256 ranges of which most straddle two tiles).  Taken when it keeps 3/4 of the CUs.
static bool pieces_align(int G, int tiles) {
  if (tiles >= G || tiles % 8 != 0) return false;
  const int per_xcd = tiles / 8, S = (G / 8) / per_xcd;
  return S >= 2 && S * per_xcd * 4 >= (G / 8) * 3;
}
int gemm_aligned_grid(int G, int tiles) {
  return pieces_align(G, tiles) ? 8 * ((G / 8) / (tiles / 8)) * (tiles / 8) : G;
}

// ------------------------------------------------------------------------------------------
// Stream-K on 128x128 tiles (4 waves of 64x64): for shapes whose tile count does not divide
// over the 256 CUs.  The (tile, K step) pairs are numbered tile-major and cut into G equal
// contiguous ranges, one per persistent workgroup (two fit on a CU).  A workgroup finishes
// every tile it covers completely through the normal epilogue; the at most two tiles it shares
// with a neighbour are written as fp32 partial sums into slot [g][0] (its first tile) or
// [g][1] (its last tile), and a second kernel adds the pieces of each shared tile in workgroup
// order (deterministic) and applies the epilogue.  No workgroup ever waits for another.
// ------------------------------------------------------------------------------------------
constexpr int SK_BM = 128, SK_BN = 128, SK_TILE_ELEMS = SK_BM * SK_BN;

__host__ __device__ inline long long sk_begin(int g, long long U, int G) { return (long long)g * U / G; }

template <int EPI>
__global__ void __launch_bounds__(256)
gemm_sk_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
               uint16_t* __restrict__ C, const uint16_t* __restrict__ R, float* __restrict__ partial,
               int M, int N, int K, int lda, int ldw, int ldc, int tiles_m, int tiles_n, int G,
               unsigned long long* __restrict__ ssq_out, size_t wstep,
               const int32_t* __restrict__ r_rows) {
  constexpr int WM = 2, WN = 2, TM = 2, TN = 2, NWAVES = 4;
  constexpr int BM = SK_BM, BN = SK_BN;
  constexpr int A_INSTR = BM / 8 / NWAVES, W_INSTR = BN / 8 / NWAVES;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // consecutive ranges on one XCD (ids are dealt round-robin over the 8 XCDs)
  const int g = (int)(blockIdx.x & 7) * (G >> 3) + (int)(blockIdx.x >> 3);
  const int KT = K / BK;
  const long long U = (long long)tiles_m * tiles_n * KT;
  const long long u0 = sk_begin(g, U, G), u1 = sk_begin(g + 1, U, G);
  if (u0 >= u1) return;
  const int first_tile = (int)(u0 / KT);

  uint32_t koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    koff[ks] = (uint32_t)(((ks * 2 + (lane >> 5)) ^ swz64(lane & 31)) * 16);
  const uint32_t a_row = (uint32_t)((wm * TM * 32 + (lane & 31)) * ROW_BYTES);
  const uint32_t w_row = (uint32_t)(BM * ROW_BYTES + (wn * TN * 32 + (lane & 31)) * ROW_BYTES);
  const int crow = lane >> 3;
  EpiArgs ra{};
  ra.ssq_out = ssq_out;
  ra.r_rows = r_rows;

  long long u = u0;
  while (u < u1) {
    const int tile = (int)(u / KT);
    const int ka = (int)(u - (long long)tile * KT);
    const int kb = (int)min((long long)KT, ka + (u1 - u));
    const int n_it = kb - ka;
    const int tile_m = tile % tiles_m, tile_n = tile / tiles_m;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    uint32_t a_off[A_INSTR], w_off[W_INSTR];
#pragma unroll
    for (int q = 0; q < A_INSTR; ++q) {
      const int tr = (wave * A_INSTR + q) * 8 + crow;
      const int cchunk = (lane & 7) ^ swz64(tr);
      int r = m0 + tr;
      r = r < M ? r : M - 1;
      a_off[q] = (uint32_t)(((size_t)r * lda + cchunk * 8) * 2);
    }
#pragma unroll
    for (int q = 0; q < W_INSTR; ++q) {
      const int tr = (wave * W_INSTR + q) * 8 + crow;
      const int cchunk = (lane & 7) ^ swz64(tr);
      int r = n0 + tr;
      r = r < N ? r : N - 1;
      w_off[q] = (uint32_t)(((size_t)r * ldw + cchunk * 8) * 2);
    }
    auto issue = [&](int stage, int kt) {
      char* sa = lds + stage * STAGE_BYTES + (wave * A_INSTR) * 1024;
      char* sw = lds + stage * STAGE_BYTES + BM * ROW_BYTES + (wave * W_INSTR) * 1024;
      const char* ga = (const char*)A + (size_t)kt * BK * 2;
      const char* gw = (const char*)W + (size_t)kt * wstep;
#pragma unroll
      for (int q = 0; q < A_INSTR; ++q) g2l16(ga + a_off[q], sa + q * 1024);
#pragma unroll
      for (int q = 0; q < W_INSTR; ++q) g2l16(gw + w_off[q], sw + q * 1024);
    };

    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    bf16x8_t af[2][TM], wf[2][TN];
#define LZ_LOAD_FRAGS(buf, st, ks)                                                            \
  do {                                                                                        \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                            \
        af[buf][i] = *(const bf16x8_t*)((st) + a_row + i * 32 * ROW_BYTES + koff[ks]);        \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
        wf[buf][j] = *(const bf16x8_t*)((st) + w_row + j * 32 * ROW_BYTES + koff[ks]);        \
  } while (0)
#define LZ_MFMAS(buf)                                                                         \
  do {                                                                                        \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                            \
      _Pragma("unroll") for (int j = 0; j < TN; ++j)                                          \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[buf][j], af[buf][i],           \
                                                            acc[i][j], 0, 0, 0);              \
  } while (0)
    issue(0, ka);
    if (n_it > 1) issue(1, ka + 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    LZ_LOAD_FRAGS(0, lds, 0);
    for (int it = 0; it < n_it; ++it) {
      const char* cur = lds + (it & 1) * STAGE_BYTES;
      const char* nxt = lds + ((it + 1) & 1) * STAGE_BYTES;
      LZ_LOAD_FRAGS(1, cur, 1);
      LZ_MFMAS(0);
      LZ_LOAD_FRAGS(0, cur, 2);
      LZ_MFMAS(1);
      LZ_LOAD_FRAGS(1, cur, 3);
      LZ_MFMAS(0);
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();
      if (it + 2 < n_it) issue(it & 1, ka + it + 2);
      if (it + 1 < n_it) LZ_LOAD_FRAGS(0, nxt, 0);
      LZ_MFMAS(1);
    }
#undef LZ_LOAD_FRAGS
#undef LZ_MFMAS
    if (ka == 0 && kb == KT) {
      gemm_epilogue<TM, TN, EPI>(acc, C, R, M, ldc, m0, n0, wm, wn, lane, ra);
    } else {
      // fp32 partial sums of this piece, tile-local row-major [128][128]
      float* dst = partial + ((size_t)g * 2 + (tile == first_tile ? 0 : 1)) * SK_TILE_ELEMS;
      const int tok_l = lane & 31, feat_l = 4 * (lane >> 5);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            float4 v = make_float4(acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2],
                                   acc[i][j][4 * q4 + 3]);
            *(float4*)(dst + ((wm * TM + i) * 32 + tok_l) * SK_BN + (wn * TN + j) * 32 + 8 * q4 +
                       feat_l) = v;
          }
    }
    u += n_it;
    __syncthreads();            // the next piece refills stage 0: everyone must be done reading
  }
}

// Adds the pieces of every tile that more than one workgroup worked on and applies the
// epilogue.  One workgroup per tile; tiles finished by a single workgroup return at once.
template <int EPI>
__global__ void __launch_bounds__(256)
gemm_sk_fixup_kernel(const float* __restrict__ partial, uint16_t* __restrict__ C,
                     const uint16_t* __restrict__ R, int M, int ldc, int tiles_m, int KT,
                     long long U, int G, unsigned long long* __restrict__ ssq_out,
                     const int32_t* __restrict__ r_rows) {
  const int tile = blockIdx.x;
  const long long ua = (long long)tile * KT, ub = ua + KT - 1;
  // owner(u) = largest g with sk_begin(g) <= u
  int g_first = (int)(ua * G / U), g_last = (int)(ub * G / U);
  while (g_first + 1 < G && sk_begin(g_first + 1, U, G) <= ua) ++g_first;
  while (g_first > 0 && sk_begin(g_first, U, G) > ua) --g_first;
  while (g_last + 1 < G && sk_begin(g_last + 1, U, G) <= ub) ++g_last;
  while (g_last > 0 && sk_begin(g_last, U, G) > ub) --g_last;
  if (g_first == g_last) return;
  // piece pointers are worked out by one thread per batch of 64 (the range arithmetic is
  // 64-bit division); one float4 per thread: blockIdx.y picks an 8-row slab of the tile
  constexpr int MAX_PIECES = 64;
  __shared__ const float* piece[MAX_PIECES];
  __shared__ int n_piece, g_next;
  const int tile_m = tile % tiles_m, tile_n = tile / tiles_m;
  const int m0 = tile_m * SK_BM, n0 = tile_n * SK_BN;
  const int r = blockIdx.y * 8 + (threadIdx.x >> 5), c4 = (threadIdx.x & 31) * 4;
  const int row = m0 + r;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (threadIdx.x == 0) g_next = g_first;
  __syncthreads();
  while (true) {
    if (threadIdx.x == 0) {
      int np = 0, g = g_next;
      for (; g <= g_last && np < MAX_PIECES; ++g) {
        const long long b0 = sk_begin(g, U, G), b1 = sk_begin(g + 1, U, G);
        if (b0 >= b1) continue;                                        // empty range
        const int slot = ((int)(b0 / KT) == tile) ? 0 : 1;
        piece[np++] = partial + ((size_t)g * 2 + slot) * SK_TILE_ELEMS;
      }
      n_piece = np;
      g_next = g;
    }
    __syncthreads();
    const int np = n_piece;
    const bool more = g_next <= g_last;
    if (row < M) {
      int p = 0;
      for (; p + 4 <= np; p += 4) {               // four loads in flight, summed in piece order
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *(const float4*)(piece[p + u] + r * SK_BN + c4);
#pragma unroll
        for (int u = 0; u < 4; ++u) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
      }
      for (; p < np; ++p) {
        const float4 v = *(const float4*)(piece[p] + r * SK_BN + c4);
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
      }
    }
    __syncthreads();
    if (!more) break;
  }
  if (row < M) {
    const size_t off = (size_t)row * ldc + n0 + c4;
    if (EPI == EPI_RESIDUAL) {
      const uint2 r2 = *(const uint2*)(R + (size_t)(r_rows != nullptr ? r_rows[row] : row) * ldc + n0 + c4);
      acc.x += bf16_lo(r2.x); acc.y += bf16_hi(r2.x);
      acc.z += bf16_lo(r2.y); acc.w += bf16_hi(r2.y);
    }
    uint2 w2;
    w2.x = pack_bf16(acc.x, acc.y);
    w2.y = pack_bf16(acc.z, acc.w);
    *(uint2*)(C + off) = w2;
    if (EPI == EPI_RESIDUAL && ssq_out != nullptr) {
      // a row is 32 consecutive lanes (half a wave, all of them past the row < M test together)
      const float a = bf16_lo(w2.x), b = bf16_hi(w2.x), c = bf16_lo(w2.y), e = bf16_hi(w2.y);
      float ss = a * a + b * b + c * c + e * e;
#pragma unroll
      for (int sh = 16; sh >= 1; sh >>= 1) ss += __shfl_xor(ss, sh, 64);
      if ((threadIdx.x & 31) == 0) atomicAdd(ssq_out + row, ssq_to_fixed(ss));
    }
  }
}

static_assert(SK_PART_BYTES == (size_t)SK_GRID * 2 * SK_TILE_ELEMS * sizeof(float), "partial tiles of the 128x128 stream-K form");
size_t gemm_workspace_bytes() { return SK_PART_BYTES + SK_TICKET_BYTES + PSK_FLAG_BYTES; }

static hipError_t launch_sk(const void* A, const void* W, void* C, const void* R, float* partial,
                            int M, int N, int K, int lda, int ldw, int ldc, int epi,
                            unsigned long long* ssq_out, bool w_blocked, const int32_t* r_rows,
                            hipStream_t st) {
  constexpr int LDS_BYTES = 2 * (SK_BM + SK_BN) * ROW_BYTES;
  const size_t wstep = w_blocked ? (size_t)N * ROW_BYTES : (size_t)ROW_BYTES;   // bytes from one K step of a row to the next
  if (w_blocked) ldw = BK;
  const int tiles_m = (M + SK_BM - 1) / SK_BM, tiles_n = N / SK_BN, KT = K / BK;
  const long long U = (long long)tiles_m * tiles_n * KT;
  // Workgroups: as many as are resident at once (two per CU), unless a whole number S of them per
  // tile, with S dividing the K steps, comes close to that: then every range is exactly 1/S of
  // one tile, a workgroup leaves one partial tile instead of two, and the fix-up reads that much
  // less (96 tiles at 355 rows: 384 workgroups, O projection 40.9 -> 36.2 us, down 70.4 -> 61.2).
  int G = SK_GRID;
  for (int S = SK_GRID / (tiles_m * tiles_n); S >= 2; --S)
    if (KT % S == 0) {
      if (tiles_m * tiles_n * S * 10 >= SK_GRID * 7) G = tiles_m * tiles_n * S;
      break;
    }
#define LZ_GEMM(E)                                                                               \
  do {                                                                                           \
    auto kern = gemm_sk_kernel<E>;                                                               \
    static bool attr_set = false;                                                                \
    if (!attr_set) {                                                                             \
      hipError_t e = hipFuncSetAttribute((const void*)kern,                                      \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES); \
      if (e != hipSuccess) return e;                                                             \
      attr_set = true;                                                                           \
    }                                                                                            \
    hipLaunchKernelGGL(kern, dim3(G), dim3(256), LDS_BYTES, st, (const uint16_t*)A,              \
                       (const uint16_t*)W, (uint16_t*)C, (const uint16_t*)R, partial, M, N, K,   \
                       lda, ldw, ldc, tiles_m, tiles_n, G, ssq_out, wstep, r_rows);              \
    hipError_t e = hipGetLastError();                                                            \
    if (e != hipSuccess) return e;                                                               \
    hipLaunchKernelGGL(gemm_sk_fixup_kernel<E>, dim3(tiles_m * tiles_n, 16), dim3(256), 0, st,   \
                       partial, (uint16_t*)C, (const uint16_t*)R, M, ldc, tiles_m, KT, U, G,     \
                       ssq_out, r_rows);                                                         \
  } while (0)
  if (epi == EPI_STORE) LZ_GEMM(EPI_STORE);
  else if (epi == EPI_RESIDUAL) LZ_GEMM(EPI_RESIDUAL);
  else return hipErrorInvalidValue;
#undef LZ_GEMM
  return hipGetLastError();
}

// W [N][K] -> K-step-major [K / 64][N][64]: one thread per 16-byte chunk.
__global__ void __launch_bounds__(256)
pack_kblock_kernel(const uint4* __restrict__ W, int ldw8, int N, size_t n_chunks, uint4* __restrict__ Wb) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n_chunks) return;
  const int c = (int)(e & 7);
  const size_t rn = e >> 3;                          // kt * N + n
  const size_t kt = rn / N, n = rn % N;
  Wb[e] = W[n * (size_t)ldw8 + kt * 8 + c];
}

hipError_t launch_pack_kblock(const void* W, int N, int K, int ldw, void* Wb, hipStream_t st) {
  if (N <= 0 || K <= 0 || K % BK != 0 || ldw % 8 != 0 || ldw < K || ((uintptr_t)W & 15) != 0 ||
      ((uintptr_t)Wb & 15) != 0)
    return hipErrorInvalidValue;
  const size_t n_chunks = (size_t)N * K / 8;
  hipLaunchKernelGGL(pack_kblock_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st,
                     (const uint4*)W, ldw / 8, N, n_chunks, (uint4*)Wb);
  return hipGetLastError();
}

unsigned* gemm_exchange_flags(void* sk_ws) { return (unsigned*)((char*)sk_ws + SK_PART_BYTES + SK_TICKET_BYTES); }

void* gemm_counter_region(void* sk_ws, size_t* bytes) {
  *bytes = SK_TICKET_BYTES + PSK_FLAG_BYTES;
  return (char*)sk_ws + SK_PART_BYTES;
}

hipError_t launch_gemm_counters_clear(void* sk_ws, hipStream_t st) {
  size_t bytes = 0;
  void* counters = gemm_counter_region(sk_ws, &bytes);
  return launch_fill_zero(counters, bytes, st);
}

__global__ void exchange_check_kernel(const unsigned* __restrict__ give_ups, int32_t* __restrict__ status) {
  if (*give_ups != 0u) atomicOr(status, ST_EXCHANGE);
}

hipError_t launch_gemm_exchange_check(const void* sk_ws, int32_t* status, hipStream_t st) {
  const unsigned* flags = (const unsigned*)((const char*)sk_ws + SK_PART_BYTES + SK_TICKET_BYTES);
  hipLaunchKernelGGL(exchange_check_kernel, dim3(1), dim3(1), 0, st, flags + 1023, status);
  return hipGetLastError();
}

int gemm_band_height(int M, int epilogue) {
  // Band height of the tile walk (tile rows that share a run of W column blocks in an XCD's L2).
  // Measured with cold K-step-major weights, 256x256 tiles of the four-wave kernel, us by band height:
  //   gate/up (86 column blocks)  1182 rows: 1: 194, 2: 190, 5: 184;  2364 rows: 1: 371, 5: 349, 10: 355
  //                               3376 rows: 2: 486, 4..6: 479, 7: 472, 14: 482
  //                               4916 rows: 2: 671, 4: 653, 5: 654, 16: 669;  8192 rows: 2: 1076, 3: 1068,
  //                               4: 1049, 5: 1055, 8: 1048, 32: 1114
  //   QKV (48 column blocks; up to 8192 rows with an epilogue that was 3 % slower)
  //                               1182 rows: 1: 116, 5: 107;  3376 rows: 1: 301, 3..6: 289-292, 14: 301
  //                               4916 rows: 3: 401, 5: 402, 16: 420;  8192 rows: 2: 652, 4: 630, 5: 636, 32: 715
  //   O and down projections: within 1 % from 3 to 8 (4 kept).
  //   packed batches              gate/up 14528 rows: 2: 1845, 3: 1840, 4: 1842, 8: 1855;  29053 rows: 2: 3631, 3: 3604,
  //                               4: 3629, 8: 3680;  41499 rows: 2: 5170, 3: 5180, 4: 5215, 5: 5185, 8: 5281
  //                               QKV 14528 rows: 2: 1098, 4: 1085, 8: 1108;  41499 rows: 2: 3117, 3: 3095, 4: 3133, 8: 3181
  // So: column by column below 8 tile rows, about half the tile rows up to 16 of them, 4 beyond.
  const int tm256 = (M + 255) / 256;
  const int tall = tm256 <= 11 ? 5 : tm256 <= 16 ? 7 : 4;
  return epilogue == EPI_QKV_ROPE || epilogue == EPI_SWIGLU ? (tm256 < 8 ? tm256 : tall) : 4;
}

// ---- which tile.  Every form's time is estimated, in microseconds, from what its tiles cost and the smallest
// estimate is taken.  The constants are those that lose least by the choice on 409 shapes of sixteen models
// (K 256 to 18944, N 256 to 57344, up to 16384 rows, cold weights): 0.7 % behind
// the best on average, and on 227 further shapes that took no part 0.6 %, at most 12 %.
//   * a launch: a fixed cost;
//   * a K step (64 elements) of a round of tiles, one per CU: under the power limit a chip that is
//     less than about 0.6 full runs at a higher clock (256 rows: 1.02 us a step alone, 1.37 on all CUs);
//   * the end of a tile, by epilogue: residual read, rotary table, SiLU;
//   * stream-K: the whole rounds, then the remaining tiles' steps shared out evenly; the exchange costs a
//     fixed part, a part for every piece the owner of a tile adds, and more when the pieces do not
//     align with tiles (a workgroup then has two pieces), the fewer tiles the more.
// (256 compute units, the whole part; where the runtime reports fewer the launcher's grid follows it and only the
// estimate is off.)
// Slower than the eight-wave tiles that stood here before: launches of about one round with K up to 1024,
// where the end of a tile on one wave per SIMD is not hidden (QKV 6384 x 2304 x 768 32 / 35 us, 9395 x 1536 x 512
// 27 / 29, 4188 x 3072 x 1024 35 / 38; residual 13264 x 1024 x 1024 36 / 39).
static const TileCost W4_COST[3] = {                // 256, 192, 128 rows; end: residual or none, rotary, SiLU * mul
    {6.47, 1.22, 1.10, {12.41, 13.15, 5.99}, 11.25, 3.55, 20.43},
    {4.58, 1.03, 0.99, {6.40, 8.88, 5.50}, 9.80, 3.21, 19.60},
    {4.83, 0.94, 0.94, {1.49, 4.26, 2.97}, 8.17, 2.54, 7.71}};
// 128x256 with three stages, one workgroup per CU (the rotary epilogue with 128-wide heads)
static const TileCost THREE_STAGES = {-1.75, 1.03, 0.93, {0.0, 8.12, 0.0}, 0.0, 0.0, 0.0};

double gemm_w4_cost(const TileCost& c, int rows, bool stream_k, int M, int N, int KT, int epi) {
  const long T = (long)((M + rows - 1) / rows) * (N / 256);
  const double end = c.end[epi == EPI_QKV_ROPE ? 1 : epi == EPI_SWIGLU ? 2 : 0];
  if (!stream_k) {
    const long rounds = (T + 255) / 256;
    const double fill = (double)(T - (rounds - 1) * 256) / 256.0;
    const double last = c.step_low + (c.step_full - c.step_low) * (fill > 0.6 ? (fill - 0.6) / 0.4 : 0.0);
    return c.launch + KT * ((double)(rounds - 1) * c.step_full + last) + (double)rounds * end;
  }
  const int G = T < 256 ? gemm_aligned_grid(256, (int)T) : 256;
  const long full = T / G, rest = T - full * G;
  double t = c.launch + (double)full * (KT * c.step_full + end);
  if (rest > 0) {
    const bool aligned = G % rest == 0 && rest % 8 == 0;
    const double pieces = (double)G / (double)rest, slack = 2.0 * (1.0 - (double)rest / G);
    t += (double)rest * KT / G * c.step_full + end + c.exchange +
         c.per_piece * (aligned ? pieces - 1.0 : (double)((G + rest - 1) / rest)) +
         (aligned ? 0.0 : c.ragged * (slack < 1.0 ? slack : 1.0));
  }
  return t;
}

// the configuration numbers of launch_gemm's switch
static int choose_tile(int M, int N, int K, int epi, int head_dim, bool w4_ok, bool stream_k_ok, bool split_ok) {
  const int KT = K / BK;
  const long t128 = (long)((M + 127) / 128) * (N / 128);
  // 128x128, two workgroups per CU: a round of 512 tiles, or of the first 256.  A wave of the rotary
  // epilogue with 128-wide heads must hold whole heads, so that tile is then cut into 32x128 waves.
  const long rounds = t128 / 512, left = t128 % 512;
  int cfg = epi == EPI_QKV_ROPE && head_dim == 128 ? 3 : 2;
  double best = 1.5 + KT * ((double)rounds * 1.28 + (left == 0 ? 0.0 : left <= 256 ? 0.79 : 1.28)) +
                (epi == EPI_QKV_ROPE ? 3.62 : epi == EPI_SWIGLU ? 3.77 : 2.71) * (double)(rounds + (left > 0));
  auto consider = [&](int c, double t) { if (t < best) { best = t; cfg = c; } };
  if (epi == EPI_QKV_ROPE && head_dim == 128 && N % 256 == 0)
    consider(13, gemm_w4_cost(THREE_STAGES, 128, false, M, N, KT, epi));
  // stream-K on 128x128 tiles with a second kernel that adds the pieces: few tiles and a long K
  if ((epi == EPI_STORE || epi == EPI_RESIDUAL) && split_ok && KT >= 32 && t128 <= 320)
    consider(6, 19.7 + 1.34 * (double)t128 * KT / 512.0);
  if (w4_ok) {
    static const int whole[3] = {5, 7, 15}, cut[3] = {9, 10, 16};
    for (int f = 0; f < 3; ++f) consider(whole[f], gemm_w4_cost(W4_COST[f], 256 - 64 * f, false, M, N, KT, epi));
    if (stream_k_ok)
      for (int f = 0; f < 3; ++f) consider(cut[f], gemm_w4_cost(W4_COST[f], 256 - 64 * f, true, M, N, KT, epi));
  }
  return cfg;
}

int gemm_config(int M, int N, int K, int epilogue, int head_dim, bool w4_ok, bool stream_k_ok, bool split_ok, bool stream_ok) {
  // few token rows, and the weight at hand in its streaming layout: gemm_stream.hip, up to where
  // the tile kernels become the better ones (see gemm_stream_takes; row-major, the same kernel is
  // 20 - 30 % slower).  A weight so wide that
  // one round of 192- or 256-row tiles keeps five eighths of the CUs is the exception from 289 rows on
  // (us, streaming / tiles: N 22016, K 4096 at 320 / 384 rows 81 / 78, 448 / 512 rows 94 / 88, 97 / 88;
  // N 28672 95 / 86, 109 / 102, 110 / 100; N 27648, K 5120 119 / 105, 133 / 126; at 288 rows and below,
  // and for N 16384, streaming is ahead: 106 / 101, 58 / 71, 56 / 63).
  const long t256 = (long)((M + 255) / 256) * (N / 256), t192 = (long)((M + 191) / 192) * (N / 256);
  const bool one_round = w4_ok && N > 20480 && M > 288 && M <= 512 &&
                         ((t192 >= 160 && t192 <= 256) || (t256 >= 160 && t256 <= 256));
  if (stream_ok && gemm_stream_takes(M, N, K) && !one_round) return 8;
  return choose_tile(M, N, K, epilogue, epilogue == EPI_QKV_ROPE ? head_dim : 0, w4_ok, stream_k_ok, split_ok);
}

hipError_t launch_gemm(const void* A, const void* W, void* C, const void* R, int M, int N, int K,
                       int lda, int ldw, int ldc, int epilogue, hipStream_t st, const EpiArgs* rope,
                       void* sk_ws, size_t sk_ws_bytes) {
  if (M <= 0) return hipSuccess;
  if (N % 128 != 0 || K % BK != 0) return hipErrorInvalidValue;
  // Bits 8..15 of `epilogue` force a tile configuration and bits 16..21 a band height (tuning
  // hook for measurements); 0 = choose here.
  int cfg = (epilogue >> 8) & 0xff, group_m = (epilogue >> 16) & 0x3f;
  const bool packed_flag = (epilogue & (1 << 30)) != 0, blocked_flag = (epilogue & (1 << 29)) != 0;
  epilogue &= 0xff;
  EpiArgs ra{};
  if (rope != nullptr) ra = *rope;
  if (packed_flag) ra.w_packed = 1;
  if (blocked_flag) ra.w_blocked = 1;
  if (epilogue == EPI_QKV_ROPE) {
    const int kvd = rope != nullptr ? (rope->kv_dim > 0 ? rope->kv_dim : rope->d_model) : 0;
    if (rope == nullptr || (rope->head_dim != 64 && rope->head_dim != 128) ||
        N != rope->d_model + 2 * kvd || rope->d_model % 128 != 0 || kvd % 128 != 0)
      return hipErrorInvalidValue;
  }
  if (group_m == 0) group_m = gemm_band_height(M, epilogue);
  const bool ws_ok = sk_ws != nullptr && sk_ws_bytes >= gemm_workspace_bytes();
  // The four-wave kernel: operands below 4 GB, rows of the outputs on 8-byte boundaries (its 16-byte accesses to them
  // need no more on this part, and cost the same: 3376 x 22016 x 4096 SiLU * mul 428 us on 16-byte boundaries, 423 on
  // 8-byte ones, 633 on the 128x128 tile; 8192 rows 966 / 963 / 1476; 3376 x 4096 x 11008 residual 225 / 224 / 336).
  const bool w4_ok = N % 256 == 0 && operands_fit_32bit(M, N, K, lda, ldw, ra.w_blocked != 0) &&
                     rows_on_boundaries(8, epilogue, C, R, ldc, ra);
  if (cfg == 0) {
    // (streaming: only for callers that keep the workspace's tickets zeroed)
    const bool stream_ok = (ra.skinny || ra.psk_ready) && ra.w_stream != nullptr && ws_ok && lda % 8 == 0;
    cfg = gemm_config(M, N, K, epilogue, ra.head_dim, w4_ok, ws_ok && ra.psk_ready, ws_ok && ra.a_rows == nullptr, stream_ok);
  }
  if (ra.w_packed && cfg != 8) return hipErrorInvalidValue;
  if (ra.w_blocked && cfg == 8 && ra.w_stream == nullptr) return hipErrorInvalidValue;
  // (forced, but with outputs that are not on 8-byte boundaries: the 128x128 tile)
  if ((cfg == 5 || cfg == 7 || cfg == 9 || cfg == 10 || cfg >= 14) && N % 256 == 0 && !w4_ok &&
      operands_fit_32bit(M, N, K, lda, ldw, ra.w_blocked != 0))
    cfg = epilogue == EPI_QKV_ROPE && ra.head_dim == 128 ? 3 : 2;
  switch (cfg) {
    case 2:                                             // 128x128, 4 waves of 64x64
            return launch_cfg<2, 2, 2, 2>(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, st);
    case 3:                                             // 128x128, 4 waves of 32x128 (whole heads per wave)
            return launch_cfg<4, 1, 1, 4>(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, st);
    case 13: if (N % 256) return hipErrorInvalidValue;  // 128x256, 8 waves of 32x128 (whole heads), three stages
            return launch_cfg<4, 2, 1, 4, 3>(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, st);
    case 4: if (N % 256) return hipErrorInvalidValue;   // 128x256, 4 waves of 64x128
            return launch_cfg<2, 2, 2, 4>(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, st);
    case 5: case 14:                                    // 256x256, 4 waves of 128x128
    case 7:                                             // 192x256, 4 waves of 96x128
    case 15:                                            // 128x256, 4 waves of 64x128
            return launch_gemm_w4(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, 0, nullptr, nullptr,
                                  cfg == 7 ? 192 : cfg == 15 ? 128 : 256, st);
    case 9: case 10: case 16:                           // the same three, stream-K
            if (sk_ws == nullptr || sk_ws_bytes < gemm_workspace_bytes() || !ra.psk_ready) return hipErrorInvalidValue;
            return launch_gemm_w4(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, group_m, ra, 1, (float*)sk_ws,
                                  gemm_exchange_flags(sk_ws), cfg == 10 ? 192 : cfg == 16 ? 128 : 256, st);
    case 6:                                             // 128x128 stream-K + fix-up
            if (sk_ws == nullptr || sk_ws_bytes < gemm_workspace_bytes()) return hipErrorInvalidValue;
            if (ra.a_rows != nullptr) return hipErrorInvalidValue;   // (no row indirection on its A operand)
            return launch_sk(A, W, C, R, (float*)sk_ws, M, N, K, lda, ldw, ldc, epilogue, ra.ssq_out,
                             ra.w_blocked != 0, ra.r_rows, st);
    case 8:                                             // few rows: weight streaming
            if (sk_ws == nullptr || sk_ws_bytes < gemm_workspace_bytes()) return hipErrorInvalidValue;
            if (ra.w_stream != nullptr && !ra.w_packed) {
              ra.w_packed = 1;
              W = ra.w_stream;
            }
            return launch_gemm_stream(A, W, C, R, M, N, K, lda, ldw, ldc, epilogue, ra, sk_ws, SK_PART_BYTES,
                                      (unsigned*)((char*)sk_ws + SK_PART_BYTES), SK_TICKET_BYTES / 4, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lz
