// Weight-streaming GEMM for few token rows (decoding steps, short prompts, the late stages of a
// pruned prefill): C[M,N] = A[M,K] W[N,K]^T with the epilogues of the tile kernels.
//
// What bounds it: every weight byte is read once and meets few rows, so the launch is a read of W
// from HBM.  A read-only stream reaches 6.3 - 6.6 TB/s on this card with non-temporal 16-byte loads
// into registers (5.8 without the hint; 90 MB and more), 5.4 TB/s for 34 MB.  So:
//   * W goes from HBM straight into MFMA operand registers (v_mfma_f32_16x16x32: lane l holds
//     feature l & 15, k elements 8*(l >> 4) ..): no LDS round trip, no barrier waits for it, two
//     units of 64 K elements per wave in flight (four gained nothing).  Non-temporal where one row
//     chunk covers the rows, i.e. nobody else reads those bytes: gate/up 33.8 -> 30.9 us at 16 rows.
//   * A (small, resident in the L2s) is shared by the CW waves that stand side by side, 32
//     features each: whole 128-byte row pieces into registers, from there into one of two LDS
//     stages, read back as operand fragments.  Read from global memory by every wave instead, in
//     64-byte pieces of 16 rows, it bounds the launch from 32 rows on (64 rows: 63 against 36 us).
//   * KW groups of waves take the K units in turn (a step = KW units, one barrier per step that
//     drains only LDS traffic); their sums meet in LDS once, in order.
//   * More rows than TM * 16 are further workgroups (`chunks`), 8 ids apart = on the same XCD, so
//     that the weights they share come from HBM once.
//   * Where the features alone make too few workgroups, `ks` of them share the K steps of a column
//     group: each leaves its sums in the workspace (agent-scope stores: they bypass the L2s, which
//     are not coherent with each other) and draws a ticket; the one that draws the last adds all of
//     them in split order, runs the epilogue and resets the ticket.  Nobody waits for anybody and
//     the order of every sum is fixed.
// Measured, cold weights, us at 1 / 16 / 32 / 64 / 96 / 128 rows (before: the kernels this one took
// over from, a weight-streaming kernel through LDS up to 16 rows, tile kernels beyond):
//   QKV (100 MB)      26 / 37 / 58 / 59 / 60 / 62  ->  19 / 20 / 21 / 24 / 30 / 31
//   O (34 MB)         12 / 18 / 25 / 26 / 28 / 29  ->  11 / 11 / 12 / 13 / 16 / 17
//   gate/up (180 MB)  42 / 53 / 59 / 59 / 59 / 60  ->  30 / 31 / 30 / 34 / 40 / 42
//   down (90 MB)      24 / 36 / 38 / 39 / 41 / 42  ->  18 / 19 / 19 / 22 / 28 / 30
// i.e. 6.0 TB/s for gate/up at one row; from 64 rows on the LDS reads of A and the products of a step
// (about 1100 and 900 cycles at 128 rows and four column waves) no longer hide under the stream.
//   * One K group alone (KW = 1: six, eight or twelve column waves) has nothing to add up and keeps its
//     sums in registers to the end, so that LDS holds the two A stages only.
#include "common.h"
#include "gemm_shared.h"

namespace lz {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// A wave's two blocks of 16 features: neighbours, or partners PD blocks apart where the epilogue
// pairs features (gate and up: 32 features; rotary halves: hd/2).
template <int EPI>
struct StreamCols {
  static constexpr bool PAIRED = EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE64 || EPI == EPI_QKV_ROPE128;
  static constexpr int PD = EPI == EPI_QKV_ROPE128 ? 4 : PAIRED ? 2 : 1;
  static __device__ __forceinline__ int block(int w, int c) {          // c-th block of column wave w
    return (w / PD) * 2 * PD + w % PD + c * PD;
  }
};

// How W is addressed, in bytes.  A group = 128 features.  Row-major W, or the sequential streams
// of launch_pack_stream (8 KB per group and 32 K elements, chunks of a row permuted).
struct StreamW {
  unsigned long long group;          // from one group to the next
  uint32_t bytes;                    // of a group, from its first to its last
  uint32_t unit, sub;                // from one 64-wide K unit to the next, from its first half to its second
  uint32_t row, block;               // from one feature to the next inside a block of 16, from block to block
  int swz;
};

__device__ __forceinline__ uint2 stream_pack4(float a, float b, float c, float d) {
  uint2 w2;
  w2.x = pack_bf16(a, b);
  w2.y = pack_bf16(c, d);
  return w2;
}

// One finished block of 16 tokens x 16 features (x) and, where the epilogue pairs features, its
// partner block (y): a lane holds features 4*l4 .. +3 of block gb for one token row.  Every lane of
// the wave calls it.  row_ssq: this row's sum-of-squares accumulator in LDS (EPI_RESIDUAL).
template <int EPI, int PD>
__device__ __forceinline__ void stream_block_out(floatx4_t x, floatx4_t y, int row, bool valid, int gb, int lane,
                                                 uint16_t* __restrict__ C, const uint16_t* __restrict__ R, int ldc,
                                                 const EpiArgs& ra, unsigned long long* row_ssq) {
  const int l4 = lane >> 4, col = gb * 16 + 4 * l4;
  if (EPI != EPI_RESIDUAL && ra.ssq_in != nullptr) {            // RMSNorm of the A operand's row
    const float rs = valid ? rsqrtf((float)ra.ssq_in[ra.a_rows != nullptr ? ra.a_rows[row] : row] * ra.ssq_mul + ra.eps) : 0.f;
    x *= rs;
    y *= rs;
  }
  if (EPI == EPI_STORE) {
    if (valid) *(uint2*)(C + (size_t)row * ldc + col) = stream_pack4(x[0], x[1], x[2], x[3]);
  } else if (EPI == EPI_RESIDUAL) {
    float ss = 0.f;
    if (valid) {
      const size_t rrow = ra.r_rows != nullptr ? (size_t)ra.r_rows[row] : (size_t)row;
      const uint2 r2 = *(const uint2*)(R + rrow * ldc + col);
      const uint2 w2 = stream_pack4(x[0] + bf16_lo(r2.x), x[1] + bf16_hi(r2.x), x[2] + bf16_lo(r2.y), x[3] + bf16_hi(r2.y));
      *(uint2*)(C + (size_t)row * ldc + col) = w2;
      const float a = bf16_lo(w2.x), b = bf16_hi(w2.x), e = bf16_lo(w2.y), f = bf16_hi(w2.y);
      ss = a * a + b * b + e * e + f * f;
    }
    if (ra.ssq_out != nullptr) {                    // (integer sums: their order does not matter)
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      if (lane < 16) atomicAdd(row_ssq, ssq_to_fixed(ss));
    }
  } else if (EPI == EPI_SWIGLU) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = x[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-x[e])) * y[e];
    // block gb of the 64-wide unit [gate | up] is block gb % 2 of the unit's 32 outputs
    if (valid) *(uint2*)(C + (size_t)row * ldc + (gb >> 2) * 32 + (gb & 1) * 16 + 4 * l4) = stream_pack4(v[0], v[1], v[2], v[3]);
  } else if (valid) {
    constexpr int half = PD * 16;                   // rotary partner: hd / 2 features on
    const int d = ra.d_model, kvd = ra.kv_dim > 0 ? ra.kv_dim : d;
    const int region = col < d ? 0 : col < d + kvd ? 1 : 2;
    const int rcol = col - (region == 0 ? 0 : region == 1 ? d : d + kvd), rld = region == 0 ? d : kvd;
    if (region == 2) {
      const uint2 p0 = stream_pack4(x[0], x[1], x[2], x[3]), p1 = stream_pack4(y[0], y[1], y[2], y[3]);
      if (ra.v != nullptr) {
        uint16_t* dst = ra.v + (size_t)row * rld + rcol;
        *(uint2*)dst = p0;
        *(uint2*)(dst + half) = p1;
      }
      if (ra.vt != nullptr) {                       // transposed: 16 lanes hold one feature of 16 tokens
        const size_t ld = (size_t)ra.vt_ld;
        uint16_t* f = ra.vt + (size_t)rcol * ld + (ra.vt_col != nullptr ? ra.vt_col[row] : row);
        f[0] = (uint16_t)p0.x; f[ld] = (uint16_t)(p0.x >> 16); f[2 * ld] = (uint16_t)p0.y; f[3 * ld] = (uint16_t)(p0.y >> 16);
        f += (size_t)half * ld;
        f[0] = (uint16_t)p1.x; f[ld] = (uint16_t)(p1.x >> 16); f[2 * ld] = (uint16_t)p1.y; f[3 * ld] = (uint16_t)(p1.y >> 16);
      }
    } else {
      const int orow = (region == 1 && ra.k_row != nullptr) ? ra.k_row[row] : row;
      uint16_t* dst = (region == 0 ? ra.q : ra.k) + (size_t)orow * rld + rcol;
      const float2* cs = ra.table + (size_t)ra.pos[row] * half + (rcol % (2 * half));
      float lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 k2 = cs[e];
        lo[e] = x[e] * k2.x - y[e] * k2.y;
        hi[e] = y[e] * k2.x + x[e] * k2.y;
      }
      *(uint2*)dst = stream_pack4(lo[0], lo[1], lo[2], lo[3]);
      *(uint2*)(dst + half) = stream_pack4(hi[0], hi[1], hi[2], hi[3]);
    }
  }
}

template <int EPI, int TM, int CW, int KW, bool NTW>
__global__ void __launch_bounds__(CW * KW * 64)
gemm_stream_kernel(const uint16_t* __restrict__ A, const char* __restrict__ W, uint16_t* __restrict__ C,
                       const uint16_t* __restrict__ R, int M, int units, int lda, int ldc, int col_waves, int col_wgs,
                       int chunks, int ks, int grid_main, StreamW sw, float* __restrict__ part,
                       unsigned* __restrict__ tickets, EpiArgs ra) {
  using Cols = StreamCols<EPI>;
  constexpr int NW = CW * KW, NT = NW * 64;
  constexpr int UNIT_BYTES = TM * 16 * 128, STAGE_BYTES = KW * UNIT_BYTES;
  constexpr int PIECES = STAGE_BYTES / 16, NA = (PIECES + NT - 1) / NT;   // 16-byte pieces of A per step, per thread
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if ((int)blockIdx.x >= grid_main) {              // side job (see EpiArgs): Eq. 1 scores
    const int sb = (int)blockIdx.x - grid_main;
    score_finish_block<true>(ra.sf_z, ra.sf_stat, ra.sf_s, ra.sf_cu, ra.sf_n_single, ra.sf_heads,
                             ra.sf_z_ld, ra.sf_cu_z, true, sb / ra.sf_blocks_per_seq,
                             (sb % ra.sf_blocks_per_seq) * (int)blockDim.x, (float2*)lds);
    return;
  }
  // consecutive ids go to consecutive XCDs: what shares a column group (row chunks: its weights;
  // splits: its partial sums) is 8 ids apart
  const int rest = (int)blockIdx.x >> 3, per = chunks * ks;
  const int wg = (rest / per) * 8 + ((int)blockIdx.x & 7);
  if (wg >= col_wgs) return;
  const int chunk = (rest % per) / ks, split = rest % ks;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cw = wave % CW, kw = wave / CW;
  const int l15 = lane & 15, l4 = lane >> 4;
  const int m0 = chunk * (TM * 16);
  const int rows = M - m0 < TM * 16 ? M - m0 : TM * 16;
  // this workgroup's steps: a contiguous share of the row's steps (KW units each)
  const int all_steps = (units + KW - 1) / KW;
  const int step0 = all_steps * split / ks, n = all_steps * (split + 1) / ks - step0;

  // both blocks of a wave lie in one group of 128 features
  // (a wave past the last column reads nothing: zeros)
  const bool has_cols = CW % 3 != 0 || wg * CW + cw < col_waves;
  const int g0 = Cols::block(wg * CW + cw, 0), g1 = Cols::block(wg * CW + cw, 1);
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(W + (has_cols ? (unsigned long long)(g0 >> 3) * sw.group : 0)), 0, has_cols ? (int)sw.bytes : 0, 0x00020000);
  const uint32_t w_lane = (uint32_t)l15 * sw.row + (uint32_t)(sw.swz ? (l4 ^ swz32(l15)) : l4) * 16;
  const uint32_t w_off[2] = {w_lane + (uint32_t)(g0 & 7) * sw.block, w_lane + (uint32_t)(g1 & 7) * sw.block};
  // A: piece j of a step is chunk j % 8 of row (j / 8) % (TM*16) of unit j / (TM*128)
  const char* ap[NA];
  uint32_t a_dst[NA];
  int a_unit[NA];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    const int jq = q * NT + (int)threadIdx.x, j = PIECES % NT == 0 || jq < PIECES ? jq : PIECES - 1;
    const int tr = (j >> 3) % (TM * 16), ch = j & 7;
    a_unit[q] = j / (TM * 128);
    int r = m0 + (tr < rows ? tr : rows - 1);       // rows past the edge: the last row again
    if (ra.a_rows != nullptr) r = ra.a_rows[r];
    ap[q] = (const char*)A + ((size_t)r * lda + ch * 8) * 2;
    a_dst[q] = (uint32_t)(a_unit[q] * UNIT_BYTES + tr * 128 + ((ch ^ swz64(tr)) * 16));
  }
  // step i of this workgroup.  Past its end, and for units past the row's end, W is read out of the
  // buffer's range (zeros, no memory traffic) and A at a valid place; A is staged as zeros then, so
  // that the products vanish without a branch around them (which costs the compiler its count of
  // the loads in flight: it waits for the newest where it need only wait for the oldest)
  u32x4_t wb[2][2][2];
  u32x4_t areg[2][NA];
  auto load_w = [&](int slot, int i) {
    const int u = (step0 + i) * KW + kw;
    const uint32_t wu = i < n && u < units ? (uint32_t)u * sw.unit : 0x80000000u;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        wb[slot][c][h] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (int)(w_off[c] + (wu + (uint32_t)h * sw.sub)), 0, NTW ? 2 : 0);
  };
  auto load_a = [&](int slot, int i) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int u = (step0 + (i < n ? i : n - 1)) * KW + a_unit[q];
      areg[slot][q] = *(const u32x4_t*)(ap[q] + (size_t)(u < units ? u : units - 1) * 128);
    }
  };
  auto put_a = [&](int slot, int stage, int i) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      *(u32x4_t*)(lds + stage * STAGE_BYTES + a_dst[q]) = (step0 + i) * KW + a_unit[q] < units ? areg[slot][q] : zero;
    }
  };
  floatx4_t acc[TM][2];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[t][c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  uint32_t f_off[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) f_off[h] = (uint32_t)(kw * UNIT_BYTES + l15 * 128 + (((h * 4 + l4) ^ swz64(l15)) * 16));

  // (barrier without draining the loads in flight: only this wave's LDS traffic is waited for)
#define LZ_STREAM_BARRIER() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")
  load_a(0, 0);
  load_w(0, 0);
  load_a(1, 1);
  load_w(1, 1);
  put_a(0, 0, 0);
  LZ_STREAM_BARRIER();
  auto step = [&](int s, int i) {
    load_a(s, i + 2);
    const char* st = lds + s * STAGE_BYTES;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        const bf16x8_t af = *(const bf16x8_t*)(st + t * 2048 + f_off[h]);
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(&wb[s][c][h]), af, acc[t][c], 0, 0, 0);
      }
    load_w(s, i + 2);
    put_a(s ^ 1, s ^ 1, i + 1);                     // the next step's A, loaded a step ago
    LZ_STREAM_BARRIER();
  };
  int i = 0;
  for (; i + 2 <= n; i += 2) {
    step(0, i);
    step(1, i + 1);
  }
  if (i < n) step(0, i);
#undef LZ_STREAM_BARRIER
  __syncthreads();

  // ---- the waves' partial sums, added over the KW groups in order (one group: they stay in registers)
  constexpr int RED_BYTES = KW > 1 ? NW * TM * 2048 : 0;
  floatx4_t* red = (floatx4_t*)lds;                 // [wave][row block][block][lane]
  unsigned long long* row_ssq = (unsigned long long*)(lds + RED_BYTES);
  if (KW > 1) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c) red[((wave * TM + t) * 2 + c) * 64 + lane] = acc[t][c];
  }
  if (EPI == EPI_RESIDUAL && threadIdx.x < TM * 16) row_ssq[threadIdx.x] = 0;
  if (ra.ssq_clear != nullptr && wg == 0 && split == 0 && threadIdx.x < TM * 16 && (int)threadIdx.x < rows)
    ra.ssq_clear[m0 + threadIdx.x] = 0;
  __syncthreads();
  const int jobs = (rows + 15) / 16 * CW;           // (row block, column wave), two blocks each
  auto total = [&](int job, int c) {
    const int t = job / CW, w0 = job % CW;
    floatx4_t v = red[((w0 * TM + t) * 2 + c) * 64 + lane];
#pragma unroll
    for (int g = 1; g < KW; ++g) v += red[(((g * CW + w0) * TM + t) * 2 + c) * 64 + lane];
    return v;
  };
  auto finish = [&](int t, int cg, const floatx4_t (&v)[2]) {
    const int row = m0 + t * 16 + l15;
    if (CW % 3 == 0 && cg >= col_waves) return;
    unsigned long long* rsq = row_ssq + t * 16 + l15;
    if (Cols::PAIRED) {
      stream_block_out<EPI, Cols::PD>(v[0], v[1], row, row < M, Cols::block(cg, 0), lane, C, R, ldc, ra, rsq);
    } else {
      stream_block_out<EPI, Cols::PD>(v[0], v[0], row, row < M, Cols::block(cg, 0), lane, C, R, ldc, ra, rsq);
      stream_block_out<EPI, Cols::PD>(v[1], v[1], row, row < M, Cols::block(cg, 1), lane, C, R, ldc, ra, rsq);
    }
  };
  const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(part + ((size_t)wg * chunks + chunk) * ks * (TM * CW * 512)), 0, ks * (TM * CW * 2048), 0x00020000);
  constexpr int AGENT = 16;                         // sc1: at the level every XCD sees
  if (ks > 1) {
    __shared__ unsigned last_flag;
    auto leave = [&](int job, int c, floatx4_t v) {
      __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4_t*>(&v), prsrc,
                                             split * (TM * CW * 2048) + (job * 2 + c) * 1024 + lane * 16, 0, AGENT);
    };
    if (KW > 1) {
      for (int job = wave; job < jobs; job += NW)
#pragma unroll
        for (int c = 0; c < 2; ++c) leave(job, c, total(job, c));
    } else {
#pragma unroll
      for (int t = 0; t < TM; ++t)
        if (t * 16 < rows) {
          leave(t * CW + cw, 0, acc[t][0]);
          leave(t * CW + cw, 1, acc[t][1]);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned* tk = tickets + wg * chunks + chunk;
      last_flag = __hip_atomic_fetch_add(tk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(ks - 1) ? 1u : 0u;
      if (last_flag) __hip_atomic_store(tk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);     // ready for the next launch
    }
    __syncthreads();
    if (last_flag == 0) return;
  }
  if (KW == 1 && ks == 1) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
      if (t * 16 < rows) finish(t, wg * CW + cw, acc[t]);
  } else {
    for (int job = wave; job < jobs; job += NW) {
      floatx4_t v[2];
      if (ks > 1) {
#pragma unroll
        for (int c = 0; c < 2; ++c) v[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        for (int sp = 0; sp < ks; sp += 4) {
          u32x4_t p[4][2];                          // (past the last split: out of range, zeros)
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c)
              p[u][c] = __builtin_amdgcn_raw_buffer_load_b128(prsrc, (sp + u) * (TM * CW * 2048) + (job * 2 + c) * 1024 + lane * 16, 0, AGENT);
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) v[c] += *reinterpret_cast<const floatx4_t*>(&p[u][c]);
        }
      } else {
        v[0] = total(job, 0);
        v[1] = total(job, 1);
      }
      finish(job / CW, wg * CW + job % CW, v);
    }
  }
  if (EPI == EPI_RESIDUAL && ra.ssq_out != nullptr) {
    __syncthreads();
    if ((int)threadIdx.x < rows) atomicAdd(ra.ssq_out + m0 + threadIdx.x, row_ssq[threadIdx.x]);
  }
}

template <int EPI, int TM, int CW, int KW, bool NTW>
static hipError_t launch_stream_cfg(const void* A, const void* W, void* C, const void* R, int M, int N, int K,
                                        int lda, int ldc, int ks, const StreamW& sw, const EpiArgs& ra, float* part,
                                        size_t part_bytes, unsigned* tickets, size_t ticket_count, hipStream_t st) {
  constexpr int NW = CW * KW;
  constexpr int LDS_STAGES = 2 * KW * TM * 2048, LDS_RED = (KW > 1 ? NW * TM * 2048 : 0) + TM * 128;
  constexpr int LDS_BYTES = LDS_STAGES > LDS_RED ? LDS_STAGES : LDS_RED;
  static_assert(LDS_BYTES <= 159 * 1024, "LDS of a CU");
  if (CW % 3 != 0 && N % (CW * 32) != 0) return hipErrorInvalidValue;
  const int col_waves = N / 32, col_wgs = (col_waves + CW - 1) / CW, chunks = (M + TM * 16 - 1) / (TM * 16);
  const int steps = (K / BK + KW - 1) / KW;
  if (ks > steps) ks = steps;                       // every split has at least one step
  if (ks < 1) ks = 1;
  while (ks > 1 && ((size_t)col_wgs * chunks * ks * (TM * CW * 2048) > part_bytes || (size_t)col_wgs * chunks > ticket_count)) --ks;
  const int grid_main = (col_wgs + 7) / 8 * 8 * chunks * ks;
  EpiArgs ea = ra;
  ea.sf_blocks_per_seq = (ea.sf_max_rows + NW * 64 - 1) / (NW * 64);
  const int side = ea.sf_z != nullptr ? ea.sf_blocks_per_seq * ea.sf_batch : 0;
  if (ea.sf_z != nullptr && ea.sf_heads * 8 > LDS_BYTES) return hipErrorInvalidValue;
  auto kern = gemm_stream_kernel<EPI, TM, CW, KW, NTW>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3(grid_main + side), dim3(NW * 64), LDS_BYTES, st, (const uint16_t*)A,
                     (const char*)W, (uint16_t*)C, (const uint16_t*)R, M, K / BK, lda, ldc, col_waves, col_wgs, chunks, ks,
                     grid_main, sw, part, tickets, ea);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Tile by shape: TM row blocks per chunk, CW x KW waves, ks K splits.  false: the tile kernels are
// the better ones there.
//   K up to 1024: two x four waves, in the shortest chunks whose workgroups go through the 32 CUs of
//     an XCD at once (those of a column group share an XCD), and up to 32 rows in any case.  Such a
//     launch is a chain of latencies, not a stream: one to four steps where the tile kernels make up
//     to sixteen.  In one round it is the faster one, in more the tile kernels are, whose tiles reread
//     A less and overlap one tile's stores with the next one's loads.  Measured, streaming / tile, us:
//       N 1536 K 512   640 rows, 30 workgroups per XCD  7.0 / 11.9;  1536 rows, 36  18.6 / 12.4
//       N 1024 K 1024  2048 rows, 32  14.6 / 16.6;  2560 rows, 40  24.5 / 17.3;  8192 rows  63 / 40
//       N 8192 K 1024 (gate/up)  256 rows, 32  12.9 / 18.2;  384 rows, 48  23.6 / 19.1;  2048 rows  95 / 37
//     3584 rows end it for narrow N too: N 512 K 960 15.9 / 15.9 at 3072 rows, 17.6 / 16.1 at 4096.
//     A K of one step (up to 256) goes on to two and a half rounds of the tallest chunks and 3200 rows,
//     so that a packed batch of so many rows has the bits of its prompts run alone (the sums come in
//     the same order whatever the rows).  There QKV, O, gate/up and down (N 768, 256, 1536, 256; K 256
//     and 768) take 8.8 + 5.4 + 11.0 + 7.3 / 9.8 + 9.3 + 7.6 + 13.6 at 2048 rows and, the price of it,
//     10.5 + 8.0 + 13.0 + 11.4 / 9.9 + 9.5 + 7.9 + 13.9 at 2560, 12.5 + 8.1 + 14.9 + 13.6 / 10.1 + 9.5
//     + 9.3 + 14.0 at 3072.
//   Longer K, up to 640 rows: of the tiles below the one whose estimated time is the shortest, among
//     those that need one workgroup per CU at most.  From 32 rows on a workgroup's own time counts
//     (its LDS reads and products do not hide under the stream), so what wins is the tile that spreads
//     the columns over the most of the 256 CUs: 22016 columns make 172 workgroups of four column
//     waves but 230 of three, 12288 columns in two splits 192 or 256.  In us:
//       a 64-wide K unit   TM * (0.035 + 0.0104 CW): measured 0.50 for 8 x 3, 0.55 8 x 4, 0.82 8 x 6,
//                          0.86 8 x 8, 1.25 8 x 12, 0.66 6 x 6, 1.08 6 x 12, 1.48 10 x 12
//       a launch           8, and for every further row chunk a tenth of the stream of W again
//       ks > 1             2, and the partial sums out and back at 4 TB/s
//     Up to 16 rows and for narrow N up to 256 rows the sweeps leave one tile each: two column waves
//     x four K groups (a wide N: four x two, 35.5 against 43.5 at one row), O in two chunks of 64 rows
//     (65 .. 128 rows: 16.5 / 17.3 in one of 128), down in one (28 / 30), four x two beyond.
//     Measured, cold weights, the same kernel with 4 or 8 column waves / best tile kernel -> now:
//       gate/up  64 rows 37 / 59 -> 34, 97: 43 / 59 -> 40, 176: 72 / 68 -> 52, 256: 67 / 85 -> 59,
//                355: 113 / 94 -> 79, 512: 123 / 107 -> 92, 613: - / 148 -> 107
//       gate/up  N 28672, eight row blocks on twelve waves from 289 rows (six make a fourth chunk, 300
//                workgroups): 289 rows - / 107 -> 92, 384: - / 110 -> 98
//       QKV      64 rows 26 / 59 -> 24, 128: 35 / 62 -> 31, 192: 41 / 62 -> 37, 256: 47 / 62 -> 42,
//                355: 72 / 72 -> 52, 512: - / 79 -> 62, 613: - / 91 -> 69
//       down     97 rows 30 / 41 -> 28, 512: 66 / 72 -> 62, 613: - / 91 -> 74;  O  613: - / 51 -> 40
//     The estimate is fitted to 4096-wide models.  Over 450 random shapes (K 1088 .. 29000, 17 .. 640
//     rows) its tile is ahead of the tile kernels or within 4 % (461 rows, N 2176, K 8064: 4 .. 8 % behind),
//     but for these, left out:
//       twelve waves unsplit on fewer than 168 CUs (N not a multiple of 256, where eight waves do not
//       fit): N 24704, 160 / 200 rows 78 / 87 against 69 / 72; N 15488, 257 rows 41 against 36
//       N 4352 .. 5120, K from 8192, 289 .. 384 rows: 57 .. 86 against 55 .. 80
//     and for these, on the next best tile instead:
//       one K group, N below 1024, K below 2048, 385 rows and more: 19 .. 26 against 17 .. 19, now 16 .. 18
//       twelve waves, K from 16384, up to 128 rows: N 8192 K 28672, 65 rows 111 against 103, now 82
//     768 rows and taller chunks (TM 12): the accumulators spill beside twelve waves (328 us).
// ks: every split has at least four steps.
// ------------------------------------------------------------------------------------------
struct StreamPlan {
  int tm, cw, kw, ks;
};

static bool stream_plan(int M, int N, int K, StreamPlan* p) {
  const int n64 = N / 64, units = K / BK;
  if (units <= 16) {
    auto per_xcd = [&](int tm) { return (long)((n64 + 7) / 8) * ((M + tm * 16 - 1) / (tm * 16)); };
    *p = StreamPlan{2, 2, 4, 1};
    if (M <= 32 || per_xcd(2) <= 32) return true;
    if (M > 3584) return false;
    if (per_xcd(4) <= 32) p->tm = 4;
    else if (per_xcd(8) <= 32) p->tm = 8;
    else return units <= 4 && M <= 3200 && per_xcd(8) <= 80;
    return true;
  }
  if (M > 640) return false;
  const bool narrow = n64 <= 64, wide = n64 > 256;
  const double stream = 2.0 * N * K / 5.6e6;
  double best = 0.0;
  auto consider = [&](int tm, int cw, int kw) {
    if (cw % 3 != 0 && N % (cw * 32) != 0) return;
    const int cols = (N / 32 + cw - 1) / cw, chunks = (M + tm * 16 - 1) / (tm * 16);
    const int per_xcd = (cols + 7) / 8 * chunks;     // (a column group's workgroups share an XCD of 32 CUs)
    int most = (units + kw - 1) / kw / 4;
    if (most < 1) most = 1;
    for (int ks = 1; ks <= most && (ks == 1 || per_xcd * ks <= 32); ++ks) {
      double us = 8.0 + (double)units / ks * tm * (0.035 + 0.0104 * cw) + 0.1 * stream * (chunks - 1);
      us *= (per_xcd * ks + 31) / 32;                // (more than one round of the CUs)
      if (ks > 1) us += 2.0 + 8.0 * M * N * ks / 4e6;
      if (best == 0.0 || us < 0.98 * best) {
        best = us;
        *p = StreamPlan{tm, cw, kw, ks};
      }
    }
  };
  if (M <= 64) {
    const int tm = M <= 32 ? 2 : 4;
    if (!wide) consider(tm, 2, 4);
    if (!narrow && (M > 16 || wide)) consider(tm, 4, 2);
    if (!narrow && M > 16) consider(tm, 3, 2);
  } else if (M <= 256 && narrow) {
    if (M > 128) consider(M <= 192 ? 6 : 8, 4, 2);
    else if (K < 8192) consider(4, 2, 4);
    else consider(8, 2, 4);
  } else {
    const int tm = M <= 96 || (M > 128 && M <= 192) || (M > 256 && M <= 384) ? 6 : 8;
    consider(tm, 4, 2);
    consider(tm, 3, 2);
    if (n64 >= 16 || units >= 32 || M <= 384) {
      consider(8, 8, 1);
      consider(tm, 6, 1);
      if (M > 128 || units < 256) consider(tm, 12, 1);
      if (M > 384) consider(10, 12, 1);
    }
    if (M > 256 && M <= 384 && n64 > 384) consider(8, 12, 1);   // (six blocks: four chunks, two rounds)
    // (beyond 128 rows only in one round: the tile kernels are better at several)
    const int cols = (N / 32 + p->cw - 1) / p->cw, chunks = (M + p->tm * 16 - 1) / (p->tm * 16);
    if (M > 128 && (cols + 7) / 8 * chunks > 32) return false;
    if (p->cw == 12 && p->ks == 1 && M <= 288 && cols * chunks < 168) return false;
    if (!narrow && n64 <= 80 && units >= 128 && M > 288 && M <= 384) return false;
  }
  return best > 0.0;
}

bool gemm_stream_takes(int M, int N, int K, int* tile) {
  StreamPlan p;
  if (M <= 0 || N <= 0 || K <= 0 || N % 128 != 0 || K % BK != 0 || !stream_plan(M, N, K, &p)) return false;
  if (tile != nullptr) {
    tile[0] = p.tm; tile[1] = p.cw; tile[2] = p.kw; tile[3] = p.ks;
  }
  return true;
}

hipError_t launch_gemm_stream(const void* A, const void* W, void* C, const void* R, int M, int N, int K, int lda,
                              int ldw, int ldc, int epi, const EpiArgs& ra, void* part, size_t part_bytes,
                              unsigned* tickets, size_t ticket_count, hipStream_t st) {
  StreamPlan p;
  if (M <= 0 || N % 128 != 0 || K % BK != 0 || !stream_plan(M, N, K, &p)) return hipErrorInvalidValue;
  if (lda % 8 != 0 || ldw % 8 != 0 || ((uintptr_t)A & 15) != 0 || ((uintptr_t)W & 15) != 0) return hipErrorInvalidValue;
  StreamW sw{};
  if (ra.w_packed) {
    sw.unit = 16384; sw.sub = 8192; sw.row = 64; sw.block = 1024; sw.swz = 1;
    sw.group = (unsigned long long)(K / 32) * 8192;
  } else {
    sw.unit = 128; sw.sub = 64; sw.row = (uint32_t)ldw * 2; sw.block = (uint32_t)ldw * 32;
    sw.group = (unsigned long long)ldw * 256;
  }
  const unsigned long long bytes = ra.w_packed ? sw.group : ((unsigned long long)127 * ldw + K) * 2;
  if (bytes >= 0x80000000ull) return hipErrorInvalidValue;      // (offsets past the end start there)
  sw.bytes = (uint32_t)bytes;
  const bool one_chunk = M <= p.tm * 16;
#define LZ_STREAM(E, TM, CW, KW, NTW)                                                                      \
  return launch_stream_cfg<E, TM, CW, KW, NTW>(A, W, C, R, M, N, K, lda, ldc, p.ks, sw, ra, (float*)part,  \
                                               part_bytes, tickets, ticket_count, st)
#define LZ_STREAM_TILE(E, TM, CW, KW)                                                                      \
  if (p.tm == TM && p.cw == CW) {                                                                          \
    if (one_chunk) LZ_STREAM(E, TM, CW, KW, true);                                                         \
    LZ_STREAM(E, TM, CW, KW, false);                                                                       \
  }
#define LZ_STREAM_EPI(E)                                                                                   \
  do {                                                                                                     \
    LZ_STREAM_TILE(E, 2, 2, 4)                                                                             \
    LZ_STREAM_TILE(E, 4, 2, 4)                                                                             \
    LZ_STREAM_TILE(E, 8, 2, 4)                                                                             \
    if (p.tm == 2 && p.cw == 3) LZ_STREAM(E, 2, 3, 2, true);                                               \
    if (p.tm == 4 && p.cw == 3) LZ_STREAM(E, 4, 3, 2, true);                                               \
    if (p.tm == 2 && p.cw == 4) LZ_STREAM(E, 2, 4, 2, true);                                               \
    if (p.tm == 4 && p.cw == 4) LZ_STREAM(E, 4, 4, 2, true);                                               \
    LZ_STREAM_TILE(E, 6, 3, 2)                                                                             \
    LZ_STREAM_TILE(E, 8, 3, 2)                                                                             \
    LZ_STREAM_TILE(E, 6, 4, 2)                                                                             \
    LZ_STREAM_TILE(E, 8, 4, 2)                                                                             \
    if (p.tm == 6 && p.cw == 6) LZ_STREAM(E, 6, 6, 1, false);                                              \
    if (p.tm == 8 && p.cw == 6) LZ_STREAM(E, 8, 6, 1, false);                                              \
    if (p.tm == 8 && p.cw == 8) LZ_STREAM(E, 8, 8, 1, false);                                              \
    if (p.tm == 6 && p.cw == 12) LZ_STREAM(E, 6, 12, 1, false);                                            \
    if (p.tm == 8 && p.cw == 12) LZ_STREAM(E, 8, 12, 1, false);                                            \
    if (p.tm == 10 && p.cw == 12) LZ_STREAM(E, 10, 12, 1, false);                                          \
    return hipErrorInvalidValue;                                                                           \
  } while (0)
  switch (epi) {
    case EPI_STORE: LZ_STREAM_EPI(EPI_STORE);
    case EPI_RESIDUAL: LZ_STREAM_EPI(EPI_RESIDUAL);
    case EPI_SWIGLU: LZ_STREAM_EPI(EPI_SWIGLU);
    case EPI_QKV_ROPE:
      if (ra.head_dim == 64) LZ_STREAM_EPI(EPI_QKV_ROPE64);
      else LZ_STREAM_EPI(EPI_QKV_ROPE128);
    default: return hipErrorInvalidValue;
  }
#undef LZ_STREAM_EPI
#undef LZ_STREAM_TILE
#undef LZ_STREAM
}

// ------------------------------------------------------------------------------------------
// W [N][K] -> sequential streams: for every group of 128 output features and every 32-element K
// step 8 KB (row r of the group at 64-byte row r, its 16-byte chunk c at position c ^ swz32(r)),
// groups outermost, steps contiguous: a 16-feature operand block of one step is 1 KB in one piece.
__global__ void __launch_bounds__(256)
pack_stream_kernel(const uint4* __restrict__ W, int ldw8, int ksteps, size_t n_chunks, uint4* __restrict__ Wp) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n_chunks) return;
  const int p = (int)(e & 63), t = (int)((e >> 6) & 7);
  const size_t gs = e >> 9;                          // group * ksteps + step
  const int step = (int)(gs % ksteps);
  const size_t group = gs / ksteps;
  const int tr = t * 16 + (p >> 2);
  const int lc = (p & 3) ^ swz32(tr);
  Wp[e] = W[(group * 128 + tr) * (size_t)ldw8 + step * 4 + lc];
}

hipError_t launch_pack_stream(const void* W, int N, int K, int ldw, void* Wp, hipStream_t st) {
  if (N <= 0 || K <= 0 || N % 128 != 0 || K % 32 != 0 || ldw % 8 != 0 || ldw < K ||
      ((uintptr_t)W & 15) != 0 || ((uintptr_t)Wp & 15) != 0)
    return hipErrorInvalidValue;
  const size_t n_chunks = (size_t)N * K / 8;
  hipLaunchKernelGGL(pack_stream_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st,
                     (const uint4*)W, ldw / 8, K / 32, n_chunks, (uint4*)Wp);
  return hipGetLastError();
}

}  // namespace lz
