// bf16 GEMM, tile of 32*TM x 256 (TM = 8: 256 rows) on FOUR waves, one per SIMD, each holding a
// 16*TM x 128 block of the product: 8*TM accumulator blocks of 16x16 = 256 registers, the
// accumulation half of the 512-register file that a lone wave of a SIMD has.  Against a tile on eight
// waves (two per SIMD, 64x128 each) a wave reads 16 operand fragments from LDS per
// 64 MFMAs instead of 12 per 32 -- a third less LDS traffic per FLOP, i.e. less of the power that
// sets this part's clock -- and there is one workgroup barrier per K step instead of four.
//
// There is no second wave to hide anything behind: the wave's own stream carries the LDS reads of
// the next half step and the global -> LDS copies between its MFMAs, one at a time and evenly: a CU
// takes 16 cycles for one 1 KB copy, so the 64 copies of a K step keep that path half busy when
// they are spread over the step's 2048 MFMA cycles and block the MFMA stream when they are not.
//
// LDS is a ring of FIVE slots of 32 KB (all of the 160 KB): element 2s is the A slab of K step s,
// element 2s + 1 its W slab, element e lives in slot e mod 5.  Half step C0(s) multiplies the first
// 32 of the step's 64 k (already in registers) while it reads the second 32 from LDS and copies the
// A slab of step s + 2 -- into the slot of W(s-1), last read in C0(s-1); C1(s) multiplies the second
// 32, reads the first 32 of step s + 1 and copies the W slab of step s + 2 into the slot of A(s).
// The one barrier of a step stands between C0(s) and C1(s): there every wave has read the last of
// step s, and everything but the A slab of step s + 2 has landed.
//
// The workgroups are persistent, one per CU, and the ring runs through: steps are counted over all of
// a workgroup's pieces of work, the copies of the next piece's first two steps ride in the last two of
// this one.  A wave's finished block goes out through LDS in whole rows, 16 at a time, in a part of
// the ring that is free just then (the W slab of the last step) and that only this wave's own copies
// refill, so the epilogue needs no barrier and the waves of a workgroup may drift through it.
//
// Measured, cold weights, against a tile on eight waves and the same MFMAs (us): 8192 rows QKV 663 -> 603, O
// 233 -> 205, gate/up 1154 -> 1013 (1.46 PFLOP/s), down 605 -> 504; 3376 rows gate/up 497 -> 441, down
// 247 -> 228.  A K step takes 1.38 us (1.55 PFLOP/s at the clock the power limit leaves); the rest is the
// residual read and the stores of all CUs at once: without them O takes 196, gate/up 988.
//
// Work of a workgroup: tiles g, g + G, ...; under the stream-K schedule only the first
// floor(T / G) * G tiles are taken whole, and the K steps of the remaining Rm < G tiles are cut into
// equal contiguous ranges, XCD by XCD (workgroup ids are dealt round-robin over the 8 XCDs and the tile
// walk gives XCD x the tiles whose id is x mod 8: neighbours in the walk keep sharing operand slabs
// through their L2).  A range is shorter than a tile: it is the END of one tile (that workgroup OWNS
// the tile) and / or the start or a middle piece of another.  A workgroup first does the piece it does
// not own -- fp32 partial sums to the workspace, lane-major, 16 bytes per lane and store, and a flag
// once they have reached the L2 -- and its own piece LAST; the owner adds the pieces in ascending K
// order (a fixed order: results do not depend on timing) and runs the normal epilogue.  The pieces
// of a tile belong to workgroups of one XCD, which share an L2, so the exchange needs no cache
// write-back or invalidation; that the dispatcher did put them on one XCD is checked, not assumed:
// the flag's value is 1 + the writer's XCC id (hardware register XCC_ID) and the owner compares it
// with its own.  Waits are bounded: if a flag never comes (it cannot, unless fewer than G workgroups
// fit on the device, which the launcher checks) or comes from another XCD, the owner gives up, counts
// the failure in the last word of the flag area -- the prefill turns a count into
// LAZYLLM_ST_EXCHANGE of its status word -- and finishes.  Flags are zero on entry; the owner resets
// the flags it consumed.
// (Instantiated in gemm_w4.hip and gemm_w4_fp8.hip: fifteen kernels each, compiled side by side.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"
#include "gemm_shared.h"

namespace lz {

constexpr unsigned W4_SPIN_LIMIT = 1u << 22;       // about a second of polling
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_t u32x4_at_8_t __attribute__((aligned(8)));
typedef uint16_t u16x8_t __attribute__((ext_vector_type(8)));
typedef u16x8_t u16x8_at_2_t __attribute__((aligned(2)));
constexpr int W4_SLOT = 256 * ROW_BYTES;

// The accumulators live in the accumulation registers a0 .. a255 by name: block (i, j) of a wave is
// a[4 * (i * TN + j)] and the three after it.  The compiler does not know (as variables, 64 tuples that
// pass through loops and branches end in copies and spills): nothing of its own may live there.
// LZ_ACC_RESERVE tells it so at every step, for values that live across one.  Between two of them nothing
// does, and some forms use all of the other 256 registers (8-bit residual, 192 and 256 rows), so the build
// looks: it reads the assembly of these kernels and fails if the compiler itself uses an accumulation
// register, spills a vector register, or writes an operand of a product right in front of it (build.py).
#define LZ_ACC_RESERVE() asm volatile("" ::: "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", \
  "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", \
  "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", \
  "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", \
  "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", \
  "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", \
  "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", \
  "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", \
  "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", \
  "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", \
  "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", \
  "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", \
  "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", \
  "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", \
  "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", \
  "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", \
  "a222", "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", \
  "a235", "a236", "a237", "a238", "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", \
  "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255")
// products of two operand fragments into block N / 4, from it or from zero
template <int N, bool ZERO>
__device__ __forceinline__ void acc_mfma(const bf16x8_t& w, const bf16x8_t& a) {
  if constexpr (ZERO) asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, 0" ::"v"(w), "v"(a), "n"(N), "n"(N + 3));
  else asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(w), "v"(a), "n"(N), "n"(N + 3));
}
template <int N, bool ZERO>
__device__ __forceinline__ void acc_mfma(const v8i_t& w, const v8i_t& a) {        // OFP8 E4M3, 128 k at once
  if constexpr (ZERO) asm volatile("v_mfma_f32_16x16x128_f8f6f4 a[%2:%3], %0, %1, 0" ::"v"(w), "v"(a), "n"(N), "n"(N + 3));
  else asm volatile("v_mfma_f32_16x16x128_f8f6f4 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(w), "v"(a), "n"(N), "n"(N + 3));
}
template <int N>
__device__ __forceinline__ floatx4_t acc_read() {
  float x, y, z, w;
  asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\t"
               "v_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]"
               : "=&v"(x), "=&v"(y), "=&v"(z), "=&v"(w) : "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));
  return floatx4_t{x, y, z, w};
}
template <int N>
__device__ __forceinline__ void acc_write(floatx4_t v) {
  asm volatile("v_accvgpr_write_b32 a[%4], %0\n\tv_accvgpr_write_b32 a[%5], %1\n\t"
               "v_accvgpr_write_b32 a[%6], %2\n\tv_accvgpr_write_b32 a[%7], %3"
               ::"v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));
}
// f(Int<0>), f(Int<1>), ... f(Int<N-1>): an unrolled loop whose index is a constant expression
template <int V> struct Int { static constexpr int value = V; };
template <int N, int B = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (B < N) { f(Int<B>{}); unrolled<N, B + 1>(f); }
}

// A and W: rows of lda / ldw BYTES, a K step (KT of them) is 128 bytes of a row: 64 bf16 or, F8, 128 codes.
// sa, sw (F8): scale of a row of A, of a feature of W.
template <int TM, int EPI, bool F8>
__global__ void __launch_bounds__(256)
gemm_w4_kernel(const char* __restrict__ A, const char* __restrict__ W, const float* __restrict__ sa,
               const float* __restrict__ sw, uint16_t* __restrict__ C, const uint16_t* __restrict__ R,
               int M, int KT, int lda, int ldw, int ldc, int tiles_m, int tiles_n, int group_m, int G,
               int stream_k, float* __restrict__ part, unsigned* __restrict__ flags, EpiArgs ra) {
  constexpr int WN = 2, TN = 8;
  constexpr int BM = 2 * TM * 16, BN = 2 * TN * 16;
  constexpr int NCA = BM / 32, NCW = BN / 32;      // copies per wave of an A / W slab
  constexpr int SLOT = W4_SLOT;
  constexpr int TILE_FLOATS = BM * BN;
  constexpr int RE = TM == 4 ? 2 : 3;              // MFMAs per fragment read
  static_assert(BM <= 256 && BN == 256, "a slab must fit a slot");
  static_assert((TM + TN) * RE <= TM * TN + RE - 1 && NCA * 1024 >= 16 * TN * 16 * 2, "reads fit a half step, 16 rows a wave's part of a slab");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if ((int)blockIdx.x >= G) {                      // side job (see EpiArgs): Eq. 1 scores
    const int sb = (int)blockIdx.x - G;
    score_finish_block<true>(ra.sf_z, ra.sf_stat, ra.sf_s, ra.sf_cu, ra.sf_n_single, ra.sf_heads,
                             ra.sf_z_ld, ra.sf_cu_z, true, sb / ra.sf_blocks_per_seq,
                             (sb % ra.sf_blocks_per_seq) * (int)blockDim.x, (float2*)lds);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int g = (int)blockIdx.x;

  // ---- this workgroup's pieces: n_whole tiles, then (stream-K) the piece of a tile it does not own,
  // then the end of the tile it owns
  const int T = tiles_m * tiles_n;
  const int full = T / G, Rm = T - full * G;
  const int xcd = g & 7, gi = g >> 3, GX = G >> 3;
  const int Rx = Rm > xcd ? (Rm - xcd + 7) >> 3 : 0;           // remainder tiles of this XCD
  const unsigned U = (unsigned)Rx * (unsigned)KT;  // (at most 32 x K / 64: the launcher bounds K)
  auto ubegin = [&](int i) { return (int)((unsigned)i * U / (unsigned)GX); };   // first unit of the XCD's i-th workgroup
  const int n_whole = stream_k ? full : (T - g + G - 1) / G;
  int own_tile = -1, own_ka = 0, oth_tile = -1, oth_ka = 0, oth_kb = 0;
  if (stream_k) {
    const int u0 = ubegin(gi), u1 = ubegin(gi + 1);
    if (u1 > u0) {
      const int ta = u0 / KT, tb = (u1 - 1) / KT;
      if (ta == tb && u1 != (ta + 1) * KT) { oth_tile = ta; oth_ka = u0 - ta * KT; oth_kb = u1 - ta * KT; }
      else { own_tile = ta; own_ka = u0 - ta * KT; }
      if (ta != tb) { oth_tile = tb; oth_ka = 0; oth_kb = u1 - tb * KT; }   // the start of tile ta + 1
    }
  }
  const int n_oth = oth_tile >= 0 ? 1 : 0;
  const int n_items = n_whole + n_oth + (own_tile >= 0 ? 1 : 0);
  if (n_items == 0) return;
  auto item = [&](int it, int& m0, int& n0, int& ka, int& kb) {
    int pid, tm, tn;
    if (it < n_whole) { pid = it * G + g; ka = 0; kb = KT; }
    else if (it < n_whole + n_oth) { pid = full * G + xcd + 8 * oth_tile; ka = oth_ka; kb = oth_kb; }
    else { pid = full * G + xcd + 8 * own_tile; ka = own_ka; kb = KT; }
    workgroup_tile(pid, tiles_m, tiles_n, group_m, tm, tn);
    m0 = tm * BM;
    n0 = tn * BN;
  };

  // ---- copy cursor: the K step whose slabs are copied next, two steps ahead of the products
  const uint32_t wstep32 = (uint32_t)ra.w_step_bytes;
  uint32_t a_off[NCA], w_off[NCW];
  int c_it = 0, c_kt, c_kb;
  auto cursor_to = [&](int it) {
    int m0, n0;
    item(it, m0, n0, c_kt, c_kb);
    const int crow = lane >> 3;
#pragma unroll
    for (int q = 0; q < NCA; ++q) {
      const int tr = (wave * NCA + q) * 8 + crow;
      const int cchunk = (lane & 7) ^ swz64(tr);
      int r = m0 + tr;
      r = r < M ? r : M - 1;                       // rows past the edge: re-read the last row
      if (ra.a_rows != nullptr) r = ra.a_rows[r];
      a_off[q] = (uint32_t)((size_t)r * lda + cchunk * 16);
    }
#pragma unroll
    for (int q = 0; q < NCW; ++q) {
      const int tr = (wave * NCW + q) * 8 + crow;
      const int cchunk = (lane & 7) ^ swz64(tr);
      w_off[q] = (uint32_t)((size_t)(n0 + tr) * ldw + cchunk * 16);
    }
  };
  auto cursor_next = [&]() {                       // (past the last step: stays, a harmless re-copy)
    if (c_kt + 1 < c_kb) ++c_kt;
    else if (c_it + 1 < n_items) cursor_to(++c_it);
  };
  // one of the wave's copies of a slab (uniform base + 32-bit lane offset; the launcher checks
  // that both operands span less than 4 GB)
  auto copy_a = [&](uint32_t slot, int q) {
    const char* base = A + (uint32_t)c_kt * (uint32_t)ROW_BYTES;
    g2l16(base + a_off[q], lds + slot + (wave * NCA + q) * 1024);
  };
  auto copy_w = [&](uint32_t slot, int q) {
    const char* base = W + (uint32_t)c_kt * wstep32;
    g2l16(base + w_off[q], lds + slot + (wave * NCW + q) * 1024);
  };

  // MFMA operand addresses: row (l & 15) of a 16-row block, chunk 4 * half + (l >> 4)
  uint32_t aoff[2], woff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t k = (uint32_t)(((h * 4 + (lane >> 4)) ^ swz64(lane & 15)) * 16);
    aoff[h] = (uint32_t)((wm * TM * 16 + (lane & 15)) * ROW_BYTES) + k;
    woff[h] = (uint32_t)((wn * TN * 16 + (lane & 15)) * ROW_BYTES) + k;
  }
  // the fragment reads of a half step, in the order in which its MFMAs want them
#define LZ_READ(buf, la, lw, h, n)                                                             \
  do {                                                                                         \
    if ((n) == 0) wf[buf][0] = *(const bf16x8_t*)(lds + (lw) + woff[h]);                       \
    else if ((n) <= TM) af[buf][(n)-1] = *(const bf16x8_t*)(lds + (la) + aoff[h] + ((n)-1) * 16 * ROW_BYTES); \
    else wf[buf][(n)-TM] = *(const bf16x8_t*)(lds + (lw) + woff[h] + ((n)-TM) * 16 * ROW_BYTES); \
  } while (0)
  // TM * TN MFMAs on fragments `buf` (ZERO: from a zero accumulator); behind every RE-th a fragment
  // read of the next half step (buffer `nb`) until they are through, and the nc copies evenly.  The order is
  // the program's: nothing is scheduled across a slot.  RUN = false: reads and copies only.
#define LZ_HALF(ZERO, RUN, buf, nb, la, lw, h, copy, nc, slot)                                 \
  unrolled<TM * TN>([&](auto nn) {                                                             \
    constexpr int n = decltype(nn)::value, j = n / TM, i = (j & 1) ? TM - 1 - n % TM : n % TM; \
    if constexpr (RUN) acc_mfma<4 * (i * TN + j), ZERO>(wf[buf][j], af[buf][i]);               \
    if constexpr (n % RE == 0 && n / RE < TM + TN) LZ_READ(nb, la, lw, h, n / RE);             \
    constexpr int CE = TM * TN / (nc);                                                         \
    if constexpr (n % CE == CE / 2 && n / CE < (nc)) copy(slot, n / CE);                       \
    __builtin_amdgcn_sched_barrier(0);                                                         \
  })
  // The 8-bit form multiplies 128 k at once, so its half steps are the left and the right four columns of
  // blocks: in the first, the rest of the step's fragments are read (the last row block of A, the
  // right half of W), in the second each row block's fragment of the next step right behind its last
  // use, and the left half of W.  Reads and copies stand where those of the 16-bit form do, between
  // the same two barriers.
#define LZ_READ8(dst, base, off, n)                                                            \
  dst = __builtin_shufflevector(*(const v4i_t*)(lds + (base) + off[0] + (n) * 16 * ROW_BYTES), \
                                *(const v4i_t*)(lds + (base) + off[1] + (n) * 16 * ROW_BYTES), 0, 1, 2, 3, 4, 5, 6, 7)
#define LZ_HALF8(ZERO, RUN, right, la_, lw_, copy, nc, slot)                                   \
  unrolled<TM * TN / 2>([&](auto nn) {                                                         \
    constexpr int n = decltype(nn)::value, i = n / 4, jj = (i & 1) ? 3 - n % 4 : n % 4;        \
    if constexpr (RUN) acc_mfma<4 * (i * TN + 4 * (right) + jj), ZERO>(f8w[right][jj], f8a[i]); \
    if constexpr (!(right) && n == 0) LZ_READ8(f8a[TM - 1], la_, aoff, TM - 1);                \
    if constexpr (!(right) && n % 4 == 3 && n / 4 < 4) LZ_READ8(f8w[1][n / 4], lw_, woff, 4 + n / 4); \
    if constexpr ((right) && n % 4 == 3 && i < TM - 1) LZ_READ8(f8a[i], la_, aoff, i);         \
    if constexpr ((right) && n % 4 == 1 && n / 4 < 4) LZ_READ8(f8w[0][n / 4], lw_, woff, n / 4); \
    constexpr int CE = TM * TN / 2 / (nc);                                                     \
    if constexpr (n % CE == CE / 2 && n / CE < (nc)) copy(slot, n / CE);                       \
    __builtin_amdgcn_sched_barrier(0);                                                         \
  })
#define LZ_STEP(ZERO, RUN)                                                                     \
  do {                                                                                         \
    if constexpr (F8) LZ_HALF8(ZERO, RUN, 0, la, lw, copy_a, NCA, next_slot(la, 4));           \
    else LZ_HALF(ZERO, RUN, 0, 1, la, lw, 1, copy_a, NCA, next_slot(la, 4));                   \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NCA) : "memory");         \
    __builtin_amdgcn_sched_barrier(0);                                                         \
    const uint32_t freed = la;                                                                 \
    stage_slot = lw;                                                                           \
    la = next_slot(la, 2);                                                                     \
    lw = next_slot(lw, 2);                                                                     \
    if constexpr (F8) LZ_HALF8(ZERO, RUN, 1, la, lw, copy_w, NCW, freed);                      \
    else LZ_HALF(0, RUN, 1, 0, la, lw, 0, copy_w, NCW, freed);                                 \
    cursor_next();                                                                             \
    LZ_ACC_RESERVE();                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                         \
  } while (0)

  auto next_slot = [](uint32_t s, uint32_t by) { s += by * SLOT; return s >= 5 * SLOT ? s - 5 * SLOT : s; };
  cursor_to(0);
#pragma unroll
  for (int q = 0; q < NCA; ++q) copy_a(0, q);
#pragma unroll
  for (int q = 0; q < NCW; ++q) copy_w(SLOT, q);
  cursor_next();
#pragma unroll
  for (int q = 0; q < NCA; ++q) copy_a(2 * SLOT, q);
#pragma unroll
  for (int q = 0; q < NCW; ++q) copy_w(3 * SLOT, q);
  cursor_next();
  uint32_t la = 0, lw = SLOT, stage_slot = 0;      // slots of the current step; of the last step's W slab
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NCA + NCW) : "memory");
  __builtin_amdgcn_sched_barrier(0);

  for (int it = 0; it < n_items; ++it) {
    int m0, n0, ka, kb;
    item(it, m0, n0, ka, kb);
    LZ_ACC_RESERVE();
    // (the last half step of the piece before has read these fragments too: reading them again costs
    // some hundred cycles a tile, keeping them through the epilogue 64 registers that it needs)
    bf16x8_t af[2][TM], wf[2][TN];
    v8i_t f8a[TM], f8w[2][4];
    if constexpr (F8) {
#pragma unroll
      for (int n = 0; n < TM - 1; ++n) LZ_READ8(f8a[n], la, aoff, n);
#pragma unroll
      for (int n = 0; n < 4; ++n) LZ_READ8(f8w[0][n], lw, woff, n);
    } else {
#pragma unroll
      for (int n = 0; n < TM + TN; ++n) LZ_READ(0, la, lw, 0, n);
    }
    unsigned long long ssq[TM];                    // of this lane's rows: fetched here, turned into 1/rms below
    float rs[TM];
    float rowscale[TM];
    int pos[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = m0 + (wm * TM + i) * 16 + (lane & 15), rc = row < M ? row : M - 1;
      if (EPI != EPI_RESIDUAL && ra.ssq_in != nullptr) ssq[i] = ra.ssq_in[ra.a_rows != nullptr ? ra.a_rows[rc] : rc];
      if (EPI == EPI_QKV_ROPE64 || EPI == EPI_QKV_ROPE128) pos[i] = ra.pos[rc];
      if (F8) rowscale[i] = sa[rc];
    }
    const bool gives = it >= n_whole && it - n_whole < n_oth;  // a piece of somebody else's tile
    const bool takes = it >= n_whole && !gives && own_ka > 0;  // the end of a tile of several pieces
    // the tile's other pieces belong to this XCD's workgroups i_first .. gi-1 (ids xcd + 8 i)
    int i_first = gi;
    if (takes)
      while (i_first > 0 && ubegin(i_first) > own_tile * KT) --i_first;
    const unsigned my_flag = 1u + (unsigned)__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);
    auto give_done = [&]() {
      // Every wave's stores have reached the L2 (vmcnt), then the flag goes up.  The reader sits on
      // the same XCD, behind the same L2, so there is nothing to write back or to invalidate (a
      // release fence writes the whole L2 back and an acquire fence empties it for everybody on
      // the XCD, 4-8 us per launch).
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      if (threadIdx.x == 0) __hip_atomic_store(flags + g, my_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto take_done = [&]() {
      asm volatile("s_barrier" ::: "memory");                 // every wave has seen the flags
      if (threadIdx.x == 0)
        for (int ip = i_first; ip < gi; ++ip)
          __hip_atomic_store(flags + xcd + 8 * ip, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto wait_for_pieces = [&]() -> bool {
      bool failed = false;
      for (int ip = i_first; ip < gi; ++ip) {
        if (ubegin(ip + 1) <= ubegin(ip)) continue;           // an empty range wrote nothing
        unsigned spins = 0, seen;
        while ((seen = __hip_atomic_load(flags + xcd + 8 * ip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
          __builtin_amdgcn_s_sleep(8);
          if (++spins >= W4_SPIN_LIMIT) { failed = true; break; }
        }
        if (seen != 0u && seen != my_flag) failed = true;     // written behind another L2: not visible here
      }
      if (failed && lane == 0) atomicAdd(flags + 1023, 1u);   // (the last word counts give-ups)
      // (the flags are read with relaxed atomics, which do not keep the loads of the pieces behind them)
      asm volatile("" ::: "memory");
      return !failed;
    };
    if (m0 + wm * TM * 16 >= M) {
      // all of this wave's rows are past M: it reads and copies its share and keeps the barriers, but runs
      // no MFMA -- the part is power-limited, matrix work on padding would lower everybody's clock
      for (int kt = ka; kt < kb; ++kt) LZ_STEP(false, false);
      if (gives) give_done();
      if (takes) {
        wait_for_pieces();                                    // (the flags are reset below: not before they are up)
        take_done();
      }
      continue;
    }
    LZ_STEP(true, true);
    if (EPI != EPI_RESIDUAL && ra.ssq_in != nullptr) {
#pragma unroll
      for (int i = 0; i < TM; ++i) rs[i] = rsqrtf((float)ssq[i] * ra.ssq_mul + ra.eps);
    }
    for (int kt = ka + 1; kt < kb; ++kt) LZ_STEP(false, true);
    // the results of the last MFMAs are waited for (16 cycles and what the register file needs) before
    // anything reads them: the compiler does not see the dependency
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // (the lane number through an empty asm: per-lane addresses of the parts below are then made here, not
    // kept in registers through the K loops)
    int el = lane;
    asm volatile("" : "+v"(el));
    if (gives) {
      // ---- partial sums to slot g, then the flag
      float4* dst = (float4*)(part + (size_t)g * TILE_FLOATS) + (size_t)wave * (TM * TN) * 64 + el;
      unrolled<TM * TN>([&](auto nn) {
        constexpr int n = decltype(nn)::value;
        const floatx4_t x = acc_read<4 * n>();
        dst[n * 64] = make_float4(x[0], x[1], x[2], x[3]);
      });
      give_done();
      continue;
    }
    if (takes) {
      if (wait_for_pieces()) {
        for (int ip = i_first; ip < gi; ++ip) {               // ascending K order
          if (ubegin(ip + 1) <= ubegin(ip)) continue;
          const float4* src = (const float4*)(part + (size_t)(xcd + 8 * ip) * TILE_FLOATS) + (size_t)wave * (TM * TN) * 64 + el;
          constexpr int NB = TM * TN, BATCH = 16;             // 64 registers per round trip
          static_assert(NB % BATCH == 0, "blocks are fetched in batches");
          unrolled<NB / BATCH>([&](auto bb) {
            constexpr int b0 = decltype(bb)::value * BATCH;
            float4 v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) v[u] = src[(b0 + u) * 64];
            unrolled<BATCH>([&](auto uu) {
              constexpr int u = decltype(uu)::value;
              acc_write<4 * (b0 + u)>(acc_read<4 * (b0 + u)>() + floatx4_t{v[u].x, v[u].y, v[u].z, v[u].w});
            });
            LZ_ACC_RESERVE();
            __builtin_amdgcn_sched_barrier(0);
          });
        }
      }
      take_done();
    }

    // ---- epilogue: 16 rows at a time, from the MFMA layout (a lane holds token l & 15 and, of each
    // block of 16 features, the four from 4 * (l >> 4) on) through the wave's own part of the free
    // slot into whole rows, stored 16 bytes per lane
    constexpr bool ROPE = EPI == EPI_QKV_ROPE64 || EPI == EPI_QKV_ROPE128;
    constexpr int WCOLS = EPI == EPI_SWIGLU ? TN * 8 : TN * 16;           // output columns of the wave
    constexpr int NCH = WCOLS / 8;                                        // 16-byte chunks per row
    constexpr int RPI = 64 / NCH, NST = 16 / RPI;                         // rows per store, stores per 16 rows
    char* const sl = lds + stage_slot + wave * NCA * 1024;
    const int tok = el & 15, feat = 4 * (el >> 4);
    const int srow = el / NCH, schunk = el % NCH;
    // byte offset of element column c (a multiple of 4) of row r in the staged rows
    auto stage_at = [&](int r, int c) -> uint32_t {
      return (uint32_t)(r * (NCH * 16) + (((c >> 3) ^ (NCH == 16 ? r : (r >> 1) & 7)) << 4) + ((c & 7) << 1));
    };
    const int col0 = n0 + wn * TN * 16;
    const int d = ra.d_model, kvd = ra.kv_dim > 0 ? ra.kv_dim : d;
    const int region = !ROPE ? 0 : col0 < d ? 0 : col0 < d + kvd ? 1 : 2;  // q, k, v (uniform per wave)
    const int rcol0 = col0 - (region == 0 ? 0 : region == 1 ? d : d + kvd);
    uint16_t* const obase = !ROPE ? C + (EPI == EPI_SWIGLU ? col0 / 2 : col0)
                            : (region == 0 ? ra.q : region == 1 ? ra.k : ra.v) + rcol0;
    const int old = !ROPE ? ldc : region == 0 ? d : kvd;
    const int row0 = m0 + wm * TM * 16;
    // a wave's LDS accesses complete in order, so what it wrote is there when it reads: only the
    // compiler has to keep the order
#define LZ_LDS_ORDER() asm volatile("" ::: "memory")
    constexpr int RAHEAD = F8 ? 3 : 4;                    // residual rows are fetched this many blocks ahead
    u32x4_t rr[RAHEAD][NST];
    auto fetch_residual = [&](auto ii) {
      constexpr int i = decltype(ii)::value;
#pragma unroll
      for (int s = 0; s < NST; ++s) {
        int r = row0 + i * 16 + s * RPI + srow;
        r = r < M ? r : M - 1;
        if (ra.r_rows != nullptr) r = ra.r_rows[r];
        rr[i % RAHEAD][s] = *(const u32x4_at_8_t*)(R + (size_t)r * ldc + col0 + schunk * 8);
      }
    };
    if (EPI == EPI_RESIDUAL) {
      unrolled<RAHEAD>(fetch_residual);
    }
    constexpr int hd = EPI == EPI_QKV_ROPE64 ? 64 : 128, half = hd >> 1, HQ = half / 16;
    float4 tb[2][HQ][2];                           // rotary table of the rows of a block, one block ahead
    auto fetch_table = [&](auto ii) {
      constexpr int i = decltype(ii)::value;
      const float2* cs = ra.table + (size_t)pos[i] * half + feat;
#pragma unroll
      for (int q = 0; q < HQ; ++q) {
        tb[i & 1][q][0] = *(const float4*)(cs + q * 16);
        tb[i & 1][q][1] = *(const float4*)(cs + q * 16 + 2);
      }
    };
    floatx4_t colscale[F8 ? TN : 1];               // of this lane's features
    if constexpr (F8) {
#pragma unroll
      for (int j = 0; j < TN; ++j) colscale[j] = *(const floatx4_t*)(sw + col0 + 16 * j + feat);
    }
    // block i of 16 rows; VPART: the columns are V's
    auto put_rows = [&](auto ii, auto vv) {
      constexpr int i = decltype(ii)::value;
      constexpr bool VPART = decltype(vv)::value != 0;
      const int row = row0 + i * 16 + tok;
      const bool valid = row < M;
      if (row0 + i * 16 >= M) return;              // (uniform)
      LZ_ACC_RESERVE();
      floatx4_t x[TN];
      unrolled<TN>([&](auto jj) { constexpr int j = decltype(jj)::value; x[j] = acc_read<4 * (i * TN + j)>(); });
      if (ra.ssq_clear != nullptr && n0 == 0 && wn == 0 && el < 16 && valid) ra.ssq_clear[row] = 0;
      if constexpr (F8) {
#pragma unroll
        for (int j = 0; j < TN; ++j) x[j] *= rowscale[i] * colscale[j];
      }
      if (EPI != EPI_RESIDUAL && ra.ssq_in != nullptr) {
        // RMSNorm of the A operand's row, applied to the product
#pragma unroll
        for (int j = 0; j < TN; ++j) x[j] *= rs[i];
      }
      auto put = [&](int c, uint2 w2) {            // four features from column c of the wave's output on
        *(uint2*)(sl + stage_at(tok, c)) = w2;
      };
      if constexpr (ROPE && !VPART) {
        if constexpr (i + 1 < TM) fetch_table(Int<i + 1>{});
#pragma unroll
        for (int q = 0; q < TN; ++q) {
          if ((q / HQ) & 1) continue;              // second halves of a head go with their partner
          const float4 t01 = tb[i & 1][q % HQ][0], t23 = tb[i & 1][q % HQ][1];
          const float c[4] = {t01.x, t01.z, t23.x, t23.z}, sn[4] = {t01.y, t01.w, t23.y, t23.w};
          float lo[4], hi[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x1 = x[q][e], x2 = x[q + HQ][e];
            lo[e] = x1 * c[e] - x2 * sn[e];
            hi[e] = x2 * c[e] + x1 * sn[e];
          }
          put(q * 16 + feat, make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])));
          put((q + HQ) * 16 + feat, make_uint2(pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])));
        }
      } else if constexpr (ROPE) {
#pragma unroll
        for (int q = 0; q < TN; ++q) put(q * 16 + feat, make_uint2(pack_bf16(x[q][0], x[q][1]), pack_bf16(x[q][2], x[q][3])));
      } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int q = 0; q < TN; ++q) {
          if ((q >> 1) & 1) continue;              // gate and up rows alternate in blocks of 32
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gt = x[q][e], up = x[q + 2][e];
            // the hardware reciprocal (1 ulp; the result is rounded to bf16 right after): an IEEE
            // division is eleven instructions, 64 of them per lane and tile
            v[e] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
          }
          put((q >> 2) * 32 + (q & 1) * 16 + feat, make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])));
        }
      } else {
        if (EPI == EPI_RESIDUAL) {
          // the residual rows, in the slots of the values they are added to
#pragma unroll
          for (int s = 0; s < NST; ++s) *(u32x4_t*)(sl + stage_at(s * RPI + srow, schunk * 8)) = rr[i % RAHEAD][s];
          LZ_LDS_ORDER();
          if constexpr (i + RAHEAD < TM) fetch_residual(Int<i + RAHEAD>{});
        }
        uint2 r2[TN];
        if (EPI == EPI_RESIDUAL) {
#pragma unroll
          for (int q = 0; q < TN; ++q) r2[q] = *(const uint2*)(sl + stage_at(tok, q * 16 + feat));
          LZ_LDS_ORDER();
        }
        float ss = 0.f;
#pragma unroll
        for (int q = 0; q < TN; ++q) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = x[q][e];
          if (EPI == EPI_RESIDUAL) {
            v[0] += bf16_lo(r2[q].x); v[1] += bf16_hi(r2[q].x);
            v[2] += bf16_lo(r2[q].y); v[3] += bf16_hi(r2[q].y);
          }
          const uint2 w2 = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
          put(q * 16 + feat, w2);
          if (EPI == EPI_RESIDUAL) {
            const float a = bf16_lo(w2.x), b = bf16_hi(w2.x), c = bf16_lo(w2.y), e = bf16_hi(w2.y);
            ss += a * a + b * b + c * c + e * e;
          }
        }
        if (EPI == EPI_RESIDUAL && ra.ssq_out != nullptr) {
          ss += __shfl_xor(ss, 16, 64);
          ss += __shfl_xor(ss, 32, 64);
          if (el < 16 && valid) atomicAdd(ra.ssq_out + row, ssq_to_fixed(ss));
        }
      }
      if (!VPART || ra.v != nullptr) {
        LZ_LDS_ORDER();
#pragma unroll
        for (int s = 0; s < NST; ++s) {
          const int r = s * RPI + srow;
          const u32x4_t v = *(const u32x4_t*)(sl + stage_at(r, schunk * 8));
          const int orow = row0 + i * 16 + r;
          if (orow < M) {
            const size_t dr = (ROPE && region == 1 && ra.k_row != nullptr) ? (size_t)ra.k_row[orow] : (size_t)orow;
            *(u32x4_at_8_t*)(obase + dr * old + schunk * 8) = v;
          }
        }
      }
      if constexpr (ROPE && VPART) {
        if (ra.vt != nullptr) {
          // V once more, transposed, for the attention kernel's second product: from the stage a lane
          // takes eight tokens of one feature.  Where the block's 16 tokens have 16 consecutive columns
          // they leave in one store of 16 bytes (on a 2-byte boundary in packed sequences: global memory
          // takes it), else one by one.  The loop is rolled on purpose: written out per block of
          // columns, with both cases, it was 20 KB of code that did little but wait for the instruction
          // cache (64 KB for two CUs, the kernel 89 KB; now 70).  With 4-byte stores straight from the
          // accumulators / so, us: 8192 x 12288 x 4096 626 / 605, 3376 rows 298 / 290, 5000 x 3072 x 1024 45 / 41.
          const int vcol = valid ? (ra.vt_col != nullptr ? ra.vt_col[row] : row) : -1;
          const int vcol0 = __builtin_amdgcn_readfirstlane(vcol);
          const bool whole = __builtin_amdgcn_ballot_w64(vcol != vcol0 + tok) == 0;      // (and every row is below M)
          LZ_LDS_ORDER();
#pragma unroll 1
          for (int s = 0; s < 4; ++s) {
            const int f = s * 32 + (el >> 1), t0 = (el & 1) * 8;
            u16x8_t v;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = *(const uint16_t*)(sl + stage_at(t0 + e, f & ~3) + (f & 3) * 2);
            uint16_t* const vr = ra.vt + (size_t)(rcol0 + f) * ra.vt_ld;
            if (whole) *(u16x8_at_2_t*)(vr + vcol0 + t0) = v;
            else
#pragma unroll 1
              for (int e = 0; e < 8; ++e) {
                const int r = row0 + i * 16 + t0 + e;
                const uint16_t one = *(const uint16_t*)(sl + stage_at(t0 + e, f & ~3) + (f & 3) * 2);
                if (r < M) vr[ra.vt_col != nullptr ? ra.vt_col[r] : r] = one;
              }
          }
        }
      }
      LZ_LDS_ORDER();
      __builtin_amdgcn_sched_barrier(0);
    };
    if (ROPE && region == 2) {
      unrolled<TM>([&](auto ii) { put_rows(ii, Int<1>{}); });
    } else {
      if constexpr (ROPE) fetch_table(Int<0>{});
      unrolled<TM>([&](auto ii) { put_rows(ii, Int<0>{}); });
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the stage is read before it is copied over
    __builtin_amdgcn_sched_barrier(0);
  }
#undef LZ_READ
#undef LZ_HALF
#undef LZ_READ8
#undef LZ_HALF8
#undef LZ_STEP
#undef LZ_LDS_ORDER
#undef LZ_ACC_RESERVE
}

// Workgroups of the kernel that are resident at once (one per CU when the device is otherwise
// idle); 0 if the runtime cannot tell.
template <typename KernT>
static int w4_resident_workgroups(KernT kern, int lds_bytes) {
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, 256, (size_t)lds_bytes) != hipSuccess)
    return 0;
  return per_cu >= 1 ? cus : 0;
}

template <int TM, bool F8>
static hipError_t launch_w4(const void* A, const float* sa, const void* W, const float* sw, void* C, const void* R,
                            int M, int N, int K, int lda, int ldw, int ldc, int epi, int group_m,
                            const EpiArgs& ra, int stream_k, float* part, unsigned* flags, hipStream_t st) {
  constexpr int BM = 32 * TM, BN = 256, LDS_BYTES = 5 * W4_SLOT, ESIZE = F8 ? 1 : 2;
  if (N % BN != 0 || K % (ROW_BYTES / ESIZE) != 0) return hipErrorInvalidValue;
  if ((unsigned long long)M * lda * ESIZE >= (1ull << 32) ||
      (unsigned long long)N * (ra.w_blocked ? K : ldw) * ESIZE >= (1ull << 32))
    return hipErrorInvalidValue;
  if (stream_k && (part == nullptr || flags == nullptr || K > (1 << 24))) return hipErrorInvalidValue;
  if (!rows_on_boundaries(8, epi, C, R, ldc, ra)) return hipErrorInvalidValue;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN, KT = K / (ROW_BYTES / ESIZE);
  EpiArgs ea = ra;
  ea.w_step_bytes = ra.w_blocked ? (unsigned long long)N * ROW_BYTES : (unsigned long long)ROW_BYTES;
  lda *= ESIZE;
  ldw = ra.w_blocked ? ROW_BYTES : ldw * ESIZE;     // blocked: rows of one K step are 128 bytes apart
  ea.sf_blocks_per_seq = (ea.sf_max_rows + 255) / 256;
  const int side = ea.sf_z != nullptr ? ea.sf_blocks_per_seq * ea.sf_batch : 0;
#define LZ_GEMM(E)                                                                               \
  do {                                                                                           \
    auto kern = gemm_w4_kernel<TM, E, F8>;                                                       \
    static int resident = -1;                                                                    \
    if (resident < 0) {                                                                          \
      hipError_t e = hipFuncSetAttribute((const void*)kern,                                      \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES); \
      if (e != hipSuccess) return e;                                                             \
      resident = w4_resident_workgroups(kern, LDS_BYTES);                                        \
    }                                                                                            \
    int G = resident < 256 ? resident : 256;                                                     \
    G &= ~7;                                        /* whole rounds over the 8 XCDs */           \
    if (stream_k) {                                                                              \
      G = gemm_aligned_grid(G, tiles_m * tiles_n);                                               \
      if (G < 8) return hipErrorInvalidConfiguration;                                            \
    } else if (G < 8 || G > tiles_m * tiles_n) G = tiles_m * tiles_n;                            \
    hipLaunchKernelGGL(kern, dim3(G + side), dim3(256), LDS_BYTES, st, (const char*)A,           \
                       (const char*)W, sa, sw, (uint16_t*)C, (const uint16_t*)R, M, KT, lda,     \
                       ldw, ldc, tiles_m, tiles_n, group_m, G, stream_k, part, flags, ea);       \
  } while (0)
  if (epi == EPI_STORE) LZ_GEMM(EPI_STORE);
  else if (epi == EPI_RESIDUAL) LZ_GEMM(EPI_RESIDUAL);
  else if (epi == EPI_SWIGLU) LZ_GEMM(EPI_SWIGLU);
  else if (epi == EPI_QKV_ROPE) {
    if (ra.head_dim == 64) LZ_GEMM(EPI_QKV_ROPE64);
    else LZ_GEMM(EPI_QKV_ROPE128);
  }
  else return hipErrorInvalidValue;
#undef LZ_GEMM
  return hipGetLastError();
}

}  // namespace lz
