// The four-wave GEMM tile (gemm_w4.h) on OFP8 E4M3 operands.
#include "gemm_w4.h"

namespace lz {

hipError_t launch_gemm_w4_f8(const void* A, const float* sa, const void* W, const float* sw, void* C, const void* R,
                             int M, int N, int K, int lda, int ldw, int ldc, int epi, int group_m,
                             const EpiArgs& ra, int stream_k, float* part, unsigned* flags, int rows, hipStream_t st) {
#define LZ_W4(TM) launch_w4<TM, true>(A, sa, W, sw, C, R, M, N, K, lda, ldw, ldc, epi, group_m, ra, stream_k, part, flags, st)
  return rows == 256 ? LZ_W4(8) : rows == 192 ? LZ_W4(6) : rows == 128 ? LZ_W4(4) : hipErrorInvalidValue;
#undef LZ_W4
}

}  // namespace lz
