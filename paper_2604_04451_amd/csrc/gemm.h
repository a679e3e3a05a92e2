// The GEMM as the library's own callers use it: chorus_gemm_bf16 with optional scratch, with which a gated-residual
// product that would leave most compute units idle is cut into slices of K.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace chorus {

// Two pieces of scratch (16-byte aligned device memory, either may be empty), used only by the kernels of the call.
// Every slice but the last puts its fp32 [M, N] result there: the first one into `first`, the others into `rest`.
struct GemmParts {
  void* first;
  size_t first_bytes;
  void* rest;
  size_t rest_bytes;
  // kGemmCounts words that are zero when the product starts, or null: the slices may then add to the residual one behind the other instead
  uint32_t* counts;
};
constexpr int kGemmCounts = 256;
// Whether a gated-residual product of that size uses the counts: if not, nothing has to clear them.
bool gemm_bf16_chained(int64_t M, int32_t N, int32_t K, const GemmParts& parts);

// chorus_gemm_bf16 with scratch; the number of slices depends on the sizes given here and on nothing else
int32_t gemm_bf16_parts(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, int32_t epilogue, void* out,
                        const float* bias, const float* gate0, const float* gate1, float scale, const GemmParts& parts,
                        void* stream);

// out = A W^T + bias and out2 = A2 W2^T + bias2, bf16, the same K: in one launch where that does not fill the chip
int32_t gemm_bf16_two(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, uint16_t* out, const float* bias,
                      const uint16_t* A2, const uint16_t* W2, int64_t M2, int32_t N2, uint16_t* out2, const float* bias2,
                      void* stream);

}  // namespace chorus
