// bf16 projection kernels of passes of at most 128 rows (the rollout).
#include "gemm_tile.h"

#define CASE(I, E, WM, WN, ...)                                                         \
  case I * 3 + E:                                                                       \
    gemm_bf16_skinny<WM, WN, __VA_ARGS__, E, true, 0><<<grid, 64 * WM * WN, 0, st>>>(a);  \
    break;
#define CDSL_GEMM_CASE(I, ...) CASE(I, 0, __VA_ARGS__) CASE(I, 1, __VA_ARGS__) CASE(I, 2, __VA_ARGS__)

namespace cdsl {

CDSL_GEMM_KERNELS(gemm_bf16_skinny, gemm_skinny_kernels)

}  // namespace cdsl
