// bf16 projection kernels for operands that the direct copies do not take: not
// 16-byte aligned, or with a tile that spans 2 GiB (only the kernel-level entry
// points take such).
#include "gemm_tile.h"

#define CASE(I, E, WM, WN, ...)                                                         \
  case I * 3 + E:                                                                       \
    gemm_bf16_unaligned<WM, WN, __VA_ARGS__, E, false, 0><<<grid, 64 * WM * WN, 0, st>>>(a);  \
    break;
#define CDSL_GEMM_CASE(I, ...) CASE(I, 0, __VA_ARGS__) CASE(I, 1, __VA_ARGS__)

namespace cdsl {

CDSL_GEMM_KERNELS(gemm_bf16_unaligned, gemm_unaligned_kernels)

}  // namespace cdsl
