// Host side of the projections (plan and launch), the split-K reduce, the
// fp32 kernel and the split of an fp32 operand into its planes.  The bf16
// kernels are in gemm_tile.h.
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "gemm_tile.h"

namespace cdsl {

namespace {

// The sum of the split planes in split order, then the epilogue; V outputs
// per thread (4 where rows and addresses allow 16-byte accesses).  Bound by
// the planes' trip through the caches; eight planes' loads are in flight.
template <int V>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a) {
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * V;
  const long long plane = (long long)a.M * a.N;
  auto sum = [&](long long at, float (&v)[V]) {
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = 0.f;
    for (int z0 = 0; z0 < a.ksplit; z0 += 8) {
      float t[8][V];
#pragma unroll
      for (int z = 0; z < 8; ++z) {
        const float* q = a.partial + min(z0 + z, a.ksplit - 1) * plane + at;
        if constexpr (V == 4) {
          const float4 x = *(const float4*)q;
          t[z][0] = x.x, t[z][1] = x.y, t[z][2] = x.z, t[z][3] = x.w;
        } else {
          t[z][0] = *q;
        }
      }
#pragma unroll
      for (int z = 0; z < 8; ++z)
        if (z0 + z < a.ksplit)
#pragma unroll
          for (int e = 0; e < V; ++e) v[e] += t[z][e];
    }
  };
  if (a.epi == kEpiSwiGLU) {
    const int F = a.N / 2;
    if (i >= (long long)a.M * F) return;
    const int row = (int)(i / F), f = (int)(i % F);
    const long long ig = (long long)row * a.N + (f >> 4) * 32 + (f & 15);
    float g[V], u[V];
    sum(ig, g);
    sum(ig + 16, u);
    const long long o = (long long)row * a.ldc + f;
    bf16 h[V], l[V];
#pragma unroll
    for (int e = 0; e < V; ++e) split_bf16(silu(g[e]) * u[e], h[e], l[e]);
    if constexpr (V == 4) {
      *(bf16x4*)(a.Chi + o) = (bf16x4){h[0], h[1], h[2], h[3]};
      *(bf16x4*)(a.Clo + o) = (bf16x4){l[0], l[1], l[2], l[3]};
    } else {
      a.Chi[o] = h[0];
      a.Clo[o] = l[0];
    }
    return;
  }
  if (i >= plane) return;
  float v[V];
  sum(i, v);
  const int row = (int)(i / a.N), col = (int)(i % a.N);
  float* C = (float*)a.C + (long long)row * a.ldc + col;
  if constexpr (V == 4) {
    float4 x = make_float4(v[0], v[1], v[2], v[3]);
    if (a.epi == kEpiResidual) {
      const float4 c = *(const float4*)C;
      x = make_float4(c.x + v[0], c.y + v[1], c.z + v[2], c.w + v[3]);
    }
    *(float4*)C = x;
  } else {
    if (a.epi == kEpiResidual) *C += v[0];
    else *C = v[0];
  }
}

// ---------------------------------------------------------------------------
// fp32 kernel (the fp32 workload): 4 waves, a tile of 16 TM x 16 TN outputs
//
// v_mfma_f32_16x16x4: plain fp32 products and sums.  The shapes are small
// (tens of rows, K of a few hundred), so what counts is the chain of
// dependent steps: the four waves of a workgroup take the 16-deep K chunks in
// turn (wave w: chunks w, w + 4, ...), each straight from memory with every
// load of UN chunks in flight, and add their tiles through LDS in wave order.
// An output's sum is formed in the same order whatever the tile, so a row
// does not depend on the other rows of its batch.  Lane (r, g) loads 4
// consecutive K of row r; element e of the four feeds MFMA e, the same K on
// both sides.  Before, 64 x 64 tiles staged 16 K at a time through LDS with
// two barriers each: 16 x 768 x 256 took 22 us.
// ---------------------------------------------------------------------------
template <int TM, int TN, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_tiled(const float* __restrict__ A, const float* __restrict__ B,
                                                      float* __restrict__ C, int M, int N, int K, int ldc, RowStats rs) {
  constexpr int BM = 16 * TM, BN = 16 * TN, UN = TM * TN >= 8 ? 2 : 4;
  __shared__ __attribute__((aligned(16))) float part[4][BM * BN];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const float* ap[TM];
  const float* bp[TN];
#pragma unroll
  for (int t = 0; t < TM; ++t) ap[t] = A + (long long)min(m0 + t * 16 + lr, M - 1) * K + lg * 4;
#pragma unroll
  for (int j = 0; j < TN; ++j) bp[j] = B + (long long)min(n0 + j * 16 + lr, N - 1) * K + lg * 4;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int nc = K / 16;
  for (int c0 = w; c0 < nc; c0 += 4 * UN) {
    f32x4 a[UN][TM], b[UN][TN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int c = c0 + 4 * u;
      if (c >= nc) break;
#pragma unroll
      for (int t = 0; t < TM; ++t) a[u][t] = *(const f32x4u*)(ap[t] + c * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[u][j] = *(const f32x4u*)(bp[j] + c * 16);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (c0 + 4 * u >= nc) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][t][e], b[u][j][e], acc[t][j], 0, 0, 0);
    }
  }
  // lane (lr, lg) holds rows 4 lg .. + 3 of column lr of each 16 x 16 tile
  auto at = [&](int r, int c) {
    if constexpr (EPI == kEpiRowStats) return RsLayout<256, BM, BN>::at(r, c);
    else return r * BN + c;
  };
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[w][at(t * 16 + lg * 4 + e, j * 16 + lr)] = acc[t][j][e];
  __syncthreads();
  auto sum = [&](int o) { return ((part[0][o] + part[1][o]) + part[2][o]) + part[3][o]; };
  if constexpr (EPI == kEpiRowStats) {
    for (int o = tid; o < BM * BN; o += 256) part[0][o] = sum(o);
    __syncthreads();
    tile_row_stats<256, BM, BN>(part[0], m0, n0, M, N, blockIdx.x, rs);
  } else if constexpr (EPI == kEpiSwiGLU) {
    for (int o = tid; o < BM * BN / 2; o += 256) {
      const int r = o / (BN / 2), f = o % (BN / 2), c = (f >> 4) * 32 + (f & 15);
      if (m0 + r >= M || n0 + c >= N) continue;
      C[(long long)(m0 + r) * ldc + n0 / 2 + f] = silu(sum(r * BN + c)) * sum(r * BN + c + 16);
    }
  } else {
    for (int o = tid; o < BM * BN; o += 256) {
      const int row = m0 + o / BN, col = n0 + o % BN;
      if (row >= M || col >= N) continue;
      float* c = C + (long long)row * ldc + col;
      if (EPI == kEpiResidual) *c += sum(o);
      else *c = sum(o);
    }
  }
}

template <int TM, int TN>
void gemm_f32(const GemmOperand& A, const void* B, const GemmOut& out, int M, int N, int K, int epi, const RowStats& rs,
              hipStream_t st) {
  const dim3 grid((N + 16 * TN - 1) / (16 * TN), (M + 16 * TM - 1) / (16 * TM));
  const float* b = (const float*)B;
  switch (epi) {
    case kEpiRowStats:
      if constexpr (TN == 4) gemm_f32_tiled<TM, TN, kEpiRowStats><<<grid, 256, 0, st>>>(A.f32, b, out.f32, M, N, K, out.ldc, rs);
      break;
    case kEpiSwiGLU:
      gemm_f32_tiled<TM, TN, kEpiSwiGLU><<<grid, 256, 0, st>>>(A.f32, b, out.f32, M, N, K, out.ldc, rs);
      break;
    case kEpiResidual:
      gemm_f32_tiled<TM, TN, kEpiResidual><<<grid, 256, 0, st>>>(A.f32, b, out.f32, M, N, K, out.ldc, rs);
      break;
    default:
      gemm_f32_tiled<TM, TN, kEpiStore><<<grid, 256, 0, st>>>(A.f32, b, out.f32, M, N, K, out.ldc, rs);
  }
}

// split an fp32 matrix into its bf16 hi / lo planes (for operands that do not
// come from a library kernel, e.g. the kernel-level entry point)
__global__ void split_planes(const float* __restrict__ x, bf16* __restrict__ hi, bf16* __restrict__ lo, long long n) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bf16 h, l;
  split_bf16(x[i], h, l);
  hi[i] = h;
  lo[i] = l;
}
// eight values per thread (n a multiple of 8, planes 16-byte aligned): 800 x
// 4096 in 6 us, 8.4 one by one
__global__ __launch_bounds__(256) void split_planes8(const float* __restrict__ x, bf16* __restrict__ hi,
                                                     bf16* __restrict__ lo, long long n) {
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  const f32x4 a = *(const f32x4u*)(x + i), b = *(const f32x4u*)(x + i + 4);
  bf16x8 hv, lv;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    bf16 h, l;
    split_bf16(e < 4 ? a[e] : b[e - 4], h, l);
    hv[e] = h;
    lv[e] = l;
  }
  *(bf16x8*)(hi + i) = hv;
  *(bf16x8*)(lo + i) = lv;
}

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
// What a configuration's workgroups cost, fitted to 26 thousand timings on
// MI355X (1 to 4096 rows, 33 pairs of N and K, every split; weights from HBM),
// in us.  occ workgroups share a CU (DenseCfg::OCC), so a round holds 256 * occ
// of them; a round of n workgroups of `per` stages takes
//   round + per * sqrt(lone^2 + (full * (busy - 1))^2 + (fill * c)^2),
// lone the stage time of a workgroup by itself (latency), busy the workgroups
// of the fullest CU (a round lasts as long as that CU: 282 workgroups of 64 x
// 64 take what 512 take), c the time of the round's copies into LDS at 12.5
// TB/s (rows past M are not read).  The weights' trip from HBM adds as the
// root of squares, so that shapes that wait for it still differ.  A split
// costs the writes of its planes, and the launch of its reduce (2.1 to 2.5 us
// measured, and 123 MB of planes in 20) or what the consumer takes longer
// (RMSNorm of 80 rows of 2048: 2.8 us without planes, 3.7 with two to eight; of
// 800 rows of 4096 6.0, 13.3 and 23.9: planes beyond the caches).  Over those
// shapes the model's choice is on average 2% slower than the best measured pair
// (worst: 29%); a table that counted three workgroups per CU where two ran, that
// charged 4.5 us for a reduce and that took the load of all CUs for that of each
// was 6 to 9% slower (1 x 2048 x 2048 with its reduce 10.1 us unsplit, 6.4 in
// eight splits).
//
// Measured with them (product alone, us; the earlier pair of kernels, one
// for up to 128 rows with weights in registers and one with 160 x 256 tiles
// staged through registers, in brackets): 800 x 12288 x 4096 117 (160), 800 x
// 22016 x 4096 230 (271), 4096 x 22016 x 4096 1044 (1440, 708 TFLOP/s of
// product), 160 x 16384 x 2048 27 (43), 80 x 22016 x 4096 51 (81), 80 x 16384 x
// 2048 21 (27), 80 x 32000 x 2048 37 (45), 16 x 22016 x 4096 40 (49), 16 x 8192
// x 1024 5.7 (9.9).
#define CFG_SHAPE(I, WM, WN, TM, TN, P) {WM * TM * 16, WN * TN * 16},
constexpr int kShape[kGemmCfgs][2] = {CDSL_GEMM_CFGS(CFG_SHAPE)};
#undef CFG_SHAPE
#define CFG_OCC(I, ...) DenseCfg<__VA_ARGS__>::OCC,
constexpr int kOcc[kGemmCfgs] = {CDSL_GEMM_CFGS(CFG_OCC)};
#undef CFG_OCC
constexpr struct {
  float start, round, lone, full, fill;
} kCost[] = {
    {4.7f, 3.1f, 1.94f, 0.00f, 0.89f},   // 256 x 256
    {3.8f, 3.1f, 1.32f, 0.00f, 0.79f},   // 160 x 256
    {3.7f, 2.8f, 1.03f, 0.00f, 0.78f},   // 128 x 256
    {2.8f, 3.3f, 0.70f, 0.00f, 0.67f},   // 160 x 128
    {2.4f, 3.0f, 0.57f, 0.00f, 0.64f},   // 128 x 128
    {2.3f, 2.8f, 0.65f, 0.00f, 0.55f},   // 64 x 256
    {1.9f, 1.8f, 0.45f, 0.00f, 0.50f},   // 64 x 128
    {2.1f, 1.2f, 0.32f, 0.48f, 0.39f},   // 64 x 64
    {1.8f, 1.3f, 0.30f, 0.47f, 0.42f},   // 48 x 64
    {1.6f, 1.2f, 0.24f, 0.41f, 0.29f},   // 32 x 64
    {2.3f, 0.4f, 0.20f, 0.31f, 0.26f},   // 16 x 64
};
static_assert(sizeof(kCost) / sizeof(kCost[0]) == kGemmCfgs, "a cost per configuration");

struct Plan {
  int kind;          // 0 dense, 1 skinny, 2 f32
  int cfg;
  int tiles_m, tiles_n;
  int ksplit, kchunk;
  double us;         // the model's time
  size_t ws_bytes;
};

// Where the split planes of a projection go: to the kernel that consumes the
// product, which adds the planes as it reads them (kFold), or to a reduce
// launch of their own (kReduce); kNone: no split.
enum SplitUse { kFold = 0, kReduce = 1, kNone = 2 };

double cfg_us(int cfg, int rows, int tiles, int splits, int per) {
  const auto& c = kCost[cfg];
  const int n = tiles * splits, cap = 256 * kOcc[cfg], full = n / cap, rem = n % cap;
  auto round = [&](int k) {
    const double f = c.full * ((k + 255) / 256 - 1), m = c.fill * (2 * rows + kShape[cfg][1]) * (2.0 * DKC) * k / 12.5e6;
    return c.round + per * sqrt((double)c.lone * c.lone + f * f + m * m);
  };
  return c.start + full * round(cap) + (rem ? round(rem) : 0.0);
}

// What ks planes of `plane` bytes cost: their writes, then the reduce launch or
// what their consumer takes longer.
double split_us(SplitUse use, int ks, double plane) {
  if (ks == 1) return 0.0;
  const double b = (ks + 1) * plane, write = ks * plane / 8.3e6;
  return write + (use == kReduce ? 2.3 + b / 8e6 : 1.0 + b / 16e6 + std::max(0.0, b - 32e6) / 10e6);
}

// The plan of a shape: a pure function of its arguments.  hd > 0: only
// configurations whose tile holds whole heads of hd columns.  max_ws: the
// most that the split planes may take.  Rows count in 16-row tiles, so all M
// of one tile count share a plan.
Plan search_plan(int M, int N, int K, SplitUse use, int hd, size_t max_ws) {
  Plan p{};
  p.kind = M <= 128 ? 1 : 0;
  const int M16 = (M + 15) / 16 * 16, nk = (K - 1) / DKC + 1;
  // weights once from HBM, whatever the tiles
  const double stream = 1.2 + (double)N * K * 2.0 / 6.5e6;
  p.us = 1e300;
  for (int c = 0; c < kGemmCfgs; ++c) {
    const int bm = kShape[c][0], bn = kShape[c][1];
    if (hd > 0 && bn % hd != 0) continue;
    if (bm >= 2 * M16 && bm > 16) continue;   // half of the tile rows or more would be padding
    if (bm < 64 && M16 > 2 * bm + 32) continue;
    const long long tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn;
    if (tm * tn > INT32_MAX / 32) continue;
    const int tiles = (int)(tm * tn);
    int last = 0;
    for (int s = 1; s <= 16 && (s == 1 || nk / s >= 3); ++s) {
      if (s > 1 && (use == kNone || tiles * s > 1024)) break;
      const int per = (nk + s - 1) / s, ks = (nk + per - 1) / per;
      if (ks == last) continue;
      last = ks;
      if (ks > 1 && ks * ((double)M * N * 4.0) > (double)max_ws) break;
      const double us = hypot(cfg_us(c, M16 / (int)tm, tiles, ks, per), stream) + split_us(use, ks, (double)M16 * N * 4.0);
      if (us < p.us) {
        p.us = us;
        p.cfg = c;
        p.tiles_m = (int)tm;
        p.tiles_n = (int)tn;
        p.ksplit = ks;
        p.kchunk = (int)std::min<long long>((long long)per * DKC, K);
      }
    }
  }
  p.ws_bytes = p.ksplit > 1 ? (size_t)p.ksplit * M * N * sizeof(float) : 0;
  return p;
}

// search_plan, remembered per thread (a pass asks for the same few shapes
// once per layer and the search takes microseconds)
Plan make_plan(int M, int N, int K, int dtype, SplitUse use, int hd = 0, size_t max_ws = SIZE_MAX) {
  if (dtype == 0) {
    Plan p{};
    p.kind = 2;
    p.ksplit = 1;
    return p;
  }
  struct Entry {
    int M, N, K, use, hd;
    size_t ws;
    Plan p;
  };
  static thread_local Entry memo[64] = {};
  const unsigned h = ((unsigned)M * 2654435761u ^ (unsigned)N * 40503u ^ (unsigned)K * 9973u ^ (unsigned)(use * 7 + hd)) >> 5 & 63;
  Entry& e = memo[h];
  if (e.M != M || e.N != N || e.K != K || e.use != use || e.hd != hd || e.ws != max_ws)
    e = Entry{M, N, K, use, hd, max_ws, search_plan(M, N, K, use, hd, max_ws)};
  return e.p;
}

SplitUse split_use(int epi, bool deferred) {
  return epi == kEpiRowStats || epi == kEpiRope ? kNone : deferred && epi != kEpiSwiGLU ? kFold : kReduce;
}

// Column tiles of a row-statistics launch.
int rowstats_tiles(const Plan& p, int N) { return p.kind == 2 ? (N + 63) / 64 : p.tiles_n; }

}  // namespace

size_t gemm_workspace_bytes(int M, int N, int K, int dtype, bool deferred) {
  if (dtype == 0 || M <= 0) return 0;
  size_t b = make_plan(M, N, K, dtype, deferred ? kFold : kReduce).ws_bytes;
  return (b + 255) & ~(size_t)255;
}

int gemm_kind(int M, int N, int K, int dtype) { return dtype == 0 ? 2 : M <= 128 ? 1 : 0; }

int gemm_rowstats_tiles(int M, int N, int K, int dtype) {
  if (M <= 0) return 0;
  return rowstats_tiles(make_plan(M, N, K, dtype, kNone), N);
}

// The rotary epilogue needs an unsplit launch of tiles with whole heads.  It
// takes 1 to 5 us more than the stores' (up to 16 where rows of a beam do not
// start at multiples of four slots: 800 rows of ten, 12288 columns), and saves
// the rotary launch, 3 to 10 us with the product's trip through memory.  So it
// is taken where the unsplit product costs at most 2.5 us more than the best
// one with its planes (both by the plan).  Over 111 shapes of 5 models, 8 to 2000
// rows, that is 1.4% slower on average than always taking the faster (with no
// such allowance 3.8%): 160 rows of 3072 x 1024 9.9 us against 14.1, 105 of 3072 x
// 2048 17.0 and 17.3, 160 of 6144 x 2048 21.0 and 22.6, 96 of 6144 x 4096 35 and 24.
bool gemm_rope_fusable(int M, int N, int K, int dtype, int hd) {
  if (M <= 0 || dtype != 1 || (hd != 64 && hd != 128) || N % hd != 0) return false;
  const Plan f = make_plan(M, N, K, dtype, kNone, hd), s = make_plan(M, N, K, dtype, kFold);
  return f.us <= s.us + 2.5;
}

int gemm_check(int M, int N, int K, int dtype) {
  if (M < 0 || N <= 0 || K <= 0) return -1;
  if (dtype == 1 && K % DBK != 0) return -1;
  if (dtype == 0 && K % 16 != 0) return -1;
  return 0;
}

hipError_t gemm_launch(const GemmOperand& A, const void* B, const GemmOut& out, int M, int N, int K, int dtype,
                       int epi, void* ws, size_t ws_bytes, hipStream_t st, bool prefill, GemmHook* hook,
                       int* deferred, RowStats* rs, const RopeEpi* rope, size_t max_ws) {
  if (deferred) *deferred = 1;
  if (M == 0) return hipSuccess;
  const bool stats = epi == kEpiRowStats;
  if (stats != (rs != nullptr)) return hipErrorInvalidValue;
  if ((epi == kEpiRope) != (rope != nullptr)) return hipErrorInvalidValue;
  if (rope && !gemm_rope_fusable(M, N, K, dtype, rope->hd)) return hipErrorInvalidValue;
  Plan p = make_plan(M, N, K, dtype, split_use(epi, deferred != nullptr), rope ? rope->hd : 0, max_ws);
  if (stats) {
    rs->tiles = rowstats_tiles(p, N);
    if (rs->tiles == 0 || rs->kk < 0 || rs->kk > 16) return hipErrorInvalidValue;
  }
  if (p.kind == 2) {
    // the smallest tiles until they give every CU a workgroup
    const RowStats r = stats ? *rs : RowStats{};
    const long long blocks = (long long)((M + 15) / 16) * ((N + 31) / 32);
    if (stats) {
      if (M <= 16) gemm_f32<1, 4>(A, B, out, M, N, K, epi, r, st);
      else gemm_f32<4, 4>(A, B, out, M, N, K, epi, r, st);
    } else if (blocks <= 512) {
      gemm_f32<1, 2>(A, B, out, M, N, K, epi, r, st);
    } else if (blocks <= 2048) {
      gemm_f32<2, 4>(A, B, out, M, N, K, epi, r, st);
    } else {
      gemm_f32<4, 4>(A, B, out, M, N, K, epi, r, st);
    }
    return hipGetLastError();
  }
  if (p.ws_bytes > ws_bytes) return hipErrorInvalidValue;
  GemmArgs a;
  a.Ahi = A.hi;
  a.Alo = A.lo;
  a.B = (const bf16*)B;
  a.M = M;
  a.N = N;
  a.K = K;
  a.C = out.f32;
  a.Chi = out.hi;
  a.Clo = out.lo;
  a.ldc = out.ldc;
  a.epi = epi;
  a.ksplit = p.ksplit;
  a.kchunk = p.kchunk;
  a.tiles_m = p.tiles_m;
  a.tiles_n = p.tiles_n;
  a.band = p.tiles_m <= 8 ? p.tiles_m : 4;
  a.partial = (float*)ws;
  a.rs = stats ? *rs : RowStats{};
  a.re = rope ? *rope : RopeEpi{};
  const int variant = stats ? 1 : rope ? 2 : 0;
  const dim3 grid(p.tiles_m * p.tiles_n, 1, p.ksplit);
  // the copies into LDS move whole 16-byte chunks at 32-bit offsets within a
  // tile: operands that are not aligned so, or whose tile of the larger side
  // spans 2 GiB (a caller's own; the library's are neither), go through registers
  const long long span = (long long)std::max(kShape[p.cfg][0], kShape[p.cfg][1]) * K * 2;
  const bool direct = (((uintptr_t)A.hi | (uintptr_t)A.lo | (uintptr_t)B) & 15) == 0 && span < (1LL << 31);
  if (!direct) {
    if (variant == 2) return hipErrorInvalidValue;
    gemm_unaligned_kernels(p.cfg, variant, grid, a, st);
  } else if (p.kind == 1) {
    gemm_skinny_kernels(p.cfg, variant, grid, a, st);
  } else if (prefill) {
    gemm_prefill_kernels(p.cfg, variant, grid, a, st);
  } else {
    gemm_dense_kernels(p.cfg, variant, grid, a, st);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.ksplit == 1) return e;
  if (deferred && epi != kEpiSwiGLU) {
    *deferred = p.ksplit;
    return hipSuccess;
  }
  const long long outs = epi == kEpiSwiGLU ? (long long)M * (N / 2) : (long long)M * N;
  if (hook) hook->before_reduce(p.ksplit);
  const bool four = epi == kEpiSwiGLU
                        ? N % 32 == 0 && out.ldc % 4 == 0 && (((uintptr_t)a.partial & 15) | ((uintptr_t)a.Chi & 7) |
                                                              ((uintptr_t)a.Clo & 7)) == 0
                        : N % 4 == 0 && out.ldc % 4 == 0 && (((uintptr_t)a.partial | (uintptr_t)a.C) & 15) == 0;
  if (four) splitk_reduce_kernel<4><<<(unsigned)((outs / 4 + 255) / 256), 256, 0, st>>>(a);
  else splitk_reduce_kernel<1><<<(unsigned)((outs + 255) / 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t split_planes_launch(const float* x, bf16* hi, bf16* lo, long long n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (n % 8 == 0 && (((uintptr_t)hi | (uintptr_t)lo) & 15) == 0 && ((uintptr_t)x & 3) == 0)
    split_planes8<<<(unsigned)((n / 8 + 255) / 256), 256, 0, st>>>(x, hi, lo, n);
  else
    split_planes<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(x, hi, lo, n);
  return hipGetLastError();
}

}  // namespace cdsl
