// Device code of the bf16 projection kernels: C[M,N] = A[M,K] * W[N,K]^T with
// fp32 accumulation.
//
// The activation operand arrives as two bf16 planes, A = A_hi + A_lo (written
// that way by the kernel that produced it), and every MFMA step is done twice
// (A_hi * W, A_lo * W) into one fp32 accumulator: the weights are exactly
// bf16, so the product keeps fp32-level accuracy at twice the MFMA work of a
// plain bf16 product.
//
// Both operands are K-contiguous ([rows][K] row-major), which is what the
// CDNA4 MFMA fragments want: lane (r, g) of v_mfma_f32_16x16x32_bf16 holds 8
// consecutive K elements of row r, so every fragment is one 16-byte load.
//
// One kernel serves every row count; its tile shapes are listed at
// CDSL_GEMM_CFGS and chosen per shape by the plan in gemm.hip.  When the tile
// grid cannot fill the 256 CUs, K is split across workgroups; each split
// writes its own fp32 plane, summed in split order (bitwise deterministic) by
// a reduce kernel or by the kernel that consumes the result.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"
#include "gemm.h"

namespace cdsl {

struct GemmArgs {
  const bf16* Ahi;
  const bf16* Alo;
  const bf16* B;
  int M, N, K;
  void* C;          // fp32 [M, ldc] (store / residual)
  bf16* Chi;        // SwiGLU output planes [M, ldc]
  bf16* Clo;
  int ldc;
  int epi;
  int ksplit, kchunk;
  float* partial;   // split planes [ksplit][M][N]
  int tiles_m, tiles_n;
  int band;         // row blocks per band of the tile order
  RowStats rs;      // kEpiRowStats: per-tile row statistics instead of C
  RopeEpi re;       // kEpiRope: rotary + KV write instead of C
};

// Tile configurations X(index, WM, WN, TM, TN, P): WM x WN waves of
// TM x TN 16 x 16 tiles, P the prefetch distance in K stages.
#define CDSL_GEMM_CFGS(X)   \
  X(0, 4, 2, 4, 8, 1)       \
  X(1, 2, 4, 5, 4, 1)       \
  X(2, 2, 4, 4, 4, 1)       \
  X(3, 2, 4, 5, 2, 2)       \
  X(4, 2, 4, 4, 2, 2)       \
  X(5, 2, 4, 2, 4, 2)       \
  X(6, 2, 4, 2, 2, 2)       \
  X(7, 2, 2, 2, 2, 2)       \
  X(8, 1, 4, 3, 1, 2)       \
  X(9, 2, 2, 1, 2, 3)       \
  X(10, 1, 4, 1, 1, 3)

constexpr int kGemmCfgs = 11;
constexpr int DBK = 32;         // K granularity (one MFMA k-step)
constexpr int DKC = 64;         // K per stage

// The kernels by use, each in its own file (and under its own name in a
// profile): passes of more than 128 rows, prompt prefill, passes of at most
// 128 rows.  epi: 0 the stores, 1 kEpiRowStats, 2 kEpiRope.
void gemm_dense_kernels(int cfg, int epi, dim3 grid, const GemmArgs& a, hipStream_t st);
void gemm_prefill_kernels(int cfg, int epi, dim3 grid, const GemmArgs& a, hipStream_t st);
void gemm_skinny_kernels(int cfg, int epi, dim3 grid, const GemmArgs& a, hipStream_t st);
// operands that the direct copies do not take: not 16-byte aligned, or a tile
// that spans 2 GiB (epi 0 and 1)
void gemm_unaligned_kernels(int cfg, int epi, dim3 grid, const GemmArgs& a, hipStream_t st);

namespace {

__device__ __forceinline__ float silu(float x) { return x / (1.f + __expf(-x)); }

__device__ __forceinline__ void epi_store(const GemmArgs& a, int row, int col, float v) {
  if (row >= a.M || col >= a.N) return;
  float* C = (float*)a.C;
  long long idx = (long long)row * a.ldc + col;
  if (a.epi == kEpiResidual) C[idx] += v;
  else C[idx] = v;
}

// The packed gate/up weight puts 16 gate rows then the 16 matching up rows in
// every group of 32, so output column f of silu(gate) * up pairs packed
// columns 32*(f/16) + f%16 and that + 16.
__device__ __forceinline__ void epi_swiglu(const GemmArgs& a, int row, int col_gate, float g, float u) {
  if (row >= a.M || col_gate >= a.N) return;
  const int f = (col_gate >> 5) * 16 + (col_gate & 15);
  bf16 h, l;
  split_bf16(silu(g) * u, h, l);
  a.Chi[(long long)row * a.ldc + f] = h;
  a.Clo[(long long)row * a.ldc + f] = l;
}

__device__ __forceinline__ void part_store(const GemmArgs& a, int row, int col, float v) {
  if (row >= a.M || col >= a.N) return;
  a.partial[((long long)blockIdx.z * a.M + row) * a.N + col] = v;
}

// kEpiRowStats: statistics of the rows of an fp32 tile [BM][BN] held in LDS
// (rows m0 + r, columns n0 + c; rows >= M and columns >= N left out).  Four
// adjacent lanes share a row, each owning a run of CW columns.  The tile is
// stored with the 16-byte chunks of each run XOR-permuted by a row- and
// run-dependent key (RsLayout::at), so that the eight lanes that an LDS
// cycle serves read eight different chunks.  A lane reads its run into
// registers once: the maxima of its groups of 8 columns, and the sum of
// exp(v - max).  The top-kk places then cost a few instructions each: the
// row's best is the best of the four lanes' own bests, and only its owner
// reads a group again (from LDS) to find what is left of it.  Order: value
// descending, column ascending; entries of -inf are never picked.  t is the
// column tile's index in the RowStats layout.
//
// This pass is VALU-bound (one 160 x 256 tile took about 27 us when every
// place scanned the whole run in registers; the 800-row head of 32000 tokens
// with five places went from 455 to 368 us, planes and merge included).
template <int NT, int BM, int BN>
struct RsLayout {
  static constexpr int CW = BN / 4;                                     // columns per lane
  static_assert(CW == 16 || CW == 32 || CW == 64, "whole groups of 8 columns per lane");
  __device__ static int key(int r, int part) { return (part + 4 * ((r ^ (r >> 2)) & 1)) & (CW / 4 - 1); }
  __device__ static int at(int r, int c) {
    const int part = c / CW, i = c % CW;
    return r * BN + part * CW + (((i >> 2) ^ key(r, part)) << 2) + (i & 3);
  }
};

// the value of lane (lane ^ 1) or (lane ^ 2), within a quad
template <int X>
__device__ __forceinline__ int quad_xor(int v) {
  return __builtin_amdgcn_mov_dpp(v, X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
  return __int_as_float(quad_xor<X>(__float_as_int(v)));
}

template <int NT, int BM, int BN>
__device__ void tile_row_stats(const float* tile, int m0, int n0, int M, int N, int t, const RowStats& s) {
  using L = RsLayout<NT, BM, BN>;
  constexpr int CW = L::CW, GN = CW / 8;
  constexpr int RPP = NT / 4;                                     // rows per pass
  const int part = threadIdx.x & 3;
  const int c0 = part * CW;
  const int cbase = n0 + c0;
  const int nv = N - cbase;                                       // valid columns of this lane if < CW
  auto row_best = [&](float& v, int& id) {
    float ov = quad_xor<1>(v);
    int oi = quad_xor<1>(id);
    bool b = vi_better(ov, oi, v, id);
    v = b ? ov : v;
    id = b ? oi : id;
    ov = quad_xor<2>(v);
    oi = quad_xor<2>(id);
    b = vi_better(ov, oi, v, id);
    v = b ? ov : v;
    id = b ? oi : id;
  };
#pragma unroll 1
  for (int r0 = 0; r0 < BM; r0 += RPP) {
    // a wave whose first row is past the tile has no live row (uniform)
    if (r0 + (int)(threadIdx.x & ~63u) / 4 >= BM) continue;
    const int r = min(r0 + (int)threadIdx.x / 4, BM - 1);
    const int m = m0 + r;
    const bool live = r0 + (int)threadIdx.x / 4 < BM && m < M;
    const float* rowp = tile + r * BN + c0;
    const int key = L::key(r, part);
    // eight columns of group q: 16-byte chunks 2q and 2q + 1 of the run
    auto group = [&](int q, float (&x)[8]) {
      const float4 a = *(const float4*)(rowp + (((2 * q) ^ key) << 2));
      const float4 b = *(const float4*)(rowp + (((2 * q + 1) ^ key) << 2));
      x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w;
      x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
    };
    float v[GN][8], g[GN];
#pragma unroll
    for (int q = 0; q < GN; ++q) group(q, v[q]);
    if (n0 + BN > N) {   // the last tile: columns past N count as -inf
#pragma unroll
      for (int q = 0; q < GN; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[q][e] = q * 8 + e < nv ? v[q][e] : -INFINITY;
    }
    float av = -INFINITY;
#pragma unroll
    for (int q = 0; q < GN; ++q) {
      g[q] = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) g[q] = fmaxf(g[q], v[q][e]);
      av = fmaxf(av, g[q]);
    }
    // the lane's best entry ordered after (pv, pc): its value is the largest
    // group maximum (the maxima hold such entries only), its column the
    // lowest of that value in the lowest such group
    auto lane_best = [&](float pv, int pc, float& cv, int& ci) {
      cv = g[0];
#pragma unroll
      for (int q = 1; q < GN; ++q) cv = fmaxf(cv, g[q]);
      int gi = 0;
#pragma unroll
      for (int q = GN - 1; q > 0; --q) gi = g[q] == cv ? q : gi;
      gi = g[0] == cv ? 0 : gi;
      float x[8];
      group(gi, x);
      int e0 = -1;
#pragma unroll
      for (int e = 7; e >= 0; --e) {
        const int c = gi * 8 + e;
        const bool hit = (x[e] == cv) & ((cv < pv) | (cbase + c > pc)) & (c < nv);
        e0 = hit ? e : e0;
      }
      ci = (e0 >= 0 && cv != -INFINITY) ? cbase + gi * 8 + e0 : 0x7fffffff;
    };
    float cv;
    int ci;
    lane_best(INFINITY, -1, cv, ci);
    float bv = cv;
    int bi = ci;
    row_best(bv, bi);
    av = bv;
    // sum of exp(v - max) as 2^(v log2 e - max log2 e): one FMA per value
    constexpr float kL2e = 1.4426950408889634f;
    const float nb = -av * kL2e;
    float se = 0.f;
#pragma unroll
    for (int q = 0; q < GN; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) se += __builtin_amdgcn_exp2f(fmaf(v[q][e], kL2e, nb));   // 2^-inf = 0 past N
    se += quad_xor<1>(se);
    se += quad_xor<2>(se);
    const long long o = (long long)m * s.tiles + t;
    if (live && part == 0) {
      s.mx[o] = av;
      s.se[o] = se;
      s.am[o] = bi;
      if (s.kk > 0) {
        s.tv[o * s.kk] = av;
        s.tc[o * s.kk] = bi;
      }
    }
#pragma unroll 1
    for (int u = 1; u < s.kk; ++u) {
      // (bv, bi) is the previous pick: its owner takes it out of its group
      if (ci == bi && bi != 0x7fffffff) {
        const int gp = (bi - cbase) >> 3;
        float x[8], gm = -INFINITY;
        group(gp, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int c = gp * 8 + e;
          const bool after = (x[e] < bv) | ((x[e] == bv) & (cbase + c > bi));
          gm = after & (c < nv) ? fmaxf(gm, x[e]) : gm;
        }
#pragma unroll
        for (int q = 0; q < GN; ++q) g[q] = q == gp ? gm : g[q];
        lane_best(bv, bi, cv, ci);
      }
      bv = cv;
      bi = ci;
      row_best(bv, bi);
      if (live && part == 0) {
        s.tv[o * s.kk + u] = bv;
        s.tc[o * s.kk + u] = bi;
      }
    }
    if (live && s.gather_tok) {
      const int x = min(max(s.gather_tok[rowmap_index(s.gather_map, m)], 0), N - 1);
      const int c = x - cbase;
      if (c >= 0 && c < CW) s.zx[m] = rowp[(((c >> 2) ^ key) << 2) + (c & 3)];
    }
  }
}

template <int I>
using ic = std::integral_constant<int, I>;

// kEpiRope.  The tile holds whole heads.  For its rotary heads the fp32
// output tile [BM][BN] is staged in LDS (rope_at: 16-column groups
// XOR-permuted by (row / 4) % 4, so that the four row groups of an MFMA
// fragment write different banks; float4 runs stay whole), and:
//  - rotary heads (q, then k): unit = (row, head, 8 dims of the first half)
//    with its 8 partners; BM * BN / 16 units, a fixed number per thread, so
//    every row record and cos / sin load of a thread is issued before the
//    tile is staged.  q goes out as 16-byte fp32 runs, K as 16-byte runs of
//    each bf16 plane.
//  - value heads: straight from the accumulators, which hold four
//    consecutive rows (slots) of one dim per lane; a tile without rotary
//    heads is not staged.
template <int BN>
__device__ __forceinline__ int rope_at(int r, int c) {
  return r * BN + (c ^ (((r >> 2) & 3) << 4));
}

template <int NT, int BM, int PR, int BN, int HD, int TM, int TN>
__device__ __forceinline__ void rope_epilogue(const GemmArgs& a, const f32x4 (&acc)[TM * TN], float* tile, int m0,
                                              int n0, int wm, int wn, int lr, int lg) {
  constexpr int HALF = HD / 2, C8 = HALF / 8, UN = PR * BN / 16, UPT = (UN + NT - 1) / NT;
  static_assert(BN % HD == 0 && HALF % 8 == 0, "whole heads");
  const RopeEpi& re = a.re;
  const int H = re.H, Hkv = re.Hkv, Hqk = H + Hkv;
  const long long unit = split_unit_elems(HD), plane = (long long)kBlock * HD;
  bf16* kl = (bf16*)re.pool.k + (long long)re.layer * 2 * re.pool.layer_elems;
  bf16* vl = (bf16*)re.pool.v + (long long)re.layer * 2 * re.pool.layer_elems;
  const int2* __restrict__ rinfo = re.rowinfo;
  const int rows = min(BM, a.M - m0);
  const int h0 = n0 / HD, nh = min(BN, a.N - n0) / HD;
  const int nrot = max(0, min(nh, Hqk - h0));
  auto tile4 = [&](int r, int c) { return *(const float4*)&tile[rope_at<BN>(r, c)]; };

  // value columns (below) come straight from the accumulators: this lane's
  // rows' KV places are loaded up front
  const int nv = nh - nrot;
  const int rw = wm * TM * 16 + lg * 4;   // first local row of this lane
  int kvr[TM][4];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) kvr[t][e] = nv > 0 ? rinfo[m0 + min(rw + t * 16 + e, rows - 1)].x : 0;

  // rotary units u = tid + NT * w: chunk fastest, then head, then row
#pragma unroll 1
  for (int p0 = 0; p0 < BM; p0 += PR) {
    if (nrot <= 0) break;
    // cos and sin of every unit where the accumulators leave the registers
    // for them; 256 x 256 tiles, whose 128 do not, as a unit is done (prompts of
    // 4096 rows, 12288 columns: 396 us with 48 registers spilled, now 389)
    constexpr bool AHEAD = TM * TN <= 20;
    int2 ri[UPT];
    float4 cs[AHEAD ? UPT : 1][4];
    bool live[UPT];
    auto load_cs = [&](int w, float4 (&x)[4]) {
      const int d = (threadIdx.x + NT * w) % C8 * 8;
      const float* ct = re.cos_t + (long long)ri[w].y * HALF + d;
      const float* st = re.sin_t + (long long)ri[w].y * HALF + d;
      x[0] = *(const float4*)ct;
      x[1] = *(const float4*)(ct + 4);
      x[2] = *(const float4*)st;
      x[3] = *(const float4*)(st + 4);
    };
#pragma unroll
    for (int w = 0; w < UPT; ++w) {
      const int u = threadIdx.x + NT * w;
      const int r = p0 + u / (C8 * (BN / HD)), hh = u / C8 % (BN / HD);
      live[w] = u < UN && r < rows && hh < nrot;
      ri[w] = rinfo[m0 + min(r, rows - 1)];
    }
    if constexpr (AHEAD)
#pragma unroll
      for (int w = 0; w < UPT; ++w) load_cs(w, cs[w]);
    // the loads above are in flight while the tile goes to LDS (the K
    // stages' buffers are free once every wave has left the K loop)
    __syncthreads();
    const int w0 = wm * TM * 16 - p0;
    if (PR == BM || (w0 >= 0 && w0 < PR)) {
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            tile[rope_at<BN>(w0 + t * 16 + lg * 4 + e, wn * TN * 16 + j * 16 + lr)] = acc[t * TN + j][e];
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < UPT; ++w) {
      if (!live[w]) continue;
      const int u = threadIdx.x + NT * w;
      const int r = u / (C8 * (BN / HD)), hh = u / C8 % (BN / HD), d = u % C8 * 8;
      const int m = m0 + p0 + r, head = h0 + hh, lc = hh * HD + d;
      const float4 x1a = tile4(r, lc), x1b = tile4(r, lc + 4), x2a = tile4(r, lc + HALF), x2b = tile4(r, lc + HALF + 4);
      const float x1[8] = {x1a.x, x1a.y, x1a.z, x1a.w, x1b.x, x1b.y, x1b.z, x1b.w};
      const float x2[8] = {x2a.x, x2a.y, x2a.z, x2a.w, x2b.x, x2b.y, x2b.z, x2b.w};
      if constexpr (!AHEAD) load_cs(w, cs[0]);
      const float4(&q4)[4] = cs[AHEAD ? w : 0];
      const float c[8] = {q4[0].x, q4[0].y, q4[0].z, q4[0].w, q4[1].x, q4[1].y, q4[1].z, q4[1].w};
      const float sn[8] = {q4[2].x, q4[2].y, q4[2].z, q4[2].w, q4[3].x, q4[3].y, q4[3].z, q4[3].w};
      float y1[8], y2[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        y1[e] = rope_first(x1[e], x2[e], c[e], sn[e]);
        y2[e] = rope_second(x1[e], x2[e], c[e], sn[e]);
      }
      if (head < H) {
        float* q = re.qout + ((long long)m * H + head) * HD + d;
        *(float4*)q = make_float4(y1[0], y1[1], y1[2], y1[3]);
        *(float4*)(q + 4) = make_float4(y1[4], y1[5], y1[6], y1[7]);
        *(float4*)(q + HALF) = make_float4(y2[0], y2[1], y2[2], y2[3]);
        *(float4*)(q + HALF + 4) = make_float4(y2[4], y2[5], y2[6], y2[7]);
      } else {
        bf16x8 h1, l1, h2, l2;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          bf16 h, l;
          split_bf16(y1[e], h, l);
          h1[e] = h;
          l1[e] = l;
          split_bf16(y2[e], h, l);
          h2[e] = h;
          l2[e] = l;
        }
        bf16* kr = kl + ((long long)(ri[w].x / kBlock) * Hkv + (head - H)) * unit + (long long)(ri[w].x % kBlock) * HD + d;
        *(bf16x8*)kr = h1;
        *(bf16x8*)(kr + plane) = l1;
        *(bf16x8*)(kr + HALF) = h2;
        *(bf16x8*)(kr + plane + HALF) = l2;
      }
    }
  }

  if (nv <= 0) return;
  // value heads.  V is stored [hd][16 slots] per block and KV head, so a lane's four
  // consecutive rows of one dim are four consecutive slots of its dim row
  // when they lie in one block from a slot that is a multiple of 4: one
  // 8-byte store per plane; otherwise slot by slot
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn * TN * 16 + j * 16 + lr;
    const int head = col / HD;
    if (col >= a.N || head < Hqk) continue;
    const int d = col - head * HD;
    bf16* vh0 = vl + (long long)(head - Hqk) * unit + (long long)d * kBlock;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int k0 = kvr[t][0];
      const bool live0 = rw + t * 16 < rows;
      const bool run = rw + t * 16 + 3 < rows && (k0 & 3) == 0 && kvr[t][1] == k0 + 1 && kvr[t][2] == k0 + 2 &&
                       kvr[t][3] == k0 + 3;
      if (run) {
        bf16x4 hv, lv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bf16 h, l;
          split_bf16(acc[t * TN + j][e], h, l);
          hv[e] = h;
          lv[e] = l;
        }
        bf16* vr = vh0 + (long long)(k0 / kBlock) * Hkv * unit + k0 % kBlock;
        *(bf16x4*)vr = hv;
        *(bf16x4*)(vr + plane) = lv;
      } else if (live0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (rw + t * 16 + e >= rows) continue;
          bf16 h, l;
          split_bf16(acc[t * TN + j][e], h, l);
          bf16* vr = vh0 + (long long)(kvr[t][e] / kBlock) * Hkv * unit + kvr[t][e] % kBlock;
          vr[0] = h;
          vr[plane] = l;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The bf16 projection kernel: WM x WN waves, each owning TM x TN tiles of
// 16 x 16, P the prefetch distance in K stages
//
// Block tile BM x BN = (WM * TM * 16) x (WN * TN * 16), 64-deep K stages.  A
// stage is three units of 128-byte rows in LDS: W [BN][64], A_hi [BM][64] and
// A_lo [BM][64], copied from memory straight into LDS (no staging
// registers).  The units are consumed one after the other (W x A_hi, then
// W x A_lo, with the W fragments kept in registers), so a slot is free again
// as soon as its last fragments have been read: with P = 1, two W slots and three A
// slots hold a stage and a half, and every unit has at least one whole stage
// to arrive.  A wave's work on a stage is four steps, one 32-deep k-step of
// A_hi or A_lo each; the fragments of a step are read while the MFMAs of the
// step before run.  Two barriers a stage: one before the first A_lo
// fragments are read (A_hi and W are then read out), one before the next
// stage's first.
//
// 16-byte chunk c of row r sits at chunk c ^ (r & 7) of its row, so 8
// consecutive rows cover the banks exactly once.  The copies put 16 bytes
// per lane at consecutive LDS addresses, so the permutation is applied to
// the address that a lane reads.  Rows past M or N and the half stage past
// K read as zero (the buffer's range check), without memory traffic.
// ---------------------------------------------------------------------------

template <int WM, int WN, int TM, int TN, int P>
struct DenseCfg {
  static constexpr int NT = 64 * WM * WN;          // threads
  static constexpr int BM = WM * TM * 16, BN = WN * TN * 16;
  static constexpr int AU = BM * DKC * 2, WU = BN * DKC * 2;   // unit bytes
  static constexpr int RING = (P + 1) * WU + (2 * P + 1) * AU;
  // 1 KB copies per wave and unit; the copies of A_hi and A_lo are made up
  // to whole rounds of the waves with ones that read nothing and write a pad
  static constexpr int NW = WM * WN;
  static constexpr int CA = (BM / 8 + NW - 1) / NW, CW = BN / 8 / NW;
  static constexpr int PAD = BM / 8 % NW ? NW * 1024 : 0;
  // the row-statistics and rotary epilogues stage PR rows of the output
  // tile at a time in LDS
  static constexpr int NP = BM * BN * 4 <= 160 * 1024 ? 1 : 2;
  static constexpr int PR = BM / NP;
  static constexpr int TILE = PR * BN * 4;
  static constexpr int LDS = RING + PAD > TILE ? RING + PAD : TILE;
  // workgroups that share a CU: by LDS and, but for four waves of one or two
  // 16 x 16 tiles each, by registers (two waves per SIMD)
  static constexpr int OCC = 160 * 1024 / LDS;
  static constexpr int WAVES = OCC * NW / 4;   // per SIMD
  static_assert(WAVES == 2 || (WAVES == 3 && TM * TN <= 2), "the registers of the waves that LDS lets in");
  static_assert(BN / 8 % NW == 0 && LDS <= 160 * 1024 && PR % (TM * 16) == 0, "tile fits");
};

// R LDS reads and V global loads between the MF MFMAs of a step, one load
// after each of the first MFMAs
template <int R, int V, int MF>
__device__ __forceinline__ void sched_step() {
#pragma unroll
  for (int u = 0; u < (R < MF ? R : MF); ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
#pragma unroll
  for (int u = 0; u < V; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
  }
  if (MF > R + V) __builtin_amdgcn_sched_group_barrier(0x008, MF - R - V, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// EPI: 0 the stores (product, residual, SwiGLU, split planes), 1
// kEpiRowStats, 2 kEpiRope (each its own kernel, so that the registers of an
// epilogue do not weigh on the others).
// DMA: the copies go from memory straight into LDS (16-byte aligned operands
// whose tiles span less than 2 GiB: buffer offsets are 32-bit and the upper
// half marks lanes that read nothing); else through registers.
template <int WM, int WN, int TM, int TN, int P, int EPI, bool DMA = true>
__device__ __forceinline__ void gemm_bf16(const GemmArgs& a) {
  using C = DenseCfg<WM, WN, TM, TN, P>;
  constexpr int BM = C::BM, BN = C::BN, NW = WM * WN;
  __shared__ __attribute__((aligned(128))) char lds[C::LDS];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lr = lane & 15, lg = lane >> 4;
  // XCD-aware tile order.  Workgroups are dispatched round-robin over the 8
  // XCDs (each with its own L2), so workgroup p runs on XCD p % 8.  Give each
  // XCD a contiguous range of logical tiles, ordered in bands of a.band row
  // blocks (all of up to 8, else 4: an XCD's 32 tiles are then 4 x 8, which
  // read the fewest rows of two planes and columns of one; 4096 x 22016 x
  // 4096: 1236 us, 1263 with bands of 8) with the row block fastest: the tiles an XCD runs together then
  // share weight column blocks and activation row blocks through its L2.
  const int T = a.tiles_m * a.tiles_n;
  const int p = blockIdx.x, xcd = p & 7, slot = p >> 3;
  const int per = T >> 3, rem = T & 7;
  const int tile = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
  const int band = tile / (a.band * a.tiles_n), b0 = band * a.band;
  const int bh = min(a.band, a.tiles_m - b0), in = tile - b0 * a.tiles_n;
  const int tm_blk = b0 + in % bh, tn_blk = in / bh;
  const int m0 = tm_blk * BM, n0 = tn_blk * BN;
  const int kbeg = blockIdx.z * a.kchunk;
  const int klen = min(a.K - kbeg, a.kchunk);
  const int nk = (int)(((unsigned)klen + DKC - 1) / DKC);

  // copies: KB q of a unit is rows 8q .. 8q + 7; lane l reads row l / 8,
  // chunk (l % 8) ^ (l / 8) of it
  const int chunk = (lane & 7) ^ (lane >> 3);
  const unsigned row_b = (unsigned)a.K * 2;
  const unsigned voff = (unsigned)(wave * 8 + (lane >> 3)) * row_b + chunk * 16;
  const unsigned half = (klen & (DKC - 1)) && chunk >= 4 ? 0x80000000u : 0u;   // past K in the last stage
  const bf16* hi0 = a.Ahi + (long long)m0 * a.K + kbeg;
  const bf16* lo0 = a.Alo + (long long)m0 * a.K + kbeg;
  const bf16* w0 = a.B + (long long)n0 * a.K + kbeg;
  // what the copies are checked against: bytes from the unit's base (DMA), or rows
  const unsigned a_lim = (unsigned)min(BM, a.M - m0) * (DMA ? row_b : 1u) - (DMA ? kbeg * 2 : 0);
  const unsigned w_lim = (unsigned)min(BN, a.N - n0) * (DMA ? row_b : 1u) - (DMA ? kbeg * 2 : 0);
  auto copy = [&](const bf16* base, unsigned lim, int t, int dst, auto np_c, auto nb_c) __attribute__((always_inline)) {
    constexpr int np = decltype(np_c)::value, nb = decltype(nb_c)::value;   // copies per wave, 1 KB blocks of the unit
    if constexpr (!DMA) {
      // 64-bit addresses, rows and columns compared as such
      const int k = t * DKC + chunk * 8;
#pragma unroll
      for (int u = 0; u < np; ++u) {
        if (wave + NW * u >= nb) continue;
        const unsigned r = (wave + NW * u) * 8 + (lane >> 3);
        u32x4 x = {0u, 0u, 0u, 0u};
        if (t < nk && r < lim && k < klen) x = *(const u32x4*)(base + (long long)r * a.K + k);
        *(u32x4*)(lds + dst + (wave + NW * u) * 1024 + lane * 16) = x;
      }
      return;
    }
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + (long long)t * DKC), 0, t < nk ? lim - (unsigned)t * (DKC * 2) : 0u, 0x00020000);
    const unsigned vo = t == nk - 1 ? voff | half : voff;
#pragma unroll
    for (int u = 0; u < np; ++u) {
      const bool in = NW * u + NW <= nb || wave + NW * u < nb;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          r, (__attribute__((address_space(3))) void*)(lds + (in ? dst + (wave + NW * u) * 1024 : C::RING + wave * 1024)),
          16, in ? vo + (unsigned)(NW * 8 * u) * row_b : 0x80000000u, 0, 0, 0);
    }
  };
  auto copy_w = [&](int t, int slot) __attribute__((always_inline)) {
    copy(w0, w_lim, t, slot * C::WU, ic<C::CW>{}, ic<BN / 8>{});
  };
  auto copy_a = [&](const bf16* base, int t, int slot) __attribute__((always_inline)) {
    copy(base, a_lim, t, (P + 1) * C::WU + slot * C::AU, ic<C::CA>{}, ic<BM / 8>{});
  };
  // waits until at most nw W units and na A units of this wave's copies, the
  // youngest, are outstanding, and for its LDS reads; then the barrier
  auto sync = [&](auto nw_c, auto na_c) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(decltype(nw_c)::value * C::CW +
                                                                     decltype(na_c)::value * C::CA)
                 : "memory");
  };

  // fragments: row lr of a 16-row tile, chunk 4s + lg
  const int f0 = lr * 128 + ((lg ^ (lr & 7)) << 4);
  const int fa = (P + 1) * C::WU + wm * TM * 2048 + f0, fw = wn * TN * 2048 + f0;
  bf16x8 af[2][TM], wf[2][TN];
  auto read_a = [&](int slot, auto s_c) __attribute__((always_inline)) {
    constexpr int s = decltype(s_c)::value;
    const char* b = lds + ((fa + slot * C::AU) ^ (s * 64));
#pragma unroll
    for (int t = 0; t < TM; ++t) af[s][t] = *(const bf16x8*)(b + t * 2048);
  };
  auto read_w = [&](int st, auto s_c) __attribute__((always_inline)) {
    constexpr int s = decltype(s_c)::value;
    const char* b = lds + ((fw + st * C::WU) ^ (s * 64));
#pragma unroll
    for (int j = 0; j < TN; ++j) wf[s][j] = *(const bf16x8*)(b + j * 2048);
  };
  f32x4 acc[TM * TN];
#pragma unroll
  for (int v = 0; v < TM * TN; ++v) acc[v] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto mma = [&](auto s_c) __attribute__((always_inline)) {
    constexpr int s = decltype(s_c)::value;
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[t * TN + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s][t], wf[s][j], acc[t * TN + j], 0, 0, 0);
  };
  constexpr int MF = TM * TN;

  // A unit 2t is A_hi of stage t, 2t + 1 its A_lo; unit u sits in slot
  // u % (2P + 1), W of stage t in slot t % (P + 1)
  constexpr int NA = 2 * P + 1, NWS = P + 1;
#pragma unroll
  for (int t = 0; t <= P; ++t) {
    copy_w(t, t);
    copy_a(hi0, t, 2 * t % NA);
    if (t < P) copy_a(lo0, t, 2 * t + 1);
  }
  sync(ic<P>{}, ic<2 * P>{});
  read_a(0, ic<0>{});
  read_w(0, ic<0>{});
  int sh = 0, sw = 0;
  for (int t = 0; t < nk; ++t) {
    const int sl = sh + 1 == NA ? 0 : sh + 1, sn = sl + 1 == NA ? 0 : sl + 1;   // slots of A_lo, and of the next A_hi
    const int swn = sw + 1 == NWS ? 0 : sw + 1;
    __builtin_amdgcn_sched_barrier(0);
    read_a(sh, ic<1>{});
    read_w(sw, ic<1>{});
    mma(ic<0>{});
    sched_step<TM + TN, 0, MF>();
    sync(ic<P>{}, ic<2 * P - 1>{});   // A_lo is in; A_hi and W are read out
    read_a(sl, ic<0>{});
    copy_a(lo0, t + P, sh);
    copy_w(t + P + 1, sw);
    mma(ic<1>{});
    sched_step<TM, C::CA + C::CW, MF>();
    read_a(sl, ic<1>{});
    mma(ic<0>{});
    sched_step<TM, 0, MF>();
    sync(ic<P>{}, ic<2 * P - 1>{});   // the next W and A_hi are in; A_lo is read out
    read_a(sn, ic<0>{});
    read_w(swn, ic<0>{});
    copy_a(hi0, t + P + 1, sl);
    mma(ic<1>{});
    sched_step<TM + TN, C::CA, MF>();
    sh = sn;
    sw = swn;
  }
  sync(ic<0>{}, ic<0>{});   // the copies past the last stage

  const int rbase = m0 + wm * TM * 16 + lg * 4, cbase = n0 + wn * TN * 16 + lr;
  if constexpr (EPI == 1) {
    // the units are consumed: the tile goes through LDS for the row pass
    float* tile = reinterpret_cast<float*>(lds);
#pragma unroll 1
    for (int ps = 0; ps < C::NP; ++ps) {
      __syncthreads();
      const int r0 = wm * TM * 16 - ps * C::PR;
      if (C::NP == 1 || (r0 >= 0 && r0 < C::PR)) {
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              tile[RsLayout<C::NT, C::PR, BN>::at(r0 + t * 16 + lg * 4 + e, wn * TN * 16 + j * 16 + lr)] =
                  acc[t * TN + j][e];
      }
      __syncthreads();
      tile_row_stats<C::NT, C::PR, BN>(tile, m0 + ps * C::PR, n0, a.M, a.N, tn_blk, a.rs);
    }
    return;
  }
  if constexpr (EPI == 2) {
    float* tile = reinterpret_cast<float*>(lds);
    if constexpr (BN % 128 == 0) {
      if (a.re.hd == 128) {
        rope_epilogue<C::NT, BM, C::PR, BN, 128, TM, TN>(a, acc, tile, m0, n0, wm, wn, lr, lg);
        return;
      }
    }
    rope_epilogue<C::NT, BM, C::PR, BN, 64, TM, TN>(a, acc, tile, m0, n0, wm, wn, lr, lg);
    return;
  }
  if constexpr (TN % 2 == 1) {
    if (a.epi == kEpiSwiGLU && a.ksplit == 1) {
      // a gate tile and its up tile are in two waves: through LDS
      float* tile = reinterpret_cast<float*>(lds);
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            tile[(wm * TM * 16 + t * 16 + lg * 4 + e) * BN + wn * TN * 16 + j * 16 + lr] = acc[t * TN + j][e];
      __syncthreads();
      for (int u = tid; u < BM * BN / 2; u += C::NT) {
        const int r = u / (BN / 2), f = u % (BN / 2), c = (f >> 4) * 32 + (f & 15);
        epi_swiglu(a, m0 + r, n0 + c, tile[r * BN + c], tile[r * BN + c + 16]);
      }
      return;
    }
  }
  if (a.ksplit > 1) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) part_store(a, rbase + t * 16 + e, cbase + j * 16, acc[t * TN + j][e]);
    return;
  }
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = rbase + t * 16 + e, col = cbase + j * 16;
        if (a.epi == kEpiSwiGLU) {
          if (j + 1 < TN && (j & 1) == 0) epi_swiglu(a, row, col, acc[t * TN + j][e], acc[t * TN + j + 1][e]);
        } else {
          epi_store(a, row, col, acc[t * TN + j][e]);
        }
      }
}

}  // namespace

// One kernel per (configuration, epilogue) under the given name, and the
// function that launches it.
#define CDSL_GEMM_KERNELS(KERNEL, LAUNCH)                                                                   \
  namespace {                                                                                               \
  template <int WM, int WN, int TM, int TN, int P, int EPI, bool DMA, int KIND>                             \
  __global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(                                    \
      2, DenseCfg<WM, WN, TM, TN, P>::WAVES))) void KERNEL(GemmArgs a) {                                    \
    gemm_bf16<WM, WN, TM, TN, P, EPI, DMA>(a);                                                              \
  }                                                                                                         \
  }                                                                                                         \
  void LAUNCH(int cfg, int epi, dim3 grid, const GemmArgs& a, hipStream_t st) {                             \
    switch (cfg * 3 + epi) { CDSL_GEMM_CFGS(CDSL_GEMM_CASE) }                                               \
  }

}  // namespace cdsl
