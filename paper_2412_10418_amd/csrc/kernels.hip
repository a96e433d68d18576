// Row-wise kernels of the CDSL step: embedding gather, RMSNorm, rotary
// embedding + KV write, the fused log-softmax / gather / argmax / top-k of a
// logits row, hard rejection and beam scores, rewards, beam selection, and
// the commit (emit, next beams, prefix promotion).
#include <float.h>

#include "block_pool.h"
#include "common.h"
#include "kernels.h"

namespace cdsl {

namespace {

template <int NW>
__device__ __forceinline__ float block_sum(float v, float* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int u = 0; u < NW; ++u) t += sh[u];
  return t;
}

// ---------------------------------------------------------------------------
// A token id outside [0, V) sets *bad (the library reports it as an invalid
// argument at its next synchronisation) and is clamped for the read, so it
// never reads out of bounds.
// With rowinfo, row m's KV place is also recorded for the pass's layers:
// rowinfo[m] = (block * 16 + slot, position).
template <typename T>
__global__ __launch_bounds__(256) void embed_rows(PassDesc p, const T* __restrict__ emb, float* __restrict__ h,
                                                  int D, int V, int* __restrict__ bad, int2* __restrict__ rowinfo) {
  const int m = blockIdx.x;
  int bi, b, i, j;
  row_decode(p, m, bi, b, i, j);
  if (rowinfo && threadIdx.x == 0) {
    int blk, slot, pos;
    kv_slot(p, b, i, j, p.Lp[b], blk, slot, pos);
    rowinfo[m] = make_int2(blk * kBlock + slot, pos);
  }
  const int raw = p.tok[(long long)(b * p.kp + i) * p.tok_stride + p.tok_off + j];
  if ((raw < 0 || raw >= V) && threadIdx.x == 0 && bad) *bad = 1;
  const int tok = min(max(raw, 0), V - 1);
  const T* e = emb + (long long)tok * D;
  float* o = h + (long long)m * D;
  for (int c = threadIdx.x; c < D; c += 256) o[c] = to_f32<T>(e[c]);
}

// out[r] = x[src(r)] / sqrt(mean(x^2) + eps) * g.  src(r) = r, or the last
// row of beam r when last_only (prompt prefill: only the last position needs
// logits).  The result goes to out32 (fp32) or, for bf16-weight models, to
// the hi / lo planes that the next projection consumes.  hid (fp32)
// additionally receives the normed row of every beam's last row (the reward
// reads it).
//
// With S > 0 split planes part[S][rows][D] of a residual projection, the
// row is first completed: x[r] += sum of the planes in split order (the
// same arithmetic as the split-K reduce), written back to x.  g == null
// then only folds.
// The row stays in registers between the two phases: float4 column groups
// threadIdx.x + NT * u, u < kNormU (D <= 4 * NT * kNormU).
constexpr int kNormU = 8;

template <int NT>
__global__ __launch_bounds__(NT) void rmsnorm_rows(float* __restrict__ x, const float* __restrict__ g,
                                                    float* __restrict__ out32, bf16* __restrict__ ohi,
                                                    bf16* __restrict__ olo, int D, float eps, int last_only, int R,
                                                    float* __restrict__ hid, const float* __restrict__ part, int S,
                                                    int rows) {
  __shared__ float sh[NT / 64];
  const int r = blockIdx.x;
  const int src = last_only ? r * R + (R - 1) : r;
  float* xr = x + (long long)src * D;
  float4 v[kNormU];
  float ss = 0.f;
  const long long plane = (long long)rows * D;
  const float* pr = part + (long long)src * D;
#pragma unroll
  for (int u = 0; u < kNormU; ++u) {
    const int c = (threadIdx.x + NT * u) * 4;
    v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c >= D) continue;
    if (S > 0) {
      // the planes are loaded eight at a time (independent loads in flight)
      // and added in split order
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int z0 = 0; z0 < S; z0 += 8) {
        float4 t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          t[e] = z0 + e < S ? *(const float4*)(pr + (z0 + e) * plane + c) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (z0 + e < S) {
            a.x += t[e].x;
            a.y += t[e].y;
            a.z += t[e].z;
            a.w += t[e].w;
          }
      }
      const float4 h = *(const float4*)(xr + c);
      a.x += h.x;
      a.y += h.y;
      a.z += h.z;
      a.w += h.w;
      *(float4*)(xr + c) = a;
      v[u] = a;
    } else {
      v[u] = *(const float4*)(xr + c);
    }
    ss = fmaf(v[u].x, v[u].x, ss);
    ss = fmaf(v[u].y, v[u].y, ss);
    ss = fmaf(v[u].z, v[u].z, ss);
    ss = fmaf(v[u].w, v[u].w, ss);
  }
  if (!g) return;
  ss = block_sum<NT / 64>(ss, sh);
  const float inv = rsqrtf(ss / (float)D + eps);
  const long long o = (long long)r * D;
  const bool want_hid = hid && (last_only || (r % R) == R - 1);
  float* hr = want_hid ? hid + (long long)(last_only ? r : r / R) * D : nullptr;
#pragma unroll
  for (int u = 0; u < kNormU; ++u) {
    const int c = (threadIdx.x + NT * u) * 4;
    if (c >= D) continue;
    const float4 gg = *(const float4*)(g + c);
    const float4 y = make_float4(v[u].x * inv * gg.x, v[u].y * inv * gg.y, v[u].z * inv * gg.z, v[u].w * inv * gg.w);
    if (out32) {
      *(float4*)(out32 + o + c) = y;
    } else {
      bf16x4 h4, l4;
      const float yy[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bf16 h, l;
        split_bf16(yy[e], h, l);
        h4[e] = h;
        l4[e] = l;
      }
      *(bf16x4*)(ohi + o + c) = h4;
      *(bf16x4*)(olo + o + c) = l4;
    }
    if (hr) *(float4*)(hr + c) = y;
  }
}

// Rotary embedding of q and k (rotate-half pairs (d, d + hd/2), angle
// pos * theta^(-2d/hd) from the host-built tables), then q -> Q buffer and
// k, v -> the row's KV slot: prefix block for kAppend, the beam's suffix
// block for kSuffix.
template <typename T>
__global__ __launch_bounds__(256) void rope_kv_write(PassDesc p, const float* __restrict__ qkv, T* __restrict__ qout,
                                                     KVPool pool, int layer, const float* __restrict__ cos_t,
                                                     const float* __restrict__ sin_t, int H, int Hkv, int hd) {
  const int m = blockIdx.x;
  int bi, b, i, j;
  row_decode(p, m, bi, b, i, j);
  int pos, blk, slot;
  kv_slot(p, b, i, j, p.Lp[b], blk, slot, pos);
  const int half = hd / 2;
  const float* row = qkv + (long long)m * (H + 2 * Hkv) * hd;
  const float* ct = cos_t + (long long)pos * half;
  const float* stt = sin_t + (long long)pos * half;
  T* kb = (T*)pool.k + (long long)layer * pool.layer_elems + ((long long)blk * Hkv) * kBlock * hd;
  T* vb = (T*)pool.v + (long long)layer * pool.layer_elems + ((long long)blk * Hkv) * kBlock * hd;
  // q and k heads: pairs
  const int npairs = (H + Hkv) * half;
  for (int u = threadIdx.x; u < npairs; u += 256) {
    const int hh = u / half, d = u % half;
    const float x1 = row[hh * hd + d], x2 = row[hh * hd + d + half];
    const float c = ct[d], s = stt[d];
    const float y1 = rope_first(x1, x2, c, s), y2 = rope_second(x1, x2, c, s);
    if (hh < H) {
      T* q = qout + ((long long)m * H + hh) * hd;
      q[d] = from_f32<T>(y1);
      q[d + half] = from_f32<T>(y2);
    } else {
      T* kr = kb + ((long long)(hh - H) * kBlock + slot) * hd;
      kr[d] = from_f32<T>(y1);
      kr[d + half] = from_f32<T>(y2);
    }
  }
  // v: transposed [hd][16] per block and head
  const float* vrow = row + (long long)(H + Hkv) * hd;
  for (int u = threadIdx.x; u < Hkv * hd; u += 256) {
    const int hh = u / hd, d = u % hd;
    vb[((long long)hh * hd + d) * kBlock + slot] = from_f32<T>(vrow[u]);
  }
}

// Same for bf16-weight models, whose KV pool holds each fp32 value as a
// bf16 (hi, lo) pair in the split unit format (K [plane][16][hd], V
// [plane][hd][16]).  q stays fp32.  With S > 0, qkv holds S split planes
// [S][M][(H + 2 Hkv) hd] of the projection, summed here in split order.
//
// Workgroups 0..M-1 take one row each (rotary q and k, the K write).
// Workgroups M.. take a (beam, KV head, block of slots) each, one thread per
// head dim, and write V: the rows of a beam sit in consecutive slots, so each
// thread writes a run of slots of its dim row with wide stores instead of one
// 2-byte store per row into a different 32-byte row.
struct QkvRow {
  const float* qkv;
  long long split_plane;
  int S;
  // four consecutive values of row m at column idx (summed over the split
  // planes in split order, eight planes' loads in flight at a time)
  __device__ __forceinline__ float4 val4(long long m, int W, int idx) const {
    const float* row = qkv + m * W;
    if (S <= 0) return *(const float4*)(row + idx);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z0 = 0; z0 < S; z0 += 8) {
      float4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        t[u] = z0 + u < S ? *(const float4*)(row + (z0 + u) * split_plane + idx) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z0 + u < S) {
          v.x += t[u].x;
          v.y += t[u].y;
          v.z += t[u].z;
          v.w += t[u].w;
        }
    }
    return v;
  }
};

// the blocks of 16 slots that R consecutive rows reach at most
__host__ __device__ inline int v_blocks(int R) { return (R + kBlock - 2) / kBlock + 1; }

template <int NT>
__global__ __launch_bounds__(NT) void rope_kv_write_split(PassDesc p, const float* __restrict__ qkv,
                                                           float* __restrict__ qout, KVPool pool, int layer,
                                                           const float* __restrict__ cos_t,
                                                           const float* __restrict__ sin_t, int H, int Hkv, int hd,
                                                           int S) {
  const int M = p.nb * p.kp * p.R;
  const int W = (H + 2 * Hkv) * hd;
  const QkvRow src{qkv, (long long)M * W, S};
  const int half = hd / 2;
  const long long unit = split_unit_elems(hd);
  const long long plane = (long long)kBlock * hd;
  bf16* kl = (bf16*)pool.k + (long long)layer * 2 * pool.layer_elems;
  bf16* vl = (bf16*)pool.v + (long long)layer * 2 * pool.layer_elems;
  if ((int)blockIdx.x < M) {
    const int m = blockIdx.x;
    int bi, b, i, j;
    row_decode(p, m, bi, b, i, j);
    int blk, slot, pos;
    kv_slot(p, b, i, j, p.Lp[b], blk, slot, pos);
    const float* ct = cos_t + (long long)pos * half;
    const float* stt = sin_t + (long long)pos * half;
    bf16* kb = kl + (long long)blk * Hkv * unit;
    // q and k heads: rotate-half pairs (d, d + hd/2), four d at a time
    const int q4 = half / 4;
    for (int u = threadIdx.x; u < (H + Hkv) * q4; u += NT) {
      const int hh = u / q4, d = (u % q4) * 4;
      const float4 x1 = src.val4(m, W, hh * hd + d), x2 = src.val4(m, W, hh * hd + d + half);
      const float4 c = *(const float4*)(ct + d), sn = *(const float4*)(stt + d);
      const float y1[4] = {rope_first(x1.x, x2.x, c.x, sn.x), rope_first(x1.y, x2.y, c.y, sn.y),
                           rope_first(x1.z, x2.z, c.z, sn.z), rope_first(x1.w, x2.w, c.w, sn.w)};
      const float y2[4] = {rope_second(x1.x, x2.x, c.x, sn.x), rope_second(x1.y, x2.y, c.y, sn.y),
                           rope_second(x1.z, x2.z, c.z, sn.z), rope_second(x1.w, x2.w, c.w, sn.w)};
      if (hh < H) {
        float* q = qout + ((long long)m * H + hh) * hd + d;
        *(float4*)q = make_float4(y1[0], y1[1], y1[2], y1[3]);
        *(float4*)(q + half) = make_float4(y2[0], y2[1], y2[2], y2[3]);
      } else {
        bf16* kr = kb + (long long)(hh - H) * unit + (long long)slot * hd + d;
        bf16x4 h1, l1, h2, l2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bf16 h, l;
          split_bf16(y1[e], h, l);
          h1[e] = h;
          l1[e] = l;
          split_bf16(y2[e], h, l);
          h2[e] = h;
          l2[e] = l;
        }
        *(bf16x4*)kr = h1;
        *(bf16x4*)(kr + plane) = l1;
        *(bf16x4*)(kr + half) = h2;
        *(bf16x4*)(kr + plane + half) = l2;
      }
    }
    return;
  }
  // V of (beam group, KV head, block of slots) tasks, NT / hd of them per
  // workgroup: thread d < hd of a task owns dim row d
  const int per = NT / hd, nq = v_blocks(p.R);
  const int task = ((int)blockIdx.x - M) * per + (int)threadIdx.x / hd;
  const int d = (int)threadIdx.x % hd;
  if ((int)threadIdx.x >= per * hd || task >= p.nb * p.kp * Hkv * nq) return;
  const int q = task % nq, hh = task / nq % Hkv, g = task / nq / Hkv;
  const int bi = g / p.kp, i = g % p.kp;
  const int b = pass_batch(p, bi);
  const int Lp = p.Lp[b];
  int blk, slot, pos;
  kv_slot(p, b, i, 0, Lp, blk, slot, pos);
  const int j = q == 0 ? 0 : q * kBlock - slot;   // the first row in this block
  if (j >= p.R) return;
  if (q > 0) kv_slot(p, b, i, j, Lp, blk, slot, pos);
  const int n = min(p.R - j, kBlock - slot);      // its rows: slots [slot, slot + n)
  // the loads of every row and of four split planes are issued before any is
  // used: one latency per four planes (a beam's blocks one after the other, and
  // one latency per value and plane, made 105 rows of prompts, split in five,
  // 17 us instead of 8)
  const float* vr = qkv + ((long long)g * p.R + j - slot) * W + (H + Hkv) * hd + hh * hd + d;
  auto row_in = [&](int t) { return t >= slot && t < slot + n; };
  float vv[kBlock];
#pragma unroll
  for (int t = 0; t < kBlock; ++t) vv[t] = S <= 0 && row_in(t) ? vr[(long long)t * W] : 0.f;
  for (int z0 = 0; z0 < S; z0 += 4) {
    float x[4][kBlock];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int t = 0; t < kBlock; ++t)
        x[u][t] = row_in(t) ? vr[min(z0 + u, S - 1) * src.split_plane + (long long)t * W] : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (z0 + u < S)
#pragma unroll
        for (int t = 0; t < kBlock; ++t) vv[t] += x[u][t];
  }
  store_v_run(vl + ((long long)blk * Hkv + hh) * unit + (long long)d * kBlock, plane, vv, slot, n);
}

// ---------------------------------------------------------------------------
// A token id that indexes the vocabulary even for a row without a finite
// logit (all NaN), so that the next pass's embedding never reads out of
// bounds; the NaN still reaches the scores and makes the selection fail.
__device__ __forceinline__ int vocab_id(int id, int V) { return (id >= 0 && id < V) ? id : 0; }

// The kk best entries (value descending, id ascending) of a row whose entries
// are spread over a workgroup's threads, in one round whatever kk <= 16 is:
// each thread offers its best entry, 32 groups of threads (by tid % 32) keep
// theirs, and the kk-th best of those bounds the kk-th best of the row.  The
// entries at or above the bound are collected (for values in no order about
// 32 ln(32 / (32 - kk)): 5 at five places, 22 at sixteen; sixteen groups let
// through 54 at sixteen places, and often twice that) and ranked by counting.
constexpr int kTopList = 512;   // entries that a workgroup collects at most
constexpr int kTopGroups = 32;
constexpr int kNoId = 0x7fffffff;

template <int NW>
struct TopShared {
  float gv[NW][kTopGroups];
  int gi[NW][kTopGroups];
  int n;
  float v[kTopList];
  int id[kTopList];
};

// rank += how many of a row of 16 lanes hold a better entry than (v, i),
// each lane holding (ov, oi)
template <int O = 0>
__device__ __forceinline__ void row_rank(float ov, int oi, float v, int i, int& rank) {
  float rv = ov;
  int ri = oi;
  if constexpr (O > 0) {
    rv = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(ov), 0x120 + O, 0xF, 0xF, true));
    ri = __builtin_amdgcn_mov_dpp(oi, 0x120 + O, 0xF, 0xF, true);
  }
  rank += vi_better(rv, ri, v, i) ? 1 : 0;
  if constexpr (O < 15) row_rank<O + 1>(ov, oi, v, i, rank);
}

__device__ __forceinline__ void xor_best(int o, float& v, int& id) {
  const float ov = __shfl_xor(v, o, 64);
  const int oi = __shfl_xor(id, o, 64);
  if (vi_better(ov, oi, v, id)) v = ov, id = oi;
}

// before the barrier: this thread's best entry (id kNoId: none)
template <int NW>
__device__ __forceinline__ void top_offer(float v, int id, TopShared<NW>& t) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  xor_best(32, v, id);
  if (lane < kTopGroups) {
    t.gv[w][lane] = v;
    t.gi[w][lane] = id;
  }
  if (threadIdx.x == 0) t.n = 0;
}

// after it: the bound (bv, bi) that the kk-th best entry of the row reaches
// ((-inf, about kNoId) where the groups hold fewer entries), and the row's
// best value
template <int NW>
__device__ __forceinline__ void top_bound(const TopShared<NW>& t, int kk, float& bv, int& bi, float& best) {
  const int lane = threadIdx.x & 63, j = lane & 31;
  float v = -INFINITY;
  int id = kNoId;
#pragma unroll
  for (int w0 = 0; w0 < NW; w0 += 2) {
    const int w = min(w0 + (lane >> 5), NW - 1);
    const float ov = t.gv[w][j];
    const int oi = t.gi[w][j];
    if (vi_better(ov, oi, v, id)) v = ov, id = oi;
  }
  if (NW > 1) xor_best(32, v, id);
  id = min(id, kNoId - kTopGroups + j);   // groups without an entry differ
  int rank = 0;
  row_rank(v, id, v, id, rank);
  row_rank(__shfl_xor(v, 16, 64), __shfl_xor(id, 16, 64), v, id, rank);
  const int at = __builtin_ctzll(__ballot(rank == kk - 1)), first = __builtin_ctzll(__ballot(rank == 0));
  bv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), at));
  bi = __builtin_amdgcn_readlane(id, at);
  best = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), first));
}

// the entries of x whose bit of mask is set; id_of(e) is the id of x[e]
template <int NW, int N, typename Id>
__device__ __forceinline__ void top_push(const float (&x)[N], unsigned mask, Id id_of, TopShared<NW>& t) {
  if (!mask) return;
  int at = atomicAdd(&t.n, __popc(mask));
#pragma unroll
  for (int e = 0; e < N; ++e)
    if (mask >> e & 1) {
      if (at < kTopList) {
        t.v[at] = x[e];
        t.id[at] = id_of(e);
      }
      ++at;
    }
}

// after the barrier that follows the pushes: put(place, value, id) for every
// place below kk (places that no entry is left for: -inf, kNoId)
template <int NW, typename Put>
__device__ __forceinline__ void top_place(const TopShared<NW>& t, int n, int kk, Put put) {
  for (int i = threadIdx.x; i < n; i += 64 * NW) {
    const float v = t.v[i];
    const int id = t.id[i];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) rank += vi_better(t.v[j], t.id[j], v, id) ? 1 : 0;
    if (rank < kk) put(rank, v, id);
  }
  if ((int)threadIdx.x >= n && (int)threadIdx.x < kk) put(threadIdx.x, -INFINITY, kNoId);
}

// the best entry of a workgroup (every thread returns it); the barrier before
// the next call of it is the caller's
template <int NW>
__device__ __forceinline__ void top_one(float& v, int& id, TopShared<NW>& t) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) xor_best(o, v, id);
  if ((threadIdx.x & 63) == 0) {
    t.gv[threadIdx.x >> 6][0] = v;
    t.gi[threadIdx.x >> 6][0] = id;
  }
  __syncthreads();
  v = t.gv[0][0];
  id = t.gi[0][0];
#pragma unroll
  for (int u = 1; u < NW; ++u)
    if (vi_better(t.gv[u][0], t.gi[u][0], v, id)) v = t.gv[u][0], id = t.gi[u][0];
}

// A row of V floats read as 16-byte slots: slot q holds ids 4q - shift .. + 3,
// shift chosen so that the slots are aligned whatever V and the row are.  Ids
// outside the row read as -inf.
struct RowSlots {
  const float* z;
  int V, shift, slots;
  bool vec;   // the slots of this row are 16-byte aligned
  __device__ __forceinline__ void load(int q, float (&x)[4]) const {
    const int id = 4 * q - shift;
    if (vec && id >= 0 && id + 4 <= V) {
      const float4 v = *(const float4*)(z + id);
      x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = id + e >= 0 && id + e < V ? z[id + e] : -INFINITY;
    }
  }
};
__device__ __forceinline__ RowSlots row_slots(const float* z, int V, int shift) {
  return {z, V, shift, (V + shift + 3) / 4, ((uintptr_t)z / 4 & 3) == (unsigned)shift};
}

constexpr float kLog2e = 1.4426950408889634f;

// Adds N values to a running (maximum m, sum s of exp(v - m)).  A chunk's own
// maximum is taken first, so s is scaled at most once per chunk; a NaN among
// the values makes s NaN.
template <int N>
__device__ __forceinline__ void lse_add(const float (&x)[N], float cm, float& m, float& s) {
  const float mn = fmaxf(m, cm);
  if (mn == -INFINITY) {
#pragma unroll
    for (int e = 0; e < N; ++e)
      if (x[e] != x[e]) s = x[e];
    return;
  }
  s *= __builtin_amdgcn_exp2f((m - mn) * kLog2e);   // m = -inf: 0
  m = mn;
#pragma unroll
  for (int e = 0; e < N; ++e) s += __builtin_amdgcn_exp2f((x[e] - mn) * kLog2e);
}

// the logsumexp of a workgroup's (m, s): put before a barrier, then taken by
// every thread
template <int NW>
__device__ __forceinline__ void lse_put(float m, float s, float (&sm)[NW], float (&ss)[NW]) {
  const float wm = wave_max(m);
  const float ws = wave_sum(wm == -INFINITY ? s : s * __builtin_amdgcn_exp2f((m - wm) * kLog2e));
  if ((threadIdx.x & 63) == 0) {
    sm[threadIdx.x >> 6] = wm;
    ss[threadIdx.x >> 6] = ws;
  }
}
template <int NW>
__device__ __forceinline__ float lse_take(const float (&sm)[NW], const float (&ss)[NW]) {
  float M = -INFINITY, t = 0.f;
#pragma unroll
  for (int u = 0; u < NW; ++u) M = fmaxf(M, sm[u]);
#pragma unroll
  for (int u = 0; u < NW; ++u) t += sm[u] == -INFINITY ? ss[u] : ss[u] * __builtin_amdgcn_exp2f((sm[u] - M) * kLog2e);
  return M + __logf(t);
}

// Logits row statistics, one workgroup per row, one read of the row: online
// logsumexp, argmax, top-kk.  Ordering: value descending, then id ascending.
//
// Bound by the read.  A thread keeps the maximum of each of its GN groups of
// columns (16 columns of every GN-th chunk) and the first slot that holds its
// best, which is what it offers; only the groups that reach the bound are read
// again (from L2).  Places taken one by one, each with two dependent reads and
// a round of the workgroup, cost 2 to 3 us apiece: 500 rows of 50257, top-5,
// took 37 us, now 32; 20 rows of 1000, top-16, 58, now 11.
template <int NT, bool LSE, bool ONE>   // ONE: kk <= 1
__global__ __launch_bounds__(NT) void logit_rows_kernel(LogitArgs a) {
  constexpr int NW = NT / 64, GN = 4;
  __shared__ TopShared<NW> top;
  __shared__ float sm[NW], ss[NW];
  const int row = blockIdx.x;
  const int tid = threadIdx.x;
  const float* z = a.logits + (long long)row * (a.ld ? a.ld : (long long)a.V);
  const RowSlots rs = row_slots(z, a.V, (int)((uintptr_t)z / 4 & 3));
  const int nc = (rs.slots + 4 * NT - 1) / (4 * NT);   // chunks of 4 slots per thread
  auto chunk = [&](int c, float (&x)[16]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float t[4];
      rs.load(tid + NT * (4 * c + i), t);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * i + e] = t[e];
    }
  };
  auto id_of = [&](int c, int e) { return 4 * (tid + NT * (4 * c + (e >> 2))) - rs.shift + (e & 3); };

  float g[GN], m = -INFINITY, s = 0.f, bv = -INFINITY;
  int bs = kNoId;   // the first slot that holds this thread's best value bv
#pragma unroll
  for (int u = 0; u < GN; ++u) g[u] = -INFINITY;
  for (int c0 = 0; c0 < nc; c0 += GN) {
#pragma unroll
    for (int u = 0; u < GN; ++u) {
      if (c0 + u >= nc) break;
      float x[16], sx[4];
      chunk(c0 + u, x);
#pragma unroll
      for (int i = 0; i < 4; ++i) sx[i] = fmaxf(fmaxf(x[4 * i], x[4 * i + 1]), fmaxf(x[4 * i + 2], x[4 * i + 3]));
      float cm = fmaxf(fmaxf(sx[0], sx[1]), fmaxf(sx[2], sx[3]));
      cm = fmaxf(cm, -INFINITY);   // all NaN: -inf
      g[u] = fmaxf(g[u], cm);
      if (cm > bv) {
        bv = cm;
        bs = tid + NT * (4 * (c0 + u) + (sx[0] == cm ? 0 : sx[1] == cm ? 1 : sx[2] == cm ? 2 : 3));
      }
      if (LSE) lse_add(x, cm, m, s);
    }
  }
  if (bv == -INFINITY) {
    // nothing above -inf: the first slot with a -inf of the row itself (the
    // row may begin and end inside a slot)
    for (int q = tid; q < rs.slots && bs == kNoId; q += NT) {
      float x[4];
      rs.load(q, x);
      const int id = 4 * q - rs.shift;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (x[e] == bv && id + e >= 0 && id + e < a.V) bs = q;
    }
  }
  const int dst = a.topk_rows ? a.topk_rows[row] : row;
  float lse = 0.f;
  auto put = [&](int r, float v, int id) {
    if (r == 0 && a.amax) a.amax[rowmap_index(a.amax_map, row)] = vocab_id(id, a.V);
    if (!LSE || r >= a.kk) return;
    a.topk_ids[(long long)dst * a.kk + r] = vocab_id(id, a.V);
    a.topk_lp[(long long)dst * a.kk + r] = v - lse;
  };
  auto gather = [&]() {
    if (!LSE || !a.lp || tid != 0) return;
    const int tok = a.gather_tok[rowmap_index(a.gather_map, row)];
    const bool in = tok >= 0 && tok < a.V;
    if (!in && a.bad) *a.bad = 1;
    a.lp[row] = in ? z[tok] - lse : __int_as_float(0x7fc00000);
  };
  if (LSE) lse_put<NW>(m, s, sm, ss);
  if constexpr (ONE) {
    top_one<NW>(bv, bs, top);
    if (LSE) lse = lse_take<NW>(sm, ss);
    gather();
    // the thread that read the slot finds the first of its four ids
    if (tid == (bs == kNoId ? 0 : bs % NT)) {
      int id = kNoId;
      if (bs != kNoId) {
        float x[4];
        rs.load(bs, x);
#pragma unroll
        for (int e = 3; e >= 0; --e) {
          const int t = 4 * bs - rs.shift + e;
          if (x[e] == bv && t >= 0 && t < a.V) id = t;
        }
      }
      put(0, bv, id);
    }
    return;
  }
  top_offer<NW>(bv, bs, top);
  __syncthreads();
  if (LSE) lse = lse_take<NW>(sm, ss);
  gather();
  float cv, best;
  int ci;
  top_bound<NW>(top, a.kk, cv, ci, best);
  // at least kk entries are above cv, or equal to it with an id up to ci
  ci = ci >= kNoId - kTopGroups ? kNoId : 4 * ci + 3 - rs.shift;
  if (bv >= cv) {
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
      float gc = g[0];
#pragma unroll
      for (int u = 1; u < GN; ++u) gc = (c & (GN - 1)) == u ? g[u] : gc;
      if (gc < cv || (gc == cv && id_of(c, 0) > ci)) continue;
      float x[16];
      chunk(c, x);
      unsigned mask = 0;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int id = id_of(c, e);
        mask |= ((x[e] > cv || (x[e] == cv && id <= ci)) && id >= 0 && id < a.V ? 1u : 0u) << e;
      }
      top_push<NW>(x, mask, [&](int e) { return id_of(c, e); }, top);
    }
  }
  __syncthreads();
  const int n = top.n;
  if (n <= kTopList) {
    top_place<NW>(top, n, a.kk, put);
    return;
  }
  // more entries at the bound than the list holds (the best entries all with
  // few threads): place by place
  float pv = INFINITY;
  int pi = -1;
  for (int r = 0; r < a.kk; ++r) {
    float v = -INFINITY;
    int id = kNoId;
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
      float x[16];
      chunk(c, x);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int t = id_of(c, e);
        if (t >= 0 && t < a.V && vi_better(pv, pi, x[e], t) && vi_better(x[e], t, v, id)) v = x[e], id = t;
      }
    }
    __syncthreads();
    top_one<NW>(v, id, top);
    pv = v;
    pi = id;
    if (tid == 0) put(r, pv, pi);
  }
}

// ---------------------------------------------------------------------------
// Hard rejection (leading matches of target argmax and lookahead) and beam
// scores, one thread per (b, i).
// With lq and u (soft rejection, speculative sampling): x_j is kept while
// u_j <= min(1, p_j(x_j) / q_j(x_j)), the ratio formed from the two log-probs.
__global__ void beam_scores_kernel(int BK, int d, const int* __restrict__ look, const int* __restrict__ y,
                                   const float* __restrict__ lp, const float* __restrict__ head_lp,
                                   const float* __restrict__ lq, const float* __restrict__ u,
                                   int* __restrict__ n_accept, float* __restrict__ scores) {
  const int bk = blockIdx.x * blockDim.x + threadIdx.x;
  if (bk >= BK) return;
  int n = 0;
  bool run = true;
  float s = head_lp ? head_lp[bk] : 0.f;
  for (int j = 0; j < d; ++j) {
    const long long r = (long long)bk * d + j;
    bool keep;
    if (lq) keep = u[r] <= fminf(1.f, expf(lp[r] - lq[r]));
    else keep = y[r] == look[(long long)bk * (d + 1) + j + 1];
    if (run && keep) ++n;
    else run = false;
    s += lp[r];
  }
  n_accept[bk] = n;
  scores[bk] = s;
}

// first_at (optional, [B]): Step-1 of the controller with b = 1 keeps the
// greedy head (beam 0) when its reward reaches first_at[b]; NaN = no such rule.
__global__ void select_kernel(int B, int k, const float* __restrict__ scores, const float* __restrict__ reward,
                              float alpha, int reward_only, const float* __restrict__ first_at,
                              int* __restrict__ beam) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  if (first_at) {
    const float t = first_at[b], r0 = reward[b * k];
    if (isnan(r0)) {
      beam[b] = -1;
      return;
    }
    if (!isnan(t) && r0 >= t) {
      beam[b] = 0;
      return;
    }
  }
  int best = -1;
  float bv = -INFINITY;
  bool bad = false;
  for (int i = 0; i < k; ++i) {
    const float sc = scores[b * k + i], r = reward[b * k + i];
    if (isnan(sc) || isnan(r)) bad = true;
    const float v = reward_only ? r : sc + alpha * r;
    if (best < 0 || v > bv) {
      best = i;
      bv = v;
    }
  }
  beam[b] = bad ? -1 : best;
}

// Speculative sampling rows (Sec. 3.2.2), one workgroup per fed row m of a
// verification (rows ordered (b, i, j), both logit arrays [M][V]):
//   draft_lp[m] = log q(x), x the row's lookahead token;
//   res_ids[m]  = the draw at v[m] from w = max(0, p - q) / Z, inverting the
//                 cumulative sum over token ids in ascending order (argmax p
//                 when Z = 0), and res_lp[m] = log p of it.
//
// Bound by the two reads of the two rows, from HBM and then from the caches
// (holding both rows in the registers of 1024 threads leaves one workgroup per
// CU, whose loads and sums then do not overlap: 91 against 78 us for 800 rows
// of 32000; the floor of one read is 45 us).  Blocks of 4 NT consecutive ids
// (f of them per segment) are summed per wave; the segment that holds v * Z,
// then its block, its wave (256 consecutive ids) and a scan over that wave's
// lanes find the draw.  Before, four waves walked a quarter of the row each,
// 64 ids at a time: 219 us.
template <int NT>
__global__ __launch_bounds__(NT) void soft_rows_kernel(const float* __restrict__ zp_all,
                                                       const float* __restrict__ zq_all, int V, int d,
                                                       const int* __restrict__ look, const float* __restrict__ v,
                                                       float* __restrict__ draft_lp, int* __restrict__ res_ids,
                                                       float* __restrict__ res_lp) {
  constexpr int NW = NT / 64, NSEG = 64;
  __shared__ float sm[2][NW], ss[2][NW], part[NSEG][NW], seg[NSEG], wsum[NW];
  __shared__ int sh_res, sh_arg[NW];
  const int row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float* zp = zp_all + (long long)row * V;
  const float* zq = zq_all + (long long)row * V;
  const int shift = (int)((uintptr_t)zp / 4 & 3);
  const RowSlots rp = row_slots(zp, V, shift), rq = row_slots(zq, V, shift);
  const int nb = (rp.slots + NT - 1) / NT;      // blocks of NT slots
  const int f = (nb + NSEG - 1) / NSEG, ns = (nb + f - 1) / f;
  float mp = -INFINITY, sp = 0.f, mq = -INFINITY, sq = 0.f;
  for (int b0 = 0; b0 < nb; b0 += 4) {
    float x[16], y[16];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float tx[4], ty[4];
      rp.load(tid + NT * (b0 + u), tx);
      rq.load(tid + NT * (b0 + u), ty);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * u + e] = tx[e], y[4 * u + e] = ty[e];
    }
    float cp = -INFINITY, cq = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      cp = fmaxf(cp, x[e]);
      cq = fmaxf(cq, y[e]);
    }
    lse_add(x, cp, mp, sp);
    lse_add(y, cq, mq, sq);
  }
  lse_put<NW>(mp, sp, sm[0], ss[0]);
  lse_put<NW>(mq, sq, sm[1], ss[1]);
  __syncthreads();
  const float lp = lse_take<NW>(sm[0], ss[0]);
  const float lq = lse_take<NW>(sm[1], ss[1]);
  // w of this thread's four ids of block b
  auto weights = [&](const float (&x)[4], const float (&y)[4], float (&t)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      t[e] = fmaxf(0.f, __builtin_amdgcn_exp2f((x[e] - lp) * kLog2e) - __builtin_amdgcn_exp2f((y[e] - lq) * kLog2e));
  };
  auto block_weights = [&](int b, float (&t)[4]) __attribute__((always_inline)) {
    float x[4], y[4];
    rp.load(tid + NT * b, x);
    rq.load(tid + NT * b, y);
    weights(x, y, t);
  };
  if (f == 1) {   // four blocks' loads in flight
    for (int b0 = 0; b0 < nb; b0 += 4) {
      float x[4][4], y[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        rp.load(tid + NT * (b0 + u), x[u]);
        rq.load(tid + NT * (b0 + u), y[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float t[4];
        weights(x[u], y[u], t);
        const float ws = wave_sum((t[0] + t[1]) + (t[2] + t[3]));
        if (lane == 0 && b0 + u < nb) part[b0 + u][wv] = ws;
      }
    }
  } else {
    for (int g = 0; g < ns; ++g) {
      float acc = 0.f;
      for (int b = g * f; b < min(nb, g * f + f); ++b) {
        float t[4];
        block_weights(b, t);
        acc += (t[0] + t[1]) + (t[2] + t[3]);
      }
      acc = wave_sum(acc);
      if (lane == 0) part[g][wv] = acc;
    }
  }
  if (tid == 0) sh_res = -1;
  __syncthreads();
  if (tid < ns) {
    float t = 0.f;
#pragma unroll
    for (int u = 0; u < NW; ++u) t += part[tid][u];
    seg[tid] = t;
  }
  __syncthreads();
  float Z = 0.f;
  for (int g = 0; g < ns; ++g) Z += seg[g];
  const float T = v[row] * Z;
  // the first entry of p[0..n) whose running sum passes T (the last one with
  // mass when rounding leaves T past the total; -1: no mass); before: the sum
  // in front of it
  auto locate = [](const float* p, int n, float T, float& before) {
    float run = 0.f;
    int at = -1;
    before = 0.f;
    for (int u = 0; u < n; ++u) {
      if (p[u] > 0.f) {
        at = u;
        before = run;
        if (run + p[u] > T) break;
      }
      run += p[u];
    }
    return at;
  };
  float before;
  const int sg = Z > 0.f ? locate(seg, ns, T, before) : -1;
  if (sg >= 0) {   // uniform over the workgroup
    float Tl = T - before;
    for (int b = sg * f; b < min(nb, sg * f + f); ++b) {
      float t[4];
      block_weights(b, t);
      const float mine = (t[0] + t[1]) + (t[2] + t[3]);
      const float ws = wave_sum(mine);
      __syncthreads();
      if (lane == 0) wsum[wv] = ws;
      __syncthreads();
      float bs = 0.f, bw;
#pragma unroll
      for (int u = 0; u < NW; ++u) bs += wsum[u];
      const int wl = bs > 0.f ? locate(wsum, NW, Tl, bw) : -1;
      if (wl == wv) {
        const float Tw = Tl - bw;
        // inclusive scan over the lanes, then over a lane's four ids
        float sc = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const float n = __shfl_up(sc, o, 64);
          if (lane >= o) sc += n;
        }
        float run = __shfl_up(sc, 1, 64);
        if (lane == 0) run = 0.f;
        int hit = -1, last = -1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (t[e] > 0.f) {
            last = e;
            if (hit < 0 && run + t[e] > Tw) hit = e;
          }
          run += t[e];
        }
        const unsigned long long hits = __ballot(hit >= 0), mass = __ballot(last >= 0);
        const int from = hits ? __builtin_ctzll(hits) : 63 - __builtin_clzll(mass | 1ull);
        if (lane == from && (hits || mass)) sh_res = 4 * (tid + NT * b) - shift + (hits ? hit : last);
      }
      // done when the draw's running sum was inside this block; a later block
      // of the segment that holds mass takes over when rounding left T past it
      if (bs > Tl) break;
      Tl -= bs;
    }
  }
  __syncthreads();
  int res = sh_res;
  if (res < 0) {   // no mass: the argmax of p, lowest id (uniform)
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int b = 0; b < nb; ++b) {
      float x[4];
      rp.load(tid + NT * b, x);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int id = 4 * (tid + NT * b) - shift + e;
        if (id >= 0 && id < V && vi_better(x[e], id, bv, bi)) {
          bv = x[e];
          bi = id;
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (vi_better(ov, oi, bv, bi)) {
        bv = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      wsum[wv] = bv;
      sh_arg[wv] = bi;
    }
    __syncthreads();
    bv = wsum[0];
    res = sh_arg[0];
    for (int u = 1; u < NW; ++u)
      if (vi_better(wsum[u], sh_arg[u], bv, res)) {
        bv = wsum[u];
        res = sh_arg[u];
      }
  }
  if (tid == 0) {
    const bool ok = res >= 0 && res < V;   // false only for rows without a finite logit
    if (!ok) res = 0;
    const int x = look[(long long)(row / d) * (d + 1) + (row % d) + 1];
    draft_lp[row] = (x >= 0 && x < V) ? zq[x] - lq : __int_as_float(0x7fc00000);
    res_ids[row] = res;
    res_lp[row] = ok ? zp[res] - lp : __int_as_float(0x7fc00000);
  }
}

// Alg. 1 state of each prompt after a k = 1 lookahead: a = n / d (float64,
// as the thresholds are given), r = the accepted window's reward.
// state: 1 = S1 (a >= a_t and r >= r_t), 2 = S2/S3 (a < a_t), 4 = S4.
// first_at[b] = r_t where Step-1 with b = 1 applies (state 2, b1 set), else NaN.
__global__ void controller_states_kernel(int B, int d, const int* __restrict__ n_accept,
                                         const float* __restrict__ reward, double a_t, double r_t, int b1,
                                         int* __restrict__ state, float* __restrict__ first_at) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const double a = (double)n_accept[b] / (double)d;
  const double r = (double)reward[b];
  const int s = a < a_t ? 2 : (r >= r_t ? 1 : 4);
  state[b] = s;
  first_at[b] = (s == 2 && b1) ? (float)r_t : __int_as_float(0x7fc00000);
}

// Keyword reward, one workgroup per (b, i): distinct keywords present in
// generated-so-far + the row's head (when head is set) + its first
// upto[b, i] lookahead tokens (all d when upto is null).
__global__ __launch_bounds__(256) void reward_keywords_kernel(int k, int d, const int* __restrict__ gen,
                                                              int gen_stride, const int* __restrict__ gen_len,
                                                              const int* __restrict__ look,
                                                              const int* __restrict__ upto, int head,
                                                              const int* __restrict__ kws, int n_kw, int normalize,
                                                              float* __restrict__ reward) {
  __shared__ int hit[64];
  __shared__ int uniq[64];
  const int bk = blockIdx.x;
  const int b = bk / k;
  for (int u = threadIdx.x; u < 64; u += 256) hit[u] = 0;
  __syncthreads();
  const int* kw = kws + (long long)b * n_kw;
  const int gl = gen_len[b];
  const int nx = upto ? min(max(upto[bk], 0), d) : d;
  const int skip = head ? 0 : 1;
  const int total = gl + nx + 1 - skip;
  for (int t = threadIdx.x; t < total; t += 256) {
    const int tok = t < gl ? gen[(long long)b * gen_stride + t] : look[(long long)bk * (d + 1) + skip + (t - gl)];
    for (int u = 0; u < n_kw; ++u)
      if (kw[u] == tok) atomicOr(&hit[u], 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int cnt = 0, nd = 0;
    for (int u = 0; u < n_kw; ++u) {
      bool dup = false;
      for (int v = 0; v < u; ++v) dup |= kw[v] == kw[u];
      if (dup) continue;
      ++nd;
      cnt += hit[u];
    }
    reward[bk] = normalize ? (float)cnt / (float)(nd > 0 ? nd : 1) : (float)cnt;
  }
}

__global__ __launch_bounds__(256) void reward_linear_kernel(const float* __restrict__ hidden,
                                                            const float* __restrict__ w, int D,
                                                            float* __restrict__ reward) {
  __shared__ float sh[4];
  const int bk = blockIdx.x;
  const float* h = hidden + (long long)bk * D;
  float s = 0.f;
  for (int c = threadIdx.x; c < D; c += 256) s = fmaf(h[c], w[c], s);
  s = block_sum<4>(s, sh);
  if (threadIdx.x == 0) reward[bk] = s;
}

// The commit kernels only stage their decisions, one record per prompt (see
// the layout in kernels.h); commit_apply_kernel carries a record out after
// the host has checked every prompt's record, so a commit that fails
// validation changes no generated tokens and no next heads.
__device__ __forceinline__ void stage_heads(int* st, int tcap, int kk, int u, int id, float lp) {
  st[kStageHdr + tcap + u] = id;
  st[kStageHdr + tcap + kk + u] = __float_as_int(lp);
}

// Beam commit, one thread per prompt: emit [c_i*, x_i*,1..n] of the selected
// beam.  res_ids / res_lp (soft rejection, [B, k, d]): when n < d the
// residual draw at the rejected position leads the next heads, followed by
// the row's top tokens without it.
__global__ void commit_kernel(int B, int k, int d, int kk, const int* __restrict__ look, const int* __restrict__ beam,
                              const int* __restrict__ n_accept, const int* __restrict__ rtk_ids,
                              const float* __restrict__ rtk_lp, const int* __restrict__ res_ids,
                              const float* __restrict__ res_lp, int* __restrict__ stage, int stage_stride,
                              int tcap) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int* st = stage + (long long)b * stage_stride;
  const int i = beam[b];
  const int n = (i >= 0 && i < k) ? n_accept[b * k + i] : -1;
  if (i < 0 || i >= k || n < 0 || n > d) {
    st[0] = -1;
    return;
  }
  const int bk = b * k + i;
  const int* row = look + (long long)bk * (d + 1);
  st[0] = n + 1;
  st[1] = n == d;
  st[2] = i;
  st[3] = n < d;
  for (int t = 0; t <= n; ++t) st[kStageHdr + t] = row[t];
  if (n < d && res_ids) {
    const long long q = (long long)bk * d + n;
    const long long r = q * kk;
    const int lead = res_ids[q];
    stage_heads(st, tcap, kk, 0, lead, res_lp[q]);
    int o = 1;
    for (int u = 0; u < kk && o < kk; ++u) {
      if (rtk_ids[r + u] == lead) continue;
      stage_heads(st, tcap, kk, o, rtk_ids[r + u], rtk_lp[r + u]);
      ++o;
    }
  } else if (n < d) {
    const long long r = ((long long)bk * d + n) * kk;
    for (int u = 0; u < kk; ++u) stage_heads(st, tcap, kk, u, rtk_ids[r + u], rtk_lp[r + u]);
  }
}

// Alg. 1 commit of a lookahead drafted from the prefix (one sequence per
// prompt, lookahead row [last prefix token, x_1..x_d]): emit x_1..x_n.  The
// next heads are row n's top-kk (the target after x_1..x_n) when n < d;
// when n = d, x_d is fed as a catch-up row.  n = 0 emits nothing.
__global__ void commit_prefix_kernel(int B, int d, int kk, const int* __restrict__ look,
                                     const int* __restrict__ n_accept, const int* __restrict__ rtk_ids,
                                     const float* __restrict__ rtk_lp, int* __restrict__ stage, int stage_stride,
                                     int tcap) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int* st = stage + (long long)b * stage_stride;
  const int n = n_accept[b];
  if (n < 0 || n > d) {
    st[0] = -1;
    return;
  }
  const int* row = look + (long long)b * (d + 1);
  st[0] = n;
  st[1] = n == d;
  st[2] = 0;
  st[3] = n < d;
  for (int t = 0; t < n; ++t) st[kStageHdr + t] = row[1 + t];
  if (n < d) {
    const long long r = ((long long)b * d + n) * kk;
    for (int u = 0; u < kk; ++u) stage_heads(st, tcap, kk, u, rtk_ids[r + u], rtk_lp[r + u]);
  }
}

// Head-only commit, one thread per prompt: prompts with mask[b] != 0 emit
// the head of their selected beam, fed afterwards as a one-row append pass
// that yields the next heads; the others emit nothing (n_emit = 0).
__global__ void commit_heads_kernel(int B, int k, int d, const int* __restrict__ look, const int* __restrict__ beam,
                                    const int* __restrict__ mask, int* __restrict__ stage, int stage_stride) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int* st = stage + (long long)b * stage_stride;
  st[1] = 0;
  st[3] = 0;
  if (!mask[b]) {
    st[0] = 0;
    return;
  }
  const int i = beam[b];
  if (i < 0 || i >= k) {
    st[0] = -1;
    return;
  }
  st[0] = 1;
  st[1] = 1;
  st[2] = i;
  st[kStageHdr] = look[(long long)(b * k + i) * (d + 1)];
}

// Append of given tokens, one thread per prompt: prompts with mask[b] != 0
// emit tokens[b] (checked against [0, V): an id outside it invalidates the
// record), fed afterwards as one appended row; the others emit nothing.
__global__ void commit_tokens_kernel(int B, const int* __restrict__ tokens, const int* __restrict__ mask, int V,
                                     int* __restrict__ stage, int stage_stride) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int* st = stage + (long long)b * stage_stride;
  st[1] = 0;
  st[3] = 0;
  if (!mask[b]) {
    st[0] = 0;
    return;
  }
  const int tok = tokens[b];
  if (tok < 0 || tok >= V) {
    st[0] = -1;
    return;
  }
  st[0] = 1;
  st[1] = 1;
  st[2] = 0;
  st[kStageHdr] = tok;
}

// Withdraw the last cnt[b] tokens of prompt b's prefix (its length and its
// generated tokens).
__global__ void withdraw_kernel(int B, const int* __restrict__ cnt, int* __restrict__ Lp, int* __restrict__ gen_len) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  Lp[b] -= cnt[b];
  gen_len[b] -= cnt[b];
}

// Carries out the checked records: append the emitted tokens to the
// generated tokens, write the staged next heads, and queue the last emitted
// token of catch-up prompts.
__global__ void commit_apply_kernel(int B, const int* __restrict__ stage, int stage_stride, int tcap, int kk,
                                    int* __restrict__ gen, int gen_stride, int* __restrict__ gen_len,
                                    int* __restrict__ next_beams, float* __restrict__ next_head_lp,
                                    int* __restrict__ catch_tok) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int* st = stage + (long long)b * stage_stride;
  const int ne = st[0];
  if (ne > 0) {
    const int gl = gen_len[b];
    for (int t = 0; t < ne; ++t) gen[(long long)b * gen_stride + gl + t] = st[kStageHdr + t];
    gen_len[b] = gl + ne;
    if (st[1]) catch_tok[b] = st[kStageHdr + ne - 1];
  }
  if (ne >= 0 && st[3] && !st[1]) {
    for (int u = 0; u < kk; ++u) {
      next_beams[b * kk + u] = st[kStageHdr + tcap + u];
      next_head_lp[b * kk + u] = __int_as_float(st[kStageHdr + tcap + kk + u]);
    }
  }
}

// Alg. 1 passes from the prefix: the lookahead row starts with the last
// token of the prefix (the prompt's last token until something is
// generated), and those passes see a prefix one token shorter: Lm1 = Lp - 1.
__global__ void prefix_tail_kernel(int B, const int* __restrict__ gen, int gen_stride, const int* __restrict__ gen_len,
                                   const int* __restrict__ ptail, const int* __restrict__ Lp, int* __restrict__ Lm1,
                                   int* __restrict__ look, int look_stride) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  Lm1[b] = Lp[b] - 1;
  if (look) {
    const int gl = gen_len[b];
    look[(long long)b * look_stride] = gl > 0 ? gen[(long long)b * gen_stride + gl - 1] : ptail[b];
  }
}

__global__ void last_tokens_kernel(int B, const int* __restrict__ tokens, int L, int* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) out[b] = tokens[(long long)b * L + L - 1];
}

// Copy cnt suffix slots of the selected beam, from slot soff on, into the
// prefix at positions Lp[b] .. Lp[b] + cnt - 1, for every layer and KV head
// (cnt = min(n_emit, dlim)).
template <typename T>
__global__ __launch_bounds__(256) void promote_kernel(int k, KVPool pool, int n_layers, const int* __restrict__ stage,
                                                      int stage_stride, int dlim, int soff, const int* __restrict__ Lp,
                                                      const int* __restrict__ ptable, int ptable_stride,
                                                      const int* __restrict__ stable, int s_stride_b,
                                                      int s_stride_i) {
  const int b = blockIdx.x;
  const int layer = blockIdx.y;
  const int* st = stage + (long long)b * stage_stride;
  const int ne = st[0];
  if (ne <= 0) return;
  const int cnt = min(ne, dlim);
  const int i = st[2];
  const int L0 = Lp[b];
  const int hd = pool.hd, Hkv = pool.Hkv;
  T* kl = (T*)pool.k + (long long)layer * pool.layer_elems;
  T* vl = (T*)pool.v + (long long)layer * pool.layer_elems;
  const int per_tok = Hkv * hd;
  for (int u = threadIdx.x; u < cnt * per_tok; u += 256) {
    const int t = u / per_tok, rem = u % per_tok;
    const int hh = rem / hd, dd = rem % hd;
    const PromoteIndex ix = promote_index(stable + (long long)b * s_stride_b + i * s_stride_i,
                                          ptable + (long long)b * ptable_stride, L0, t, soff);
    const int sblk = ix.sblk, sslot = ix.sslot, pblk = ix.pblk, pslot = ix.pslot;
    kl[(((long long)pblk * Hkv + hh) * kBlock + pslot) * hd + dd] =
        kl[(((long long)sblk * Hkv + hh) * kBlock + sslot) * hd + dd];
    vl[(((long long)pblk * Hkv + hh) * hd + dd) * kBlock + pslot] =
        vl[(((long long)sblk * Hkv + hh) * hd + dd) * kBlock + sslot];
  }
}

// promote_kernel for the split bf16 pool format
__global__ __launch_bounds__(256) void promote_split_kernel(int k, KVPool pool, int n_layers,
                                                            const int* __restrict__ stage, int stage_stride, int dlim,
                                                            int soff, const int* __restrict__ Lp,
                                                            const int* __restrict__ ptable,
                                                            int ptable_stride, const int* __restrict__ stable,
                                                            int s_stride_b, int s_stride_i) {
  const int b = blockIdx.x;
  const int layer = blockIdx.y;
  const int* st = stage + (long long)b * stage_stride;
  const int ne = st[0];
  if (ne <= 0) return;
  const int cnt = min(ne, dlim);
  const int i = st[2];
  const int L0 = Lp[b];
  const int hd = pool.hd, Hkv = pool.Hkv;
  const long long unit = split_unit_elems(hd);
  const long long plane = (long long)kBlock * hd;
  bf16* kl = (bf16*)pool.k + (long long)layer * 2 * pool.layer_elems;
  bf16* vl = (bf16*)pool.v + (long long)layer * 2 * pool.layer_elems;
  const int per_tok = Hkv * hd;
  for (int u = threadIdx.x; u < cnt * per_tok; u += 256) {
    const int t = u / per_tok, rem = u % per_tok;
    const int hh = rem / hd, dd = rem % hd;
    const PromoteIndex ix = promote_index(stable + (long long)b * s_stride_b + i * s_stride_i,
                                          ptable + (long long)b * ptable_stride, L0, t, soff);
    const int sblk = ix.sblk, sslot = ix.sslot, pblk = ix.pblk, pslot = ix.pslot;
    const bf16* ks = kl + ((long long)sblk * Hkv + hh) * unit + (long long)sslot * hd + dd;
    bf16* kd = kl + ((long long)pblk * Hkv + hh) * unit + (long long)pslot * hd + dd;
    kd[0] = ks[0];
    kd[plane] = ks[plane];
    const bf16* vs = vl + ((long long)sblk * Hkv + hh) * unit + (long long)dd * kBlock + sslot;
    bf16* vd = vl + ((long long)pblk * Hkv + hh) * unit + (long long)dd * kBlock + pslot;
    vd[0] = vs[0];
    vd[plane] = vs[plane];
  }
}

__global__ void advance_kernel(int B, const int* __restrict__ stage, int stage_stride, int dlim,
                               int* __restrict__ Lp) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int ne = stage[(long long)b * stage_stride];
  if (ne > 0) Lp[b] += min(ne, dlim);
}

__global__ void add_kernel(int n, const int* __restrict__ ids, int* __restrict__ v, int delta) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u < n) v[ids ? ids[u] : u] += delta;
}

// Row r of q2 / h2 = row r * R + R - 1 of q / h (the last row of each prompt).
__global__ __launch_bounds__(256) void last_rows_kernel(const float* __restrict__ q, const float* __restrict__ h, int R,
                                                        int Q, int D, float* __restrict__ q2, float* __restrict__ h2) {
  const int r = blockIdx.x;
  const long long src = (long long)r * R + R - 1;
  for (int c = threadIdx.x * 4; c < Q; c += 1024) *(float4*)(q2 + (long long)r * Q + c) = *(const float4*)(q + src * Q + c);
  for (int c = threadIdx.x * 4; c < D; c += 1024) *(float4*)(h2 + (long long)r * D + c) = *(const float4*)(h + src * D + c);
}

__global__ void fill_int_kernel(int* __restrict__ p, int v, long long n) {
  long long u = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (u < n) p[u] = v;
}

__global__ void heads_to_lookaheads(int BK, int d, const int* __restrict__ beams, int* __restrict__ look) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u < BK) look[(long long)u * (d + 1)] = beams[u];
}

}  // namespace

// ---------------------------------------------------------------------------
hipError_t embed_launch(const PassDesc& p, const void* emb, float* h, int D, int V, int dtype, hipStream_t st,
                        int2* rowinfo) {
  const int M = p.M();
  if (M == 0) return hipSuccess;
  if (dtype == 1) embed_rows<bf16><<<M, 256, 0, st>>>(p, (const bf16*)emb, h, D, V, p.bad, rowinfo);
  else embed_rows<float><<<M, 256, 0, st>>>(p, (const float*)emb, h, D, V, p.bad, rowinfo);
  return hipGetLastError();
}

hipError_t rmsnorm_launch(float* x, const float* g, float* out32, bf16* ohi, bf16* olo, int rows, int D,
                          float eps, int last_only, int R, float* hid, hipStream_t st, const float* part, int S) {
  if (rows == 0) return hipSuccess;
  if (S > 0 && last_only) return hipErrorInvalidValue;
  if (D % 4 != 0 || D > 4 * 256 * kNormU) return hipErrorInvalidValue;   // (narrower launches hold fewer columns)
  // Few rows (the rollout): a thread per 16 bytes of the row, so that all of
  // its loads (and those of the split planes) are in flight at once and no
  // wave is launched for nothing.
#define NORM(NT)                                                                                             \
  rmsnorm_rows<NT><<<rows, NT, 0, st>>>(x, g, out32, ohi, olo, D, eps, last_only, R, hid, part, S, rows)
  if (rows >= 256) NORM(256);
  else if (D <= 256) NORM(64);
  else if (D <= 1024) NORM(256);
  else if (D <= 2048) NORM(512);
  else NORM(1024);
#undef NORM
  return hipGetLastError();
}

hipError_t rope_kv_launch(const PassDesc& p, const float* qkv, void* qout, const KVPool& pool, int layer,
                          const float* cos_t, const float* sin_t, int H, int Hkv, int hd, int dtype, hipStream_t st,
                          int S) {
  const int M = p.M();
  if (M == 0) return hipSuccess;
  // q is fp32 for every weight dtype; the KV pool is fp32 or split bf16
  if (dtype == 1) {
    if (hd <= 0 || hd > 256) return hipErrorInvalidValue;
    const int tasks = p.nb * p.kp * Hkv * v_blocks(p.R);   // V: NT / hd of them per workgroup
    // few rows (the rollout): wider row tasks keep more split planes' loads
    // in flight
    if (M < 256)
      rope_kv_write_split<512><<<M + (tasks + 512 / hd - 1) / (512 / hd), 512, 0, st>>>(
          p, qkv, (float*)qout, pool, layer, cos_t, sin_t, H, Hkv, hd, S);
    else
      rope_kv_write_split<256><<<M + (tasks + 256 / hd - 1) / (256 / hd), 256, 0, st>>>(
          p, qkv, (float*)qout, pool, layer, cos_t, sin_t, H, Hkv, hd, S);
  }
  else if (S > 1)
    return hipErrorInvalidValue;
  else
    rope_kv_write<float><<<M, 256, 0, st>>>(p, qkv, (float*)qout, pool, layer, cos_t, sin_t, H, Hkv, hd);
  return hipGetLastError();
}

// The outputs of logit_rows_kernel from the per-tile row statistics the
// LM-head GEMM wrote (RowStats) instead of from the logits: argmax, the
// log-prob of the gathered token, and the top-kk as log-probs.  One
// workgroup per row.  A tile's list is in order, so its first entry is what
// its thread offers, and only the lists that reach the bound are read further.
// (kk rounds over all the lists, as before, read them again for each place: 24
// rows of 2004 tiles, top-8, took 112 us, now 16; 800 rows of 125 tiles,
// top-5, 14 and 8.)
template <int NT, bool ONE>   // ONE: kk <= 1
__global__ __launch_bounds__(NT) void rowstats_merge_kernel(RowStats s, LogitArgs a) {
  constexpr int NW = NT / 64;
  __shared__ TopShared<NW> top;
  __shared__ float shs[NW];
  const int m = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const long long base = (long long)m * s.tiles;
  float bv = -INFINITY, G, cv = -INFINITY;
  int bi = kNoId, ci = kNoId;
  for (int t = tid; t < s.tiles; t += NT) {
    const float v = s.mx[base + t];
    const int id = s.am[base + t];
    if (vi_better(v, id, bv, bi)) bv = v, bi = id;
  }
  if constexpr (ONE) {
    top_one<NW>(bv, bi, top);
    G = bv;
    if (tid == 0 && a.amax) a.amax[rowmap_index(a.amax_map, m)] = vocab_id(bi, a.V);
    if (!a.want_lse) return;
  } else {
    top_offer<NW>(bv, bi, top);
    __syncthreads();
    top_bound<NW>(top, a.kk, cv, ci, G);
  }
  auto reaches = [&](float v, int id) { return id != kNoId && !vi_better(cv, ci, v, id); };
  float sv = 0.f;
  for (int t = tid; t < s.tiles; t += NT) {
    const float mx = s.mx[base + t];
    if (mx != -INFINITY) sv += s.se[base + t] * __expf(mx - G);
    if constexpr (!ONE) {
      if (!reaches(mx, s.am[base + t])) continue;
      for (int u = 0; u < s.kk; ++u) {
        const float v[1] = {s.tv[(base + t) * s.kk + u]};
        const int id = s.tc[(base + t) * s.kk + u];
        if (!reaches(v[0], id)) break;
        top_push<NW>(v, 1u, [&](int) { return id; }, top);
      }
    }
  }
  sv = wave_sum(sv);
  if (lane == 0) shs[w] = sv;
  __syncthreads();
  float se = 0.f;
#pragma unroll
  for (int u = 0; u < NW; ++u) se += shs[u];
  const float lse = G + __logf(se);
  if (a.want_lse && a.lp && tid == 0) {
    const int tok = s.gather_tok ? s.gather_tok[rowmap_index(s.gather_map, m)] : 0;
    const bool in = tok >= 0 && tok < a.V;
    if (!in && a.bad) *a.bad = 1;
    a.lp[m] = in ? s.zx[m] - lse : __int_as_float(0x7fc00000);
  }
  const int dst = a.topk_rows ? a.topk_rows[m] : m;
  auto put = [&](int r, float v, int id) {
    if (r == 0 && a.amax) a.amax[rowmap_index(a.amax_map, m)] = vocab_id(id, a.V);
    if (r >= a.kk || !a.want_lse) return;
    a.topk_ids[(long long)dst * a.kk + r] = vocab_id(id, a.V);
    a.topk_lp[(long long)dst * a.kk + r] = v - lse;
  };
  if constexpr (ONE) {
    if (tid == 0) put(0, bv, bi);
    return;
  }
  const int n = top.n;
  if (n <= kTopList) {
    top_place<NW>(top, n, a.kk, put);
    return;
  }
  // more entries at the bound than the list holds (the best entries all in
  // the tiles of few threads): place by place
  float pv = INFINITY;
  int pi = -1;
  for (int r = 0; r < a.kk; ++r) {
    float v = -INFINITY;
    int id = kNoId;
    for (int t = tid; t < s.tiles; t += NT)
      for (int u = 0; u < s.kk; ++u) {   // the first of the tile's list after the last pick
        const float x = s.tv[(base + t) * s.kk + u];
        const int xi = s.tc[(base + t) * s.kk + u];
        if (!vi_better(pv, pi, x, xi)) continue;
        if (vi_better(x, xi, v, id)) v = x, id = xi;
        break;
      }
    __syncthreads();
    top_one<NW>(v, id, top);
    pv = v;
    pi = id;
    if (tid == 0) put(r, pv, pi);
  }
}

hipError_t rowstats_merge_launch(const RowStats& s, const LogitArgs& a, int M, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (a.kk != s.kk || a.kk < 0 || a.kk > 16 || s.tiles <= 0) return hipErrorInvalidValue;
  if (a.kk <= 1) rowstats_merge_kernel<256, true><<<M, 256, 0, st>>>(s, a);
  else rowstats_merge_kernel<256, false><<<M, 256, 0, st>>>(s, a);
  return hipGetLastError();
}

hipError_t logit_rows_launch(const LogitArgs& a, int M, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (a.kk > 16 || a.kk < 0) return hipErrorInvalidValue;
  // A chunk of four slots per thread, up to a limit: a row's time is its reads
  // and the exchange between its waves, so few rows take all the threads they
  // can fill and many rows share the CUs.  Us with 256 / 512 / 1024 threads:
  // top-5, 384 rows of 50257 55 / 33 / 29, 900 of 32000 43 / 32 / 38, 900 of
  // 128256 184 / 115 / 107; argmax, 20 rows of 16000 6.4 / 5.4 / 6.3, 200 of
  // 50257 22 / 14 / 12, 384 23 / 17 / 19, 900 30 / 32 / 37.  900 rows of 1000,
  // top-5, with 64 / 128 / 256: 9.3 / 10.1 / 11.4.
  const bool one = a.kk <= 1 || !a.want_lse;
  const int slots = a.V % 4 ? a.V / 4 + 2 : a.V / 4;
  const int limit = one ? (M > 512 && a.V <= 65536 ? 256 : M <= 256 && a.V > 32768 ? 1024 : 512)
                        : (M > 512 && a.V <= 65536 ? 512 : 1024);
  int nt = 64;
  while (nt < limit && 4 * nt < slots) nt *= 2;
#define LOGIT_ROWS(NT)                                                                 \
  do {                                                                                 \
    if (!a.want_lse) logit_rows_kernel<NT, false, true><<<M, NT, 0, st>>>(a);          \
    else if (one) logit_rows_kernel<NT, true, true><<<M, NT, 0, st>>>(a);        \
    else logit_rows_kernel<NT, true, false><<<M, NT, 0, st>>>(a);                      \
  } while (0)
  switch (nt) {
    case 64: LOGIT_ROWS(64); break;
    case 128: LOGIT_ROWS(128); break;
    case 256: LOGIT_ROWS(256); break;
    case 512: LOGIT_ROWS(512); break;
    default: LOGIT_ROWS(1024);
  }
#undef LOGIT_ROWS
  return hipGetLastError();
}

hipError_t beam_scores_launch(int BK, int d, const int* look, const int* y, const float* lp, const float* head_lp,
                              const float* lq, const float* u, int* n_accept, float* scores, hipStream_t st) {
  if (BK == 0) return hipSuccess;
  beam_scores_kernel<<<(BK + 127) / 128, 128, 0, st>>>(BK, d, look, y, lp, head_lp, lq, u, n_accept, scores);
  return hipGetLastError();
}

hipError_t select_launch(int B, int k, const float* scores, const float* reward, float alpha, int reward_only,
                         const float* first_at, int* beam, hipStream_t st) {
  if (B == 0) return hipSuccess;
  select_kernel<<<(B + 127) / 128, 128, 0, st>>>(B, k, scores, reward, alpha, reward_only, first_at, beam);
  return hipGetLastError();
}

hipError_t soft_rows_launch(const float* zp, const float* zq, int M, int V, int d, const int* look, const float* v,
                            float* draft_lp, int* res_ids, float* res_lp, hipStream_t st) {
  if (M == 0) return hipSuccess;
  // short rows: more of them per CU (800 rows of 4001: 15 against 35 us)
  if (V <= 8192) soft_rows_kernel<256><<<M, 256, 0, st>>>(zp, zq, V, d, look, v, draft_lp, res_ids, res_lp);
  else soft_rows_kernel<1024><<<M, 1024, 0, st>>>(zp, zq, V, d, look, v, draft_lp, res_ids, res_lp);
  return hipGetLastError();
}

hipError_t controller_states_launch(int B, int d, const int* n_accept, const float* reward, double a_t, double r_t,
                                    int b1, int* state, float* first_at, hipStream_t st) {
  if (B == 0) return hipSuccess;
  controller_states_kernel<<<(B + 127) / 128, 128, 0, st>>>(B, d, n_accept, reward, a_t, r_t, b1, state, first_at);
  return hipGetLastError();
}

hipError_t reward_keywords_launch(int B, int k, int d, const int* gen, int gen_stride, const int* gen_len,
                                  const int* look, const int* upto, int head, const int* kws, int n_kw, int normalize,
                                  float* reward, hipStream_t st) {
  if (B * k == 0) return hipSuccess;
  reward_keywords_kernel<<<B * k, 256, 0, st>>>(k, d, gen, gen_stride, gen_len, look, upto, head, kws, n_kw,
                                                normalize, reward);
  return hipGetLastError();
}

hipError_t reward_linear_launch(int BK, const float* hidden, const float* w, int D, float* reward, hipStream_t st) {
  if (BK == 0) return hipSuccess;
  reward_linear_kernel<<<BK, 256, 0, st>>>(hidden, w, D, reward);
  return hipGetLastError();
}

hipError_t commit_heads_launch(int B, int k, int d, const int* look, const int* beam, const int* mask, int* stage,
                               int stage_stride, hipStream_t st) {
  commit_heads_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, k, d, look, beam, mask, stage, stage_stride);
  return hipGetLastError();
}

hipError_t commit_tokens_launch(int B, const int* tokens, const int* mask, int V, int* stage, int stage_stride,
                                hipStream_t st) {
  commit_tokens_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, tokens, mask, V, stage, stage_stride);
  return hipGetLastError();
}

hipError_t withdraw_launch(int B, const int* cnt, int* Lp, int* gen_len, hipStream_t st) {
  withdraw_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, cnt, Lp, gen_len);
  return hipGetLastError();
}

hipError_t commit_launch(int B, int k, int d, int kk, const int* look, const int* beam, const int* n_accept,
                         const int* rtk_ids, const float* rtk_lp, const int* res_ids, const float* res_lp, int* stage,
                         int stage_stride, int tcap, hipStream_t st) {
  commit_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, k, d, kk, look, beam, n_accept, rtk_ids, rtk_lp, res_ids, res_lp,
                                              stage, stage_stride, tcap);
  return hipGetLastError();
}

hipError_t commit_prefix_launch(int B, int d, int kk, const int* look, const int* n_accept, const int* rtk_ids,
                                const float* rtk_lp, int* stage, int stage_stride, int tcap, hipStream_t st) {
  commit_prefix_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, d, kk, look, n_accept, rtk_ids, rtk_lp, stage, stage_stride,
                                                     tcap);
  return hipGetLastError();
}

hipError_t commit_apply_launch(int B, const int* stage, int stage_stride, int tcap, int kk, int* gen, int gen_stride,
                               int* gen_len, int* next_beams, float* next_head_lp, int* catch_tok, hipStream_t st) {
  commit_apply_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, stage, stage_stride, tcap, kk, gen, gen_stride, gen_len,
                                                    next_beams, next_head_lp, catch_tok);
  return hipGetLastError();
}

hipError_t prefix_tail_launch(int B, const int* gen, int gen_stride, const int* gen_len, const int* ptail,
                              const int* Lp, int* Lm1, int* look, int look_stride, hipStream_t st) {
  prefix_tail_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, gen, gen_stride, gen_len, ptail, Lp, Lm1, look, look_stride);
  return hipGetLastError();
}

hipError_t last_tokens_launch(int B, const int* tokens, int L, int* out, hipStream_t st) {
  last_tokens_kernel<<<(B + 63) / 64, 64, 0, st>>>(B, tokens, L, out);
  return hipGetLastError();
}

hipError_t promote_launch(int B, int k, const KVPool& pool, int n_layers, const int* stage, int stage_stride, int dlim,
                          int soff, const int* Lp, const int* ptable, int ptable_stride, const int* stable,
                          int s_stride_b, int s_stride_i, int dtype, hipStream_t st) {
  dim3 grid(B, n_layers);
  if (dtype == 1)
    promote_split_kernel<<<grid, 256, 0, st>>>(k, pool, n_layers, stage, stage_stride, dlim, soff, Lp, ptable,
                                                ptable_stride, stable, s_stride_b, s_stride_i);
  else
    promote_kernel<float><<<grid, 256, 0, st>>>(k, pool, n_layers, stage, stage_stride, dlim, soff, Lp, ptable,
                                                ptable_stride, stable, s_stride_b, s_stride_i);
  return hipGetLastError();
}

hipError_t advance_launch(int B, const int* stage, int stage_stride, int dlim, int* Lp, hipStream_t st) {
  advance_kernel<<<(B + 127) / 128, 128, 0, st>>>(B, stage, stage_stride, dlim, Lp);
  return hipGetLastError();
}

hipError_t add_launch(int n, const int* ids, int* v, int delta, hipStream_t st) {
  if (n == 0) return hipSuccess;
  add_kernel<<<(n + 127) / 128, 128, 0, st>>>(n, ids, v, delta);
  return hipGetLastError();
}

hipError_t last_rows_launch(int rows, int R, const float* q, int Q, const float* h, int D, float* q2, float* h2,
                            hipStream_t st) {
  if (rows == 0) return hipSuccess;
  if (Q % 4 != 0 || D % 4 != 0) return hipErrorInvalidValue;
  last_rows_kernel<<<rows, 256, 0, st>>>(q, h, R, Q, D, q2, h2);
  return hipGetLastError();
}

hipError_t fill_int_launch(int* p, int v, long long n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  fill_int_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, v, n);
  return hipGetLastError();
}

hipError_t heads_to_lookaheads_launch(int BK, int d, const int* beams, int* look, hipStream_t st) {
  if (BK == 0) return hipSuccess;
  heads_to_lookaheads<<<(BK + 127) / 128, 128, 0, st>>>(BK, d, beams, look);
  return hipGetLastError();
}

}  // namespace cdsl
