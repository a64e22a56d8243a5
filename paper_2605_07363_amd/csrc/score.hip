// Stage 3: token scoring with the routed heads (Eq. misa_score; with all heads
// Eq. dsa_score).  Also used for the candidate re-scoring of Eq. misa_final_topk.
//
// score_stream_kernel (bf16 queries, bf16 or fp8 keys, whole-cache scoring):
//   the decode hot loop.  Every key byte is read exactly once, straight from
//   HBM into registers: a wavefront takes 64 consecutive keys per step as four
//   16-key tiles, each lane loading one contiguous quarter row.  The h dot
//   products per key are evaluated by the matrix core as a 16-row (heads,
//   zero-padded) x 16-column (keys) x 128 product (v_mfma_f32_16x16x32_bf16),
//   which keeps the vector ALU nearly idle so that the kernel stays bound by
//   HBM; fp8 codes are widened to bf16 exactly and the per-token scale is
//   applied after the head sum (ReLU(c x) = c ReLU(x) for c >= 0).  The sum
//   over heads is in-lane for the four rows a lane holds and then a two-step
//   exchange across the four 16-lane groups that leaves lane i with the score
//   of key i of the 64-key group, so stores are fully coalesced.
//
// score_generic_kernel: plain fp32 FMA path for every other combination
//   (fp32 inputs, candidate lists).  A quad of lanes per key or candidate; the
//   gathered query heads sit in LDS and are read by broadcast.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "small_topk.h"

namespace misa {

// ------------------------------------------------------------------ generic
// The four lanes of a quad read 64 contiguous bytes of their key's row per load, all loads at once, and add their sums.
// Bound by latency for few keys (one query of 8 heads, 4096 fp32 keys: 6.6 us with a lane per key, whose 32 loads follow
// one another on 16 CUs; 3.8 us now) and by the multiply-adds and the LDS reads of the query for many.
template <int KDT, int QDT>
__global__ __launch_bounds__(256) void score_generic_kernel(
    Prob p, const void* __restrict__ Q, const float* __restrict__ W, const int* __restrict__ heads,
    const void* __restrict__ K, const float* __restrict__ kscale, const int* __restrict__ cand,
    int k_cand, int groups, float* __restrict__ out) {
  // query heads, padded to a multiple of 8, then their gates: no more LDS than they need, so that eight heads leave
  // room for the eight workgroups that a CU takes
  extern __shared__ __align__(16) float generic_lds[];
  using KV = Vec16<KDT>;
  using QV = Vec16<QDT>;
  const int t = blockIdx.y, seq = blockIdx.z, tid = threadIdx.x;
  const int n = visible(p, seq, t);
  const int hc = heads ? p.h : p.H;
  const int hpad = (hc + 7) & ~7;
  float (*const qs)[kD] = reinterpret_cast<float (*)[kD]>(generic_lds);
  float* const wsm = generic_lds + hpad * kD;
  const size_t qrow = (size_t)seq * p.n_q + t;

  // Gather the active heads (zero rows for padding and for invalid indices).
  for (int i = tid; i < hpad * (kD / QV::N); i += 256) {
    const int j = i / (kD / QV::N), c = i % (kD / QV::N);
    int head = -1;
    if (j < hc) head = heads ? heads[qrow * p.h + j] : j;
    float v[QV::N];
    if (head >= 0 && head < p.H) {
      QV::load(static_cast<const char*>(Q) + ((qrow * p.H + head) * kD + c * QV::N) * (QV::ROW_BYTES / kD), v);
    } else {
#pragma unroll
      for (int e = 0; e < QV::N; ++e) v[e] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < QV::N; ++e) qs[j][c * QV::N + e] = v[e];
  }
  for (int j = tid; j < hpad; j += 256) {
    int head = -1;
    if (j < hc) head = heads ? heads[qrow * p.h + j] : j;
    wsm[j] = (head >= 0 && head < p.H) ? W[qrow * p.H + head] : 0.f;
  }
  __syncthreads();

  const int row_len = cand ? k_cand : p.L;
  const int part = tid & 3;
  for (int group = 0; group < groups; ++group) {    // of 64 keys
    const int slot = (blockIdx.x * groups + group) * 64 + (tid >> 2);
    if (slot >= row_len) return;
    const int s = cand ? cand[qrow * k_cand + slot] : slot;
    float result = -INFINITY;
    if (s >= 0 && s < n) {
      constexpr int PL = kD / KV::N / 4;             // 16-byte pieces per lane: part, part + 4, ...
      const size_t kslot = key_slot(p, seq, s);
      const char* krow = static_cast<const char*>(K) + kslot * KV::ROW_BYTES + part * 16;
      float kv[PL][KV::N];
#pragma unroll
      for (int i = 0; i < PL; ++i) KV::load(krow + i * 64, kv[i]);
      const float scale = KDT == MISA_FP8_E4M3 ? kscale[kslot] : 1.f;
      float total = 0.f;
      for (int hg = 0; hg < hpad; hg += 8) {
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc[j] = 0.f;
#pragma unroll
          for (int i = 0; i < PL; ++i) {
#pragma unroll
            for (int e = 0; e < KV::N; ++e) acc[j] = fmaf(qs[hg + j][(4 * i + part) * KV::N + e], kv[i][e], acc[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[j]), 0xB1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
          acc[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[j]), 0x4E, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
          total = fmaf(wsm[hg + j], relu(acc[j]), total);
        }
      }
      result = KDT == MISA_FP8_E4M3 ? total * scale : total;
    }
    if (part == 0) out[qrow * row_len + slot] = result;
  }
}

// ------------------------------------------------------------------ streaming
// Widen 4 packed fp8 codes to 4 bf16 (exact: 3 mantissa bits fit in 7; scale 1).
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
__device__ __forceinline__ void fp8x4_to_bf16x4(uint32_t w, uint32_t& lo, uint32_t& hi) {
  union { bf16x2 v; uint32_t u; } a, b;
  a.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);  // codes 0,1
  b.v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);   // codes 2,3
  lo = a.u;
  hi = b.u;
}

union Frag {
  bf16x8 v;
  uint4 u;
  u32x4 x;
  uint32_t w[4];
};

typedef __attribute__((__vector_size__(8 * sizeof(int)))) int i32x8;
union Frag8 {   // 32 fp8 codes: one operand of the fp8 matrix instruction
  i32x8 v;
  uint4 u[2];
  u32x4 x[2];
};

__device__ __forceinline__ uint4 buffer_load16(BufferRsrc r, uint32_t lane_off, uint32_t wave_off = 0) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)wave_off, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
__device__ __forceinline__ void buffer_store8(BufferRsrc r, uint32_t lane_off, uint32_t x, uint32_t y) {
  const u32x2 v = {x, y};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)lane_off, 0, 0);
}
// Per lane: a where the lane's bit of the wave mask is set, else b (one v_cndmask on the mask).
template <typename T>
__device__ __forceinline__ T select_by_mask(unsigned long long mask, T a, T b) {
  static_assert(sizeof(T) == 4, "32-bit values");
  uint32_t r;
  asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"((uint32_t)b), "v"((uint32_t)a), "s"(mask));
  return (T)r;
}
__device__ __forceinline__ void buffer_store4(BufferRsrc r, uint32_t lane_off, uint32_t wave_off, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, (int)lane_off, (int)wave_off, 0);
}

// In the lower 32 lanes the value of lane + 32.
__device__ __forceinline__ float upper_half(float x) {
  return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false)[1]);
}

// NT = 16-row head tiles; a wavefront takes STEPS pipeline steps of G 64-key groups each.
// MQ = 0: one query per workgroup, heads <= 16 NT.  MQ = 1 or 2 (a few queries per sequence, e.g. draft
// tokens verified together): MQ queries of at most 16 / MQ heads share a head tile, NT MQ queries share
// the workgroup and its one read of the keys (16 sequences x 32768 bf16 keys, 4 queries of 8 heads:
// 25.2 us = 5.3 TB/s; 64 us when every query reads the cache).  The sums of a query are added in the same order for every MQ.
template <int KDT, int NT, int STEPS, int G, bool PAGED, int MQ>
__global__ __launch_bounds__(256) void score_stream_kernel(
    Prob p, const uint16_t* __restrict__ Q, const float* __restrict__ W,
    const int* __restrict__ heads, const void* __restrict__ K, const float* __restrict__ kscale,
    float* __restrict__ S) {
  constexpr int ROW_BYTES = KDT == MISA_BF16 ? 256 : 128;
  constexpr int NLD = KDT == MISA_BF16 ? 4 : 2;  // 16-byte loads per lane and 16-key tile
  constexpr int KPW = 256 * STEPS * G;           // keys per workgroup
  constexpr int NQ = MQ ? NT * MQ : 1;           // queries per workgroup
  // Last sequence and last keys first: a pass that has just pooled the cache read those last, and the
  // memory-side cache (256 MB) still holds part of them (32 x 131072 fp8 keys, whole pass: 215.5 us against
  // 221.0 us; a cache that was not read right before costs the same in either order).
  const int t = blockIdx.y * NQ, seq = gridDim.z - 1 - blockIdx.z;   // (first) query
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int nq = MQ ? min(NQ, p.n_q - t) : 1;
  int n = visible(p, seq, t);                    // keys the workgroup's queries see: the most of any
  if (MQ)
    for (int q = 1; q < nq; ++q) n = max(n, visible(p, seq, t + q));
  const int hc = heads ? p.h : p.H;
  const size_t qrow = (size_t)seq * p.n_q + t;

  const char* kbase = static_cast<const char*>(K) + (size_t)seq * p.L * ROW_BYTES;
  const float* sbase = kscale + (size_t)seq * p.L;
  float* srow = S + qrow * p.L;
  const int k_begin = (gridDim.x - 1 - blockIdx.x) * KPW;
  const int k_end = min(k_begin + KPW, p.L);

  Frag a[NT][4];   // query operand and gates, filled after the first key loads are issued
  float wv[NT][4];

  // A workgroup whose whole key range is invisible only writes -inf.
  if (k_begin >= n) {
    for (int q = 0; q < nq; ++q)
      for (int key = k_begin + threadIdx.x; key < k_end; key += 256) srow[(size_t)q * p.L + key] = -INFINITY;
    return;
  }
  // MQ: keys the queries of this lane's accumulator rows see, per head tile
  int nv[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const int q = MQ == 2 ? 2 * T + (g >> 1) : T;
    nv[T] = MQ && q < nq ? visible(p, seq, t + q) : 0;
  }

  // Raw 16-byte key chunks of one 64-key group: 4 tiles x NLD loads per lane.
  // Loads are unconditional and branch-free (rows clamped into the cache), so
  // that the number of loads in flight is known at every wait.
  struct Raw { uint4 v[4][NLD]; float scale; };
  // Page pool: a 64-key group starts at a multiple of 64, so with pages of 64 tokens or more
  // all its keys (and the last key, when rows are clamped to it) lie in one page, found with
  // one wavefront-uniform table read; smaller pages are looked up per lane.
  auto issue_loads = [&](Raw& r, int kg) {
    size_t group_slot = 0;
    const bool one_page = PAGED && p.page_shift >= 6;
    if (one_page)
      group_slot = (size_t)p.page_table[(size_t)seq * p.max_pages + (min(kg, p.L - 1) >> p.page_shift)] << p.page_shift;
    const int in_page = (1 << p.page_shift) - 1;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const int row = min(kg + tt * 16 + c, p.L - 1);
      const uint4* src;
      if (!PAGED) src = reinterpret_cast<const uint4*>(kbase + (size_t)row * ROW_BYTES) + g;
      else {
        const size_t slot = one_page ? group_slot + (row & in_page) : key_slot<true>(p, seq, row);
        src = reinterpret_cast<const uint4*>(static_cast<const char*>(K) + slot * ROW_BYTES) + g;
      }
#pragma unroll
      for (int i = 0; i < NLD; ++i) r.v[tt][i] = src[4 * i];
    }
    r.scale = 1.f;
    if (KDT == MISA_FP8_E4M3) {
      const int row = min(kg + lane, p.L - 1);
      if (!PAGED) r.scale = sbase[row];
      else r.scale = kscale[one_page ? group_slot + (row & in_page) : key_slot<true>(p, seq, row)];
    }
  };

  auto finish_group = [&](const Raw& r, int kg) {
    const int key = kg + lane;  // the key this lane finally owns
    if (kg >= k_end) return;
    if (kg >= n) {              // whole group invisible
      if (key < p.L)
        for (int q = 0; q < nq; ++q) srow[(size_t)q * p.L + key] = -INFINITY;
      return;
    }
    float part[4];
    float parts[MQ ? NT : 1][4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      Frag b[4];
      if (KDT == MISA_BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i].u = r.v[tt][i % NLD];
      } else {
        const uint4 lo = r.v[tt][0], hi = r.v[tt][NLD - 1];
        const uint32_t w8[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          fp8x4_to_bf16x4(w8[2 * i], b[i].w[0], b[i].w[1]);
          fp8x4_to_bf16x4(w8[2 * i + 1], b[i].w[2], b[i].w[3]);
        }
      }
      float s = 0.f;
#pragma unroll
      for (int T = 0; T < NT; ++T) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[T][i].v, b[i].v, acc, 0, 0, 0);
        if (MQ) s = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) s = fmaf(wv[T][j], relu(acc[j]), s);
        if (MQ) parts[T][tt] = s;
      }
      part[tt] = s;
    }
    const bool up2 = (g & 2) != 0, up1 = (g & 1) != 0;
    if constexpr (MQ != 0) {
      const float scale0 = KDT == MISA_FP8_E4M3 ? 0.f : 1.f;
#pragma unroll
      for (int T = 0; T < NT; ++T) {
        if constexpr (MQ == 2) {
          // a query's rows are in two lane groups: after one exchange group g holds query 2 T + g / 2,
          // tiles 2 (g & 1) and the next one
          const float r0 = __shfl_xor(up1 ? parts[T][0] : parts[T][2], 16);
          const float r1 = __shfl_xor(up1 ? parts[T][1] : parts[T][3], 16);
          const float k0 = (up1 ? parts[T][2] : parts[T][0]) + r0;
          const float k1 = (up1 ? parts[T][3] : parts[T][1]) + r1;
          const int q = 2 * T + (g >> 1), first = kg + 32 * (g & 1) + c;
          float s0 = scale0, s1 = scale0;
          if (KDT == MISA_FP8_E4M3) {      // the scale of key kg + i is in lane i
            s0 = __shfl(r.scale, 32 * (g & 1) + c);
            s1 = __shfl(r.scale, 32 * (g & 1) + 16 + c);
          }
          if (q < nq) {
            float* row = srow + (size_t)q * p.L;
            if (first < p.L) row[first] = first < nv[T] ? k0 * s0 : -INFINITY;
            if (first + 16 < p.L) row[first + 16] = first + 16 < nv[T] ? k1 * s1 : -INFINITY;
          }
        } else {
          const float r0 = __shfl_xor(up2 ? parts[T][0] : parts[T][2], 32);
          const float r1 = __shfl_xor(up2 ? parts[T][1] : parts[T][3], 32);
          const float k0 = (up2 ? parts[T][2] : parts[T][0]) + r0;
          const float k1 = (up2 ? parts[T][3] : parts[T][1]) + r1;
          const float r2 = __shfl_xor(up1 ? k0 : k1, 16);
          const float fin = (up1 ? k1 : k0) + r2;
          if (T < nq && key < p.L) srow[(size_t)T * p.L + key] = key < nv[T] ? fin * r.scale : -INFINITY;
        }
      }
      return;
    }
    // Sum over the four lane groups so that group g ends with tile g.
    const float r0 = __shfl_xor(up2 ? part[0] : part[2], 32);
    const float r1 = __shfl_xor(up2 ? part[1] : part[3], 32);
    const float k0 = (up2 ? part[2] : part[0]) + r0;
    const float k1 = (up2 ? part[3] : part[1]) + r1;
    const float r2 = __shfl_xor(up1 ? k0 : k1, 16);
    const float fin = (up1 ? k1 : k0) + r2;
    if (key < p.L) srow[key] = key < n ? fin * r.scale : -INFINITY;
  };

  // Software pipeline with two register buffers, fully unrolled: the loads of
  // the next group are all in flight before the current one is consumed.  The
  // first key loads are issued before the query operand is gathered, so the
  // dependent head-index -> gate / query loads overlap with them.
  Raw buf[2][G];
  const int kg0 = k_begin + wave * (64 * G);
#pragma unroll
  for (int q = 0; q < G; ++q) issue_loads(buf[0][q], kg0 + 64 * q);
  __builtin_amdgcn_sched_barrier(0);

  __shared__ int s_head[kMaxH];     // row of the workgroup's queries' [query, head] rows, -1: none
  __shared__ float s_gate[kMaxH];
  if (threadIdx.x < kMaxH) {
    const int r = threadIdx.x;
    const int q = MQ == 2 ? r >> 3 : MQ == 1 ? r >> 4 : 0;
    const int slot = MQ == 2 ? r & 7 : MQ == 1 ? r & 15 : r;
    int head = -1;
    if (slot < hc && q < nq) head = heads ? heads[(qrow + q) * p.h + slot] : slot;
    const bool ok = head >= 0 && head < p.H;
    s_head[r] = ok ? q * p.H + head : -1;
    s_gate[r] = ok ? W[(qrow + q) * p.H + head] : 0.f;
  }
  __syncthreads();

  // A operand: head rows.  The four lanes (c, g = 0..3) that share key column c
  // read 64 contiguous bytes of a key row per load instruction (16-byte chunk
  // 4 i + g for load i), so for bf16 keys k-step i covers components
  // 8 (4 i + g) .. + 7, and for fp8 keys load i feeds k-steps 2 i and 2 i + 1
  // with components 16 (4 i + g) + 8 j .. + 7.  The query fragments use the same
  // component mapping, so the contraction still runs over all 128.
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const int head = s_head[T * 16 + c];
    const uint16_t* src = Q + (qrow * p.H + max(head, 0)) * kD;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int comp = KDT == MISA_BF16 ? 8 * (4 * i + g) : 16 * (4 * (i >> 1) + g) + 8 * (i & 1);
      const uint4 v = *reinterpret_cast<const uint4*>(src + comp);
      a[T][i].u = head >= 0 ? v : make_uint4(0, 0, 0, 0);
    }
    // The accumulator of lane (c, g) holds head rows 4 g + j (j = 0..3) for key column c.
#pragma unroll
    for (int j = 0; j < 4; ++j) wv[T][j] = s_gate[T * 16 + 4 * g + j];
  }

#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    if (st + 1 < STEPS) {
#pragma unroll
      for (int q = 0; q < G; ++q) issue_loads(buf[(st + 1) & 1][q], kg0 + (st + 1) * 256 * G + 64 * q);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < G; ++q) finish_group(buf[st & 1][q], kg0 + st * 256 * G + 64 * q);
  }
}

// ------------------------------------------------------------------ prefill
// score_tile_kernel (bf16 queries, bf16 or fp8 keys, many queries per sequence):
//   a dense contraction [queries x heads, 128] x [128, keys] on the matrix core
//   (v_mfma_f32_32x32x16_bf16).  A workgroup owns a tile of queries and a range
//   of keys.  Each wavefront keeps the gathered head rows of its own queries
//   in registers for the whole key range (the query operand is stationary),
//   while 64-key tiles stream through LDS, double buffered, widened to bf16
//   once when they are staged, rows padded by one 16-byte slot so that fragment reads are
//   free of bank conflicts.  Head rows are placed so that all active heads of
//   a query fall into accumulator registers of the same lane: a lane of the
//   lower half-wave holds rows {0-3, 8-11, 16-19, 24-27} of a 32-row tile,
//   the upper half the others, so ReLU, gate and the sum over heads need no
//   cross-lane traffic, and 32 consecutive lanes store 32 consecutive keys.
//   blockIdx.x is the key range and a multiple of 8 of them is launched, so
//   workgroups that share a key range run on the same XCD and its L2.
//
// HS = head slots per query (h rounded up to 8, 16, 32 or 64).
// WIDE (fp8 operands, 8 head slots, scores stored): four row tiles as well - the operands are half
// as wide, and that kernel is bound by the vector work per key tile, which a wavefront with 16
// queries shares over twice as many products (0.40 ms against 0.46 ms on the 131072-key prefill
// workload).  The filter mode stays with two (its list work needs the second wavefront per SIMD
// to hide behind: 0.99 ms against 0.67 ms for the fused call with four).
template <int HS, bool WIDE>
struct TileGeom {
  static constexpr int RT = (HS > 32 || (WIDE && HS == 8)) ? 4 : 2;   // 32-row tiles per wavefront
  static constexpr int QW = RT * 32 / HS;       // queries per wavefront
  static constexpr int QWG = 4 * QW;            // queries per workgroup
  // query (within the wavefront) and head slot of accumulator register r of
  // row tile rt in half-wave hf
  __device__ static __forceinline__ int query_of(int rt, int hf, int r) {
    if (HS == 8) return rt * 4 + hf * 2 + (r >> 3);
    if (HS == 16) return rt * 2 + hf;
    return hf;
  }
  __device__ static __forceinline__ int slot_of(int rt, int r) {
    if (HS == 8) return r & 7;
    if (HS == 16) return r;
    return rt * 16 + r;
  }
};

constexpr int kKT = 64;  // keys per LDS tile
constexpr int kKP = 17;  // 16-byte slots per key row in LDS: 16 of data + 1 of padding
constexpr int kKP8 = 9;  // the same for rows kept as fp8 codes: 8 of data + 1 of padding
// Queries per sequence from which the tiled matrix-core kernel is used.
constexpr int kTileMinQueries = 8;

// MODE kTileStore: scores of all keys go to S [rows, L].
// MODE kTileSample: only one key of every group of kSampleStride consecutive
//   keys is scored (at a hashed position inside its group); the result is a
//   score matrix [rows, L / kSampleStride] in which a query sees the first
//   n / kSampleStride entries.
// MODE kTileFilter: nothing is stored densely; (key, score) pairs whose score reaches the row's
//   threshold aux.tau go to the row's candidate list.  The list of a row is cut into one
//   segment per key range (aux.seg: offsets [rows, ranges + 1], sized by the caller from the
//   sampled scores of that range), and the workgroup of a (query tile, key range) is the only
//   writer of its segments: a wavefront keeps the fill of its queries' segments in scalar
//   registers, computes the slots of a column tile's hits from the ballot, and stores them
//   straight to the list through a buffer descriptor - lanes without a hit, or past the end of
//   the segment, store to an offset outside the descriptor's range, which drops the store, so
//   there is no branch, no staging list and no atomic.  At the end the fills are written to
//   aux.seg_count [rows, ranges] (a fill above the segment's length tells the caller that it
//   overflowed).
// The work of one workgroup: query tile q_tile of sequence blockIdx.z, key range blockIdx.x.
template <int KDT, int HS, int MODE, bool PAGED, bool Q8>
__device__ __forceinline__ void score_tile_body(
    const Prob& p, int keys_per_wg, const uint16_t* __restrict__ Q, const float* __restrict__ W,
    const int* __restrict__ heads, const void* __restrict__ K, const float* __restrict__ kscale,
    float* __restrict__ S, const TileAux& aux, int q_tile) {
  using G = TileGeom<HS, Q8 && MODE == kTileStore>;
  constexpr int RT = G::RT, QW = G::QW, QWG = G::QWG;
  constexpr bool FILTER = MODE == kTileFilter, SAMPLE = MODE == kTileSample;
  constexpr int NQL_ = HS == 8 ? RT * 2 : (HS == 16 ? RT : 1);  // queries per lane
  constexpr int ROW_BYTES = KDT == MISA_BF16 ? 256 : 128;
  constexpr int NLD = KDT == MISA_BF16 ? 4 : 2;  // 16-byte global loads per thread and tile
  // Q8: queries and keys are both e4m3 codes and stay so: the tile holds raw key rows (8 slots +
  // 1 of padding) and the products run on the fp8 matrix instruction (K = 64 per instruction).
  static_assert(!Q8 || KDT == MISA_FP8_E4M3, "fp8 queries contract with fp8 keys only");
  constexpr int KP = Q8 ? kKP8 : kKP;     // 16-byte slots per key row in LDS
  constexpr int KS = Q8 ? 2 : 8;          // matrix instructions per 32 x 32 output tile
  __shared__ uint4 ktile[2][kKT * KP];
  __shared__ float kscl[2][kKT];
  __shared__ int nvis[QWG];
  __shared__ int s_head[QWG][HS];
  __shared__ float s_tau[FILTER ? QWG : 1];  // thresholds of the workgroup's queries (+inf: no such query)

  const int LT = SAMPLE ? p.L / kSampleStride : p.L;  // keys in tile space
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, hf = lane >> 5;
  const int seq = blockIdx.z;
  const int q_base = q_tile * QWG;
  const int k_begin = blockIdx.x * keys_per_wg;
  const int k_end = min(k_begin + keys_per_wg, LT);
  const int hc = heads ? p.h : p.H;

  for (int i = tid; i < QWG; i += 256) {
    const int n = q_base + i < p.n_q ? visible(p, seq, q_base + i) : 0;
    nvis[i] = SAMPLE ? n / kSampleStride : n;
    if (FILTER) s_tau[i] = q_base + i < p.n_q ? aux.tau[(size_t)seq * p.n_q + q_base + i] : INFINITY;
  }
  for (int i = tid; i < QWG * HS; i += 256) {
    const int qi = i / HS, slot = i % HS, q = q_base + qi;
    int head = -1;
    if (q < p.n_q && slot < hc) head = heads ? heads[((size_t)seq * p.n_q + q) * p.h + slot] : slot;
    s_head[qi][slot] = (head >= 0 && head < p.H) ? head : -1;
  }
  __syncthreads();
  int n_max = 0;
  for (int i = 0; i < QWG; ++i) n_max = max(n_max, nvis[i]);
  const int k_stop = min(k_end, n_max);  // keys at or beyond this are invisible to every query here

  // Stationary operand: row m = col of row tile rt belongs to half-wave (m >> 2) & 1 of the
  // accumulator and to its register r = (m >> 3) * 4 + (m & 3).
  Frag a[RT][Q8 ? 1 : 8];
  Frag8 a8[RT][Q8 ? 2 : 1];   // fp8 operands: k-step ks, half-wave hf: components 64 ks + 32 hf .. + 31
  float gate[RT][16];
  {
    const int m = col, mhf = (m >> 2) & 1, mr = (m >> 3) * 4 + (m & 3);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int qi = wave * QW + G::query_of(rt, mhf, mr), slot = G::slot_of(rt, mr);
      const int head = s_head[qi][slot];
      const size_t qhead = (((size_t)seq * p.n_q + min(q_base + qi, p.n_q - 1)) * p.H + max(head, 0)) * kD;
      if (Q8) {
        const uint8_t* src = reinterpret_cast<const uint8_t*>(Q) + qhead + hf * 32;
#pragma unroll
        for (int ks = 0; ks < (Q8 ? 2 : 0); ++ks)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const uint4 v = *reinterpret_cast<const uint4*>(src + ks * 64 + u * 16);
            a8[rt][ks].u[u] = head >= 0 ? v : make_uint4(0, 0, 0, 0);
          }
      } else {
        const uint16_t* src = Q + qhead + hf * 8;
#pragma unroll
        for (int ks = 0; ks < (Q8 ? 0 : 8); ++ks) {
          const uint4 v = *reinterpret_cast<const uint4*>(src + ks * 16);
          a[rt][ks].u = head >= 0 ? v : make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qj = wave * QW + G::query_of(rt, hf, r);
        const int hd = s_head[qj][G::slot_of(rt, r)];
        gate[rt][r] = hd >= 0 ? W[((size_t)seq * p.n_q + min(q_base + qj, p.n_q - 1)) * p.H + hd] : 0.f;
      }
    }
  }

  const char* kbase = static_cast<const char*>(K) + (PAGED ? (size_t)0 : (size_t)seq * p.L * ROW_BYTES);
  // Staging registers of the next key tile (global -> registers -> LDS).  Thread
  // tid moves the 16-byte chunks tid + 256 i of the tile.
  constexpr int CPR = ROW_BYTES / 16;  // chunks per key row
  // Which chunk of the tile a thread stages: chunk stid + 256 i.  fp8 rows that are widened on
  // the way (each 16-byte chunk becomes two LDS slots) permute the chunks inside every group of
  // 16 lanes (= two key rows), so that eight consecutive lanes cover four chunks of one row and
  // the same four of the next: their LDS stores then fall into eight different 16-byte bank
  // groups (rows are 17 slots apart), where eight chunks of one row hit only the four even ones
  // (measured: 24 % of this kernel's LDS cycles were bank conflicts, none with bf16 rows).
  const int stid = (KDT == MISA_FP8_E4M3 && !Q8)
                       ? ((tid & ~15) | (((tid >> 2) & 1) << 3) | ((tid & 3) + 4 * ((tid >> 3) & 1)))
                       : tid;
  uint4 st0 = make_uint4(0, 0, 0, 0), st1 = st0, st2 = st0, st3 = st0;
  float st_scale = 1.f;
  // A contiguous, unsampled cache is read through a buffer descriptor of the sequence's keys:
  // a tile is one linear piece (thread tid takes bytes 16 tid + 4096 i of it), so a thread's
  // offsets only advance by the tile size, and rows past the end of the cache read as zeros
  // (the descriptor's range check) instead of being clamped per lane.
  constexpr bool LINEAR = !SAMPLE && !PAGED;
  const BufferRsrc krsrc = make_rsrc(kbase, (uint32_t)p.L * (uint32_t)ROW_BYTES);
  uint32_t koff = (uint32_t)k_begin * ROW_BYTES + (uint32_t)stid * 16u;  // next tile to request
  // Cache row of key j of tile space (clamped into the cache).  Sampling takes key
  // 16 j + (top four bits of a multiplicative hash of j) of every group of 16.
  // With a page table the row is the one in the page pool and kbase the pool itself.
  auto key_row = [&](int j) -> size_t {
    j = min(j, LT - 1);
    if (SAMPLE) j = j * kSampleStride + (int)(((uint32_t)j * 2654435761u) >> 28);
    return PAGED ? key_slot<true>(p, seq, j) : (size_t)j;
  };
  // Requests the tile that starts at key k0; successive calls ask for successive tiles.
#define MISA_TILE_LOAD(k0)                                                                        \
  do {                                                                                            \
    if (LINEAR) {                                                                                 \
      st0 = buffer_load16(krsrc, koff);                                                           \
      st1 = buffer_load16(krsrc, koff + 4096u);                                                   \
      if (NLD == 4) {                                                                             \
        st2 = buffer_load16(krsrc, koff + 8192u);                                                 \
        st3 = buffer_load16(krsrc, koff + 12288u);                                                \
      }                                                                                           \
      koff += kKT * ROW_BYTES;                                                                    \
    } else {                                                                                      \
      st0 = *reinterpret_cast<const uint4*>(kbase + key_row((k0) + stid / CPR) * ROW_BYTES + (stid % CPR) * 16); \
      st1 = *reinterpret_cast<const uint4*>(kbase + key_row((k0) + (stid + 256) / CPR) * ROW_BYTES + (stid % CPR) * 16); \
      if (NLD == 4) {                                                                             \
        st2 = *reinterpret_cast<const uint4*>(kbase + key_row((k0) + (stid + 512) / CPR) * ROW_BYTES + (stid % CPR) * 16); \
        st3 = *reinterpret_cast<const uint4*>(kbase + key_row((k0) + (stid + 768) / CPR) * ROW_BYTES + (stid % CPR) * 16); \
      }                                                                                           \
    }                                                                                             \
    if (KDT == MISA_FP8_E4M3 && tid < kKT) st_scale = kscale[(PAGED ? (size_t)0 : (size_t)seq * p.L) + key_row((k0) + tid)]; \
  } while (0)
  // registers -> LDS (bf16, padded rows): chunk stid + 256 i is chunk stid % CPR of row
  // stid / CPR + (256 / CPR) i, so the four writes differ by a constant
  uint4* const lds_put = &ktile[0][0] + (stid / CPR) * KP + (KDT == MISA_BF16 || Q8 ? stid % CPR : 2 * (stid % CPR));
  auto put_chunk = [&](int b, int i, const uint4& v) {
    uint4* dst = lds_put + b * (kKT * KP) + i * ((256 / CPR) * KP);
    if (KDT == MISA_BF16 || Q8) {
      dst[0] = v;
    } else {
      uint4 lo, hi;
      fp8x4_to_bf16x4(v.x, lo.x, lo.y);
      fp8x4_to_bf16x4(v.y, lo.z, lo.w);
      fp8x4_to_bf16x4(v.z, hi.x, hi.y);
      fp8x4_to_bf16x4(v.w, hi.z, hi.w);
      dst[0] = lo;
      dst[1] = hi;
    }
  };
#define MISA_TILE_STORE(b)                                        \
  do {                                                            \
    put_chunk((b), 0, st0);                                       \
    put_chunk((b), 1, st1);                                       \
    if (NLD == 4) {                                               \
      put_chunk((b), 2, st2);                                     \
      put_chunk((b), 3, st3);                                     \
    }                                                             \
    if (KDT == MISA_FP8_E4M3 && tid < kKT) kscl[(b)][tid] = st_scale; \
  } while (0)

  // queries this lane reports: prefix lengths and 32-bit offsets of their score
  // rows relative to the first row of the tile (uniform base + lane offset stores)
  constexpr int NQL = HS == 8 ? RT * 2 : (HS == 16 ? RT : 1);  // queries per lane
  float* s_tile = S + ((size_t)seq * p.n_q + q_base) * LT;
  // Unmasked tiles store through a descriptor of the workgroup's score rows: the address of a
  // store is a per-lane constant (row, column inside the tile) plus the wave-uniform tile start.
  const BufferRsrc srsrc = make_rsrc(s_tile, (uint32_t)QWG * (uint32_t)LT * 4u);
  int qn[NQL];
  uint32_t qoff[NQL];
  // filter mode: thresholds of this lane's queries and the lengths of the wavefront's
  // staging lists (wavefront-uniform, so they live in scalar registers)
  float tauv[NQL];
  // fill of the list segments of the two queries in accumulator slot j (lower / upper half-wave):
  // wavefront-uniform; this lane's segment: first element (relative to the first list of the
  // query tile) and length
  int cnt[NQL], cnt_up[NQL];
  uint32_t seg_lo[NQL];
  int seg_len[NQL];
  const BufferRsrc crsrc = make_rsrc(FILTER ? static_cast<const void*>(aux.cand + ((size_t)seq * p.n_q + q_base) * aux.cap) : nullptr,
                                     FILTER ? (uint32_t)QWG * (uint32_t)aux.cap * 8u : 0u);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  int n_min = 0x7FFFFFFF;
#pragma unroll
  for (int j = 0; j < NQL; ++j) {
    const int qi = wave * QW + (HS == 8 ? (j >> 1) * 4 + hf * 2 + (j & 1) : (HS == 16 ? j * 2 + hf : hf));
    const bool ok = q_base + qi < p.n_q;
    qn[j] = ok ? nvis[qi] : -1;   // -1: query does not exist, nothing is stored
    qoff[j] = (uint32_t)qi * (uint32_t)LT;
    cnt[j] = 0;
    cnt_up[j] = 0;
    tauv[j] = FILTER ? s_tau[qi] : 0.f;
    seg_lo[j] = 0;
    seg_len[j] = 0;
    if (FILTER && ok) {
      const int* sg = aux.seg + ((size_t)seq * p.n_q + q_base + qi) * (aux.ranges + 1) + blockIdx.x;
      const int lo = sg[0];
      seg_lo[j] = (uint32_t)qi * (uint32_t)aux.cap + (uint32_t)lo;
      seg_len[j] = sg[1] - lo;
    }
  }
  // Stores the hits of accumulator slot j named by the ballot m (score sc, key key of this
  // lane) into the segments of its two queries and advances their fills.  Column tiles come here in key
  // order and lanes are keys: a segment is in ascending key order, which the row selection relies on.
  const unsigned long long upper_half = 0xFFFFFFFF00000000ull;
  auto append_hits = [&](int j, unsigned long long m, int key, float sc) {
    const uint32_t m_lo = (uint32_t)m, m_hi = (uint32_t)(m >> 32);
    const int n_lo = __popc(m_lo);
    // slot = fill of the lane's own segment + hits of its half-wave below it (upper lanes see
    // all n_lo lower hits in the running count, so their fill is entered less n_lo)
    const int base = select_by_mask(upper_half, cnt_up[j] - n_lo, cnt[j] - cnt_up[j]);
    const int slot = __builtin_amdgcn_mbcnt_hi(m_hi, __builtin_amdgcn_mbcnt_lo(m_lo, base));
    const unsigned long long fits = __ballot(slot < seg_len[j]) & m;
    const uint32_t off = select_by_mask(fits, (seg_lo[j] + (uint32_t)slot) << 3, 0xFFFFFFF8u);
    buffer_store8(crsrc, off, (uint32_t)key, __float_as_uint(sc));
    cnt[j] += n_lo + __popc(m_hi);      // (cnt: both halves, cnt_up: the upper one)
    cnt_up[j] += __popc(m_hi);
  };

  for (int i = 0; i < QWG; ++i) n_min = min(n_min, q_base + i < p.n_q ? nvis[i] : -1);
  // tiles that end at or before plain_end are visible to every query of the
  // workgroup, all of which exist: no masks are needed there
  const int plain_end = min(n_min, k_end);

  // LDS fragment position of this lane (16-byte units): row col of column tile 0, chunk
  // 2 ks + hf.  Rows are 17 slots apart, so the 16 lanes that read together hit 16 different
  // bank groups, and the k-step only adds a constant: one address register per step.
  // (fp8 rows: 9 slots apart, chunks 4 ks + 2 hf and the next one)
  const int frag0 = Q8 ? col * KP + 2 * hf : col * KP + hf;
  // The key fragments of one 32-key column tile (tile: (buffer * 64 + column tile * 32) * KP)
  // and one matrix instruction of it: row tile rt, k-step ks, onto acc (first: onto zero).
  struct KeyFrags {
    Frag b[Q8 ? 1 : 8];
    Frag8 b8[Q8 ? 2 : 1];
  };
  auto load_frags = [&](KeyFrags& f, int tile) {
    if (Q8) {
#pragma unroll
      for (int ks = 0; ks < (Q8 ? 2 : 0); ++ks) {
        f.b8[ks].u[0] = (&ktile[0][0])[frag0 + tile + 4 * ks];
        f.b8[ks].u[1] = (&ktile[0][0])[frag0 + tile + 4 * ks + 1];
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < (Q8 ? 0 : 8); ++ks) f.b[ks].u = (&ktile[0][0])[frag0 + tile + 2 * ks];
    }
  };
  auto mma = [&](const KeyFrags& f, int rt, int ks, const f32x16& acc, bool first) -> f32x16 {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (Q8)
      return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8[rt][ks].v, f.b8[ks].v, first ? zero : acc, 0, 0, 0, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[rt][ks].v, f.b[ks].v, first ? zero : acc, 0, 0, 0);
  };
  // One 32-key column tile: KS x RT matrix instructions.
  auto mfma_tile = [&](f32x16 (&acc)[RT], int tile) {
    KeyFrags f;
    load_frags(f, tile);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(f, rt, ks, acc[rt], ks == 0);
  };
  // ReLU, gate, head sum and store of one finished column tile.  PLAIN: every
  // query of the workgroup exists and sees the whole tile, so nothing is masked.
  // the gated ReLU of accumulator register r of row tile rt, added to its query's sum
  auto head_term = [&](float (&out)[NQL], const f32x16 (&acc)[RT], int rt, int r) {
    const int j = HS == 8 ? rt * 2 + (r >> 3) : (HS == 16 ? rt : 0);
    out[j] = fmaf(gate[rt][r], relu(acc[rt][r]), out[j]);
  };
  auto finish = [&](auto plain_tag, float (&out)[NQL], int key, float scale) {
    constexpr bool PLAIN = decltype(plain_tag)::value;
    const int key0 = __builtin_amdgcn_readfirstlane(key - col);   // first key of the column tile
    if (KDT == MISA_FP8_E4M3) {
#pragma unroll
      for (int j = 0; j < NQL; ++j) out[j] *= scale;
    }
    if (FILTER) {
#pragma unroll
      for (int j = 0; j < NQL; ++j) {
        const bool pass = out[j] >= tauv[j] && (PLAIN || (key < k_end && key < qn[j]));
        append_hits(j, __ballot(pass), key, out[j]);
      }
    } else if (PLAIN) {
#pragma unroll
      for (int j = 0; j < NQL; ++j) buffer_store4(srsrc, (qoff[j] + (uint32_t)col) * 4u, (uint32_t)key0 * 4u, out[j]);
    } else {
#pragma unroll
      for (int j = 0; j < NQL; ++j)
        if (key < k_end && qn[j] >= 0) s_tile[qoff[j] + (uint32_t)key] = key < qn[j] ? out[j] : -INFINITY;
    }
  };
  auto epilogue = [&](auto plain_tag, const f32x16 (&acc)[RT], int key, float scale) {
    float out[NQL];
#pragma unroll
    for (int j = 0; j < NQL; ++j) out[j] = 0.f;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) head_term(out, acc, rt, r);
    finish(plain_tag, out, key, scale);
  };
  constexpr int TPM = 16 / KS;   // head-sum terms that follow each matrix instruction
  static_assert(KS * RT >= NQL, "one list append per matrix instruction must cover all lists");
  // The matrix instructions of column tile ct into acc_new, each followed by its share
  // (TPM accumulator registers) of the head sums of the previous column tile acc_old;
  // scheduling barriers pin that order, so a wavefront feeds both pipes at once.
  auto tile_step = [&](auto plain_tag, f32x16 (&acc_new)[RT], int tile,
                       const f32x16 (&acc_old)[RT], int key, float scale) {
    KeyFrags f;
    load_frags(f, tile);
    float out[NQL];
#pragma unroll
    for (int j = 0; j < NQL; ++j) out[j] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        acc_new[rt] = mma(f, rt, ks, acc_new[rt], ks == 0);
        const int e = (ks * RT + rt) * TPM;   // KS RT steps x TPM = the 16 RT accumulator registers
#pragma unroll
        for (int u = 0; u < TPM; ++u) head_term(out, acc_old, (e + u) / 16, (e + u) % 16);
        // an empty volatile statement on the running sum keeps these operations between
        // the two scheduling barriers (plain arithmetic would be free to move past them)
        asm volatile("" : "+v"(out[HS == 8 ? (e / 16) * 2 + ((e % 16) >> 3) : (HS == 16 ? e / 16 : 0)]));
        __builtin_amdgcn_sched_barrier(0);
      }
    finish(plain_tag, out, key, scale);
  };
  // Filter mode uses the same fixed pattern, with the list bookkeeping of a column tile put off
  // by one step: a step ends with the compare and ballot of its own sums only (the masks stay
  // in scalar registers, the sums in NQL vector registers), and the slot arithmetic and the
  // staged writes of those candidates sit between the first matrix instructions of the next
  // step instead of after the last one, where nothing of this wavefront would cover them.
  unsigned long long pend_m[NQL];
  float pend_out[NQL];
  int pend_key = 0;  // the lane's key of the step the pending sums are from
#pragma unroll
  for (int j = 0; j < NQL; ++j) {
    pend_m[j] = 0;
    pend_out[j] = 0.f;
  }
  auto append_pending = [&](int j) { append_hits(j, pend_m[j], pend_key, pend_out[j]); };
  auto drain_pending = [&]() {
#pragma unroll
    for (int j = 0; j < NQL; ++j) {
      append_pending(j);
      pend_m[j] = 0;
    }
  };
  auto filter_step = [&](auto plain_tag, f32x16 (&acc_new)[RT], int tile, const f32x16 (&acc_old)[RT],
                         int key, float scale) {
    constexpr bool PLAIN = decltype(plain_tag)::value;
    KeyFrags f;
    load_frags(f, tile);
    float out[NQL];
#pragma unroll
    for (int j = 0; j < NQL; ++j) out[j] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        acc_new[rt] = mma(f, rt, ks, acc_new[rt], ks == 0);
        const int e = (ks * RT + rt) * TPM;
#pragma unroll
        for (int u = 0; u < TPM; ++u) head_term(out, acc_old, (e + u) / 16, (e + u) % 16);
        if (ks * RT + rt < NQL) append_pending(ks * RT + rt);
        asm volatile("" : "+v"(out[HS == 8 ? (e / 16) * 2 + ((e % 16) >> 3) : (HS == 16 ? e / 16 : 0)]));
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int j = 0; j < NQL; ++j) {
      const float o = KDT == MISA_FP8_E4M3 ? out[j] * scale : out[j];
      const bool pass = o >= tauv[j] && (PLAIN || (key < k_end && key < qn[j]));
      pend_m[j] = __ballot(pass);
      pend_out[j] = o;
    }
    pend_key = key;
  };
  using Yes = std::true_type;
  using No = std::false_type;
  // The column tiles of the key range form one stream; the MFMAs of a tile are
  // issued together with the epilogue of the tile before it (two accumulator
  // sets), so matrix and vector pipes overlap inside a wavefront.  Per 64-key
  // LDS tile: [tile i, columns 32..63 | epilogue of columns 0..31], stage tile
  // i+1 into the other LDS buffer, barrier, [tile i+1, columns 0..31 | epilogue
  // of tile i, columns 32..63].
  // Per iteration j, in one straight line: request tile j + 2, [tile j+1, columns 0..31 |
  // epilogue of tile j, columns 32..63], [tile j+1, columns 32..63 | epilogue of tile j+1,
  // columns 0..31], stage tile j + 2 into the LDS buffer tile j has left, barrier.  Requests
  // and staging are unconditional (tiles past the range read zeros or clamped rows into a
  // buffer nobody reads), so an iteration has no branch between a request and its use and
  // every wait counts exactly the score stores issued in between.
  const int n_tiles = k_begin < k_stop ? (k_stop - k_begin + kKT - 1) / kKT : 0;
  if (n_tiles > 0) {
    MISA_TILE_LOAD(k_begin);
    {   // the second tile is requested before the first is staged (the registers are still free)
      const uint4 f0 = st0, f1 = st1, f2 = st2, f3 = st3;
      const float fs = st_scale;
      MISA_TILE_LOAD(k_begin + kKT);
      put_chunk(0, 0, f0);
      put_chunk(0, 1, f1);
      if (NLD == 4) {
        put_chunk(0, 2, f2);
        put_chunk(0, 3, f3);
      }
      if (KDT == MISA_FP8_E4M3 && tid < kKT) kscl[0][tid] = fs;
    }
    MISA_TILE_STORE(1);
    // Every load of the prologue (query operand, gates) has landed before the loop
    // starts, so the waits inside the loop only concern loads issued inside it.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    f32x16 accA[RT], accB[RT];
    float scaleA = 1.f, scaleB = 1.f;
    mfma_tile(accA, 0);
    if (KDT == MISA_FP8_E4M3) scaleA = kscl[0][col];
    // leading tiles that need no masks, then the rest
    const int n_plain = min(n_tiles, max(0, (plain_end - k_begin) / kKT));
    auto half = [&](auto tag) {   // tile 0, columns 32..63 | epilogue of its columns 0..31
      if (FILTER) filter_step(tag, accB, 32 * KP, accA, k_begin + col, scaleA);
      else tile_step(tag, accB, 32 * KP, accA, k_begin + col, scaleA);
      if (KDT == MISA_FP8_E4M3) scaleB = kscl[0][32 + col];
    };
    if (n_plain > 0) half(Yes{});
    else half(No{});
    auto body = [&](auto tag, int j) {
      const int nb = (j + 1) & 1, k0 = k_begin + j * kKT;
      MISA_TILE_LOAD(k0 + 2 * kKT);
      if (FILTER) filter_step(tag, accA, nb * 64 * KP, accB, k0 + 32 + col, scaleB);
      else tile_step(tag, accA, nb * 64 * KP, accB, k0 + 32 + col, scaleB);
      if (KDT == MISA_FP8_E4M3) scaleA = kscl[nb][col];
      if (FILTER) filter_step(tag, accB, (nb * 64 + 32) * KP, accA, k0 + kKT + col, scaleA);
      else tile_step(tag, accB, (nb * 64 + 32) * KP, accA, k0 + kKT + col, scaleA);
      if (KDT == MISA_FP8_E4M3) scaleB = kscl[nb][32 + col];
      MISA_TILE_STORE(nb ^ 1);
      __syncthreads();
    };
    // iteration j finishes columns of the tiles j and j + 1: unmasked when both are
    for (int j = 0; j < n_plain - 1; ++j) body(Yes{}, j);
    for (int j = max(n_plain - 1, 0); j < n_tiles - 1; ++j) body(No{}, j);
    if (FILTER) drain_pending();   // the last column tile is finished at once, after the pending one
    const int k_last = k_begin + (n_tiles - 1) * kKT + 32 + col;
    if (n_plain == n_tiles) epilogue(Yes{}, accB, k_last, scaleB);
    else epilogue(No{}, accB, k_last, scaleB);
  }
  if (FILTER) {
    // fills of this key range's segments (zero when no key of the range is visible): lanes 0
    // and 32 write those of the lower and the upper half-wave's queries
#pragma unroll
    for (int j = 0; j < NQL; ++j) {
      const int qi = wave * QW + (HS == 8 ? (j >> 1) * 4 + hf * 2 + (j & 1) : (HS == 16 ? j * 2 + hf : hf));
      if (col == 0 && q_base + qi < p.n_q)
        aux.seg_count[((size_t)seq * p.n_q + q_base + qi) * aux.ranges + blockIdx.x] = hf ? cnt_up[j] : cnt[j] - cnt_up[j];
    }
  }
#undef MISA_TILE_LOAD
#undef MISA_TILE_STORE
  if (MODE != kTileStore) return;
  // keys of this range that no query of the tile can see
  const int done = k_begin < k_stop ? k_begin + (k_stop - k_begin + kKT - 1) / kKT * kKT : k_begin;
#pragma unroll
  for (int j = 0; j < NQL; ++j) {
    if (qn[j] < 0) continue;
    for (int key = done + col; key < k_end; key += 32) s_tile[qoff[j] + (uint32_t)key] = -INFINITY;
  }
}

// Two wavefronts per SIMD (at most 256 vector registers) except with four row tiles, which
// need the whole register file.
template <int KDT, int HS, int MODE, bool PAGED, bool Q8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TileGeom<HS, Q8 && MODE == kTileStore>::RT == 4 ? 1 : 2, TileGeom<HS, Q8 && MODE == kTileStore>::RT == 4 ? 1 : 2)))
void score_tile_kernel(
    Prob p, int keys_per_wg, const uint16_t* __restrict__ Q, const float* __restrict__ W,
    const int* __restrict__ heads, const void* __restrict__ K, const float* __restrict__ kscale,
    float* __restrict__ S, TileAux aux) {
  score_tile_body<KDT, HS, MODE, PAGED, Q8>(p, keys_per_wg, Q, W, heads, K, kscale, S, aux, blockIdx.y);
}

// Store mode for the flagged query tiles only (aux.run).  Normally none is
// flagged, so the grid is kept small: blockIdx.y strides over the query tiles.
template <int KDT, int HS, bool PAGED, bool Q8>
__global__ __launch_bounds__(256) void score_tile_repair_kernel(
    Prob p, int keys_per_wg, int q_tiles, const uint16_t* __restrict__ Q,
    const float* __restrict__ W, const int* __restrict__ heads, const void* __restrict__ K,
    const float* __restrict__ kscale, float* __restrict__ S, TileAux aux) {
  for (int qt = blockIdx.y; qt < q_tiles; qt += gridDim.y) {
    if (!aux.run[blockIdx.z * q_tiles + qt]) continue;
    score_tile_body<KDT, HS, kTileStore, PAGED, Q8>(p, keys_per_wg, Q, W, heads, K, kscale, S, aux, qt);
    __syncthreads();
  }
}

// ------------------------------------------------------------------ candidate re-scoring
// score_gather_kernel (bf16 queries, bf16 or fp8 keys, or fp8 codes on both sides; candidate lists): the
// fine stage of MISA-dagger scores k' gathered keys of one query with ALL heads
// (Eq. dsa_score on the candidate set).  The query's H head rows are the
// stationary operand (RT 32-row tiles in registers); a wavefront takes 32 candidates per step, one
// column of the matrix instruction each, and the head sum is in-lane over its accumulator registers plus one
// exchange between half-waves.
// Candidates per workgroup: at most kGatherChunk.  The set-up of a workgroup (head rows, gates,
// candidate indices) costs about a fifth of the kernel with 2048 candidates each, so many-query
// problems take 4096 (0.37 ms against 0.39 ms on the 2048 x 8192 re-rank); few-query problems
// take shorter pieces to put more workgroups on the chip.
// FUSED (the whole re-rank of a query in one workgroup, Eq. misa_final_topk): the workgroup takes
// all k' <= 8192 candidates, the scores replace the candidate indices in LDS as they are
// produced (a slot's index has been consumed by then) and the row's top-k is taken from there by
// small_row_topk - no dense score matrix, no second launch.
//
// Loads: a load instruction costs the texture addresser a clock per quad of lanes and cache line, so the rows are read
// whole, by 8 (fp8) or 16 (bf16) consecutive lanes, and go through LDS that only this wavefront uses (rows padded by
// one 16-byte slot: the 16 lanes that read together hit 16 bank groups) to the lanes whose columns they are.
// (Fragments loaded straight by the lane that needs them touch 64 lines per instruction: 70 % of the kernel's time with
// widened fp8 keys.)  The head sums of a row tile stand beside the matrix instructions of the next one, so that a
// wavefront feeds both pipes, and the rows of two steps are in flight in registers.
// Bound by matrix and vector instructions at the clock that the chip holds; 2048 queries x 8192 candidates with
// their top-k: widened fp8 keys 388 -> 343 us, bf16 keys 495 -> 361 us, fp8 on both sides 313 -> 240 us (rows of one step
// in flight 342, 362, 250 us; row tiles with two sets of accumulators: spills for bf16 keys); with the query rows read
// whole as well 337, 353, 236 us, and 1023 rows of 2048 candidates 66 -> 59, 79 -> 75, 55 -> 49 us.  Two wavefronts per
// SIMD; three with one row tile of fp8 queries (1100 x 8192: 128 -> 108 us), where the others would spill.
constexpr int kGatherChunk = 4096;

template <int KDT, int RT, bool Q8, bool PAGED, bool FUSED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RT == 1 && Q8 ? 3 : 2, RT == 1 && Q8 ? 3 : 2))) void score_gather_kernel(
    Prob p, const uint16_t* __restrict__ Q, const float* __restrict__ W,
    const void* __restrict__ K, const float* __restrict__ kscale, const int* __restrict__ cand,
    int k_cand, int chunk, float* __restrict__ out, int k, int* __restrict__ idx,
    float* __restrict__ val) {
  constexpr int ROW_BYTES = KDT == MISA_BF16 ? 256 : 128;
  constexpr int PPR = ROW_BYTES / 16;            // 16-byte pieces of a row = consecutive lanes that read it
  constexpr int NLD = 32 * PPR / 64;             // 16-byte loads per lane and step
  constexpr int RPL = 64 / PPR;                  // rows per load instruction
  constexpr int PITCH = PPR + 1;                 // LDS slots per row
  constexpr bool WIDEN = KDT == MISA_FP8_E4M3 && !Q8;
  const int t = blockIdx.y, seq = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int col = lane & 31, hf = lane >> 5;
  const int n = visible(p, seq, t);
  const uint32_t n_last = (uint32_t)(max(n, 1) - 1);
  const size_t qrow = (size_t)seq * p.n_q + t;
  const int c_begin = blockIdx.x * chunk;            // chunk: a multiple of 128, at most kGatherChunk
  const int c_end = min(c_begin + chunk, k_cand);
  const int* crow = cand + qrow * k_cand;
  float* orow = out + qrow * k_cand;

  // The candidate indices of this workgroup go through LDS, so that reading them
  // in the loop does not wait on the key loads in flight.
  __shared__ __align__(16) int s_cand[FUSED ? kSmallTopkMax : kGatherChunk];
  __shared__ u32x4 s_rows[4][32 * PITCH];            // (later the scratch of the top-k)
  __shared__ __align__(16) float s_gate[RT * 32];
  // Row m of tile rt is head rt*32 + m; half-wave hf holds components 64 hf .. 64 hf + 63,
  // k-step ks the eight from 64 hf + 8 ks (the key fragments use the same mapping).
  // Q8 (fp8 query codes and fp8 keys, fp8 matrix instruction): k-step ks of 64 components,
  // half-wave hf the 32 from 64 ks + 32 hf.
  // The rows are read whole and go through LDS, like the keys' (each wavefront by itself, fragment by fragment: 4096 clocks
  // of the texture addresser per workgroup, as much as 512 candidates take).
  static_assert(!Q8 || KDT == MISA_FP8_E4M3, "fp8 queries contract with fp8 keys only");
  constexpr int KS = Q8 ? 2 : 8;
  constexpr int QPR = Q8 ? 8 : 16, QPITCH = QPR + 1, QLD = RT * 32 * QPR / 256;   // 16-byte pieces per head row, per thread
  static_assert(RT * 32 * QPITCH * 16 <= (int)sizeof(s_rows), "the query rows pass through the keys' LDS");
  u32x4* const s_q = &s_rows[0][0];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(Q) + qrow * p.H * (QPR * 16));
    u32x4 q[QLD];
#pragma unroll
    for (int i = 0; i < QLD; ++i) q[i] = src[min((int)threadIdx.x + 256 * i, p.H * QPR - 1)];
    const float w = threadIdx.x < RT * 32 ? W[qrow * p.H + min((int)threadIdx.x, p.H - 1)] : 0.f;
    for (int i0 = threadIdx.x; i0 < chunk; i0 += 4096) {   // (16 loads in flight)
      int v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = crow[min(c_begin + i0 + 256 * u, k_cand - 1)];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int i = i0 + 256 * u;
        if (i < chunk) s_cand[i] = c_begin + i < c_end ? v[u] : -1;
      }
    }
#pragma unroll
    for (int i = 0; i < QLD; ++i) {
      const int e = threadIdx.x + 256 * i, head = e / QPR;
      s_q[head * QPITCH + e % QPR] = head < p.H ? q[i] : u32x4{0, 0, 0, 0};
    }
    if (threadIdx.x < RT * 32) s_gate[threadIdx.x] = threadIdx.x < p.H ? w : 0.f;
  }
  Frag a[RT][Q8 ? 1 : 8];
  Frag8 a8[RT][Q8 ? 2 : 1];
  float gate[RT * 16];                               // of the rows this lane holds

  const char* kseq = static_cast<const char*>(K) + (PAGED ? 0 : (size_t)seq * p.L * ROW_BYTES);
  const float* sseq = kscale + (PAGED ? 0 : (size_t)seq * p.L);
  u32x4* const rows = s_rows[wave];
  u32x4* const put_at = rows + (lane / PPR) * PITCH + lane % PPR;
  const u32x4* const get_at = rows + col * PITCH + (Q8 ? 2 * hf : (PPR / 2) * hf);
  // Any candidate value gives the address of a visible key (the last one where it is none); steps past the end
  // read the last slots, of which nothing is kept.
  struct Stage { u32x4 v[NLD]; };
  struct Slots { int s[NLD]; };
  auto slots_at = [&](int c0) __attribute__((always_inline)) { return &s_cand[min(c0 - c_begin, chunk - 32)]; };
  auto read_slots = [&](Slots& sl, int c0) __attribute__((always_inline)) {   // candidates of the rows a lane helps to load
#pragma unroll
    for (int i = 0; i < NLD; ++i) sl.s[i] = slots_at(c0)[lane / PPR + i * RPL];
  };
  auto issue = [&](Stage& st, const Slots& sl) __attribute__((always_inline)) {
    const uint32_t piece_off = (uint32_t)(lane % PPR) * 16u;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const uint32_t row = min((uint32_t)sl.s[i], n_last);
      if (PAGED) st.v[i] = *reinterpret_cast<const u32x4*>(kseq + key_slot<true>(p, seq, (int)row) * ROW_BYTES + piece_off);
      else st.v[i] = *reinterpret_cast<const u32x4*>(kseq + (row * (uint32_t)ROW_BYTES + piece_off));
    }
  };
  auto put = [&](const Stage& st) __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (the fragments before have been read: LDS keeps a wavefront's order)
#pragma unroll
    for (int i = 0; i < NLD; ++i) put_at[i * RPL * PITCH] = st.v[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  // A step's key fragments: pieces of the lane's own column.
  struct Pieces { u32x4 v[Q8 ? 4 : KDT == MISA_BF16 ? 8 : 4]; };
  auto get = [&](Pieces& f, int j) __attribute__((always_inline)) { f.v[j] = get_at[Q8 ? 4 * (j >> 1) + (j & 1) : j]; };
  auto widen = [&](Frag& b, const Pieces& f, int ks) __attribute__((always_inline)) {
    const u32x4 w = f.v[ks >> 1];
    fp8x4_to_bf16x4(w[2 * (ks & 1)], b.w[0], b.w[1]);
    fp8x4_to_bf16x4(w[2 * (ks & 1) + 1], b.w[2], b.w[3]);
  };
  struct Own { int s; float scale; };                // this lane's candidate of a step
  auto own_scale = [&](Own& o) __attribute__((always_inline)) {
    o.scale = 1.f;
    if (KDT == MISA_FP8_E4M3) {
      const int row = (int)min((uint32_t)o.s, n_last);
      o.scale = PAGED ? sseq[key_slot<true>(p, seq, row)] : sseq[(uint32_t)row];
    }
  };
  // (bf16 keys: sums of eight heads, then those: as exact as 16-row head tiles would give)
  constexpr int PER = KDT == MISA_BF16 ? 8 : RT * 16;
  constexpr int NPART = RT * 16 / PER;
  float part[NPART];                                 // running head sums of the step that is being finished
  auto head_term = [&](const f32x16& acc, int i) __attribute__((always_inline)) {
    const float x = relu(acc[i % 16]);
    part[i / PER] = i % PER == 0 ? gate[i] * x : fmaf(gate[i], x, part[i / PER]);
  };
  auto finish = [&](const Own& o, int c0) __attribute__((always_inline)) {
    float sum = part[0];
#pragma unroll
    for (int i = 1; i < NPART; ++i) sum += part[i];
    sum += upper_half(sum);
    const int slot = c0 + col;
    if (hf == 0 && slot < c_end) {
      const float score = (uint32_t)o.s < (uint32_t)n ? sum * o.scale : -INFINITY;
      if (FUSED) s_cand[slot] = __float_as_int(score);   // (c_begin = 0; this slot's index has been read)
      else orow[slot] = score;
    }
  };
  // One pass: the matrix instructions of row tile rt of the step at c0, into acc_new, beside the
  // head sums of the pass before (acc_old, row tile old_rt; HEADS false: there is none), so that one set of
  // accumulators serves both.  The step's first pass puts the rows of the next step from registers into LDS (this step's
  // pieces have all been read), issues the loads of the step after the next two and finishes the step before; its last
  // pass reads the next step's pieces as this step's are used up.  (The order between the matrix instructions is left to
  // the compiler: pinned with scheduling barriers the same code took 3 to 5 % longer.)
  Stage odd, even;                                   // rows of the next two steps
  Slots sl;
  Frag b[WIDEN ? 8 : 1];
  Pieces f;
  Own own;
  auto pass = [&](auto heads_tag, auto rt_tag, f32x16& acc_new, const f32x16& acc_old, Stage& st, int c0) __attribute__((always_inline)) {
    constexpr bool HEADS = decltype(heads_tag)::value;
    constexpr int rt = decltype(rt_tag)::value, old_rt = RT - 1 - rt;
    constexpr bool FIRST = rt == 0, LAST = rt == RT - 1;
    constexpr int TPM = 16 / KS;
    constexpr int PUT = Q8 ? 0 : RT == 1 ? 1 : 2;    // k-step after which the rows go to LDS
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int s_new = 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if constexpr (Q8) {
        Frag8 k8;
        k8.x[0] = f.v[(2 * ks) & 3];
        k8.x[1] = f.v[(2 * ks + 1) & 3];
        acc_new = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8[rt][ks & 1].v, k8.v, ks == 0 ? zero : acc_new, 0, 0, 0, 0, 0, 0);
      } else {
        Frag kb;
        if (WIDEN) kb = b[ks & 7];
        else kb.x = f.v[ks % (sizeof(f.v) / 16)];
        acc_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[rt][ks & 7].v, kb.v, ks == 0 ? zero : acc_new, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < (HEADS ? TPM : 0); ++u) head_term(acc_old, old_rt * 16 + ks * TPM + u);
      if (FIRST && ks == PUT) {
        put(st);
        issue(st, sl);
        s_new = slots_at(c0)[col];
      }
      if (LAST) {
        auto next = [&](int j) __attribute__((always_inline)) {   // piece j (8 of them: bf16 fragments) of the next step
          if (WIDEN) {
            widen(b[j & 7], f, j);
          } else {
            get(f, j % (sizeof(f.v) / 16));
          }
        };
        if (Q8) {
          next(2 * ks);
          next(2 * ks + 1);
        } else if (RT == 2) {
          next(ks);
        } else if (ks >= 3) {                        // (one pass: after the rows have been put)
          if (ks == 4) next(2);
          if (ks == 5) next(4);
          if (ks == 7) next(6);
          next(ks == 3 ? 0 : ks == 4 ? 1 : ks == 5 ? 3 : ks == 6 ? 5 : 7);
        }
      }
      if (WIDEN && FIRST && ks == (RT == 2 ? 5 : 2)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) get(f, j);
      }
      if (LAST && ks == KS - 1) read_slots(sl, c0 + 512);
    }
    if (FIRST) {
      if (HEADS) finish(own, c0 - 128);
      own.s = s_new;
      own_scale(own);
    }
  };
  using Yes = std::true_type;
  using No = std::false_type;
  using Tile0 = std::integral_constant<int, 0>;
  using Tile1 = std::integral_constant<int, RT - 1>;

  const int c_first = c_begin + wave * 32;
  const int steps = (c_end - c_first + 127) / 128;   // of this wavefront (none: <= 0)
  __syncthreads();                                   // candidate indices, query rows and gates are in LDS
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const u32x4* row = s_q + (rt * 32 + col) * QPITCH;
    if (Q8) {
#pragma unroll
      for (int i = 0; i < (Q8 ? 4 : 0); ++i) a8[rt][i >> 1].x[i & 1] = row[4 * (i >> 1) + 2 * hf + (i & 1)];
    } else {
#pragma unroll
      for (int ks = 0; ks < (Q8 ? 0 : 8); ++ks) a[rt][ks].x = row[8 * hf + ks];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 w = *reinterpret_cast<const float4*>(&s_gate[rt * 32 + 8 * g + 4 * hf]);
      gate[rt * 16 + 4 * g] = w.x;
      gate[rt * 16 + 4 * g + 1] = w.y;
      gate[rt * 16 + 4 * g + 2] = w.z;
      gate[rt * 16 + 4 * g + 3] = w.w;
    }
  }
  __syncthreads();                                   // the rows' LDS is free for the keys
  if (steps > 0) {
    f32x16 acc0, acc1;
    {
      Stage first;
      read_slots(sl, c_first);
      issue(first, sl);
      read_slots(sl, c_first + 128);
      issue(odd, sl);
      read_slots(sl, c_first + 256);
      issue(even, sl);
      put(first);
    }
    read_slots(sl, c_first + 384);
#pragma unroll
    for (int j = 0; j < (int)(sizeof(f.v) / 16); ++j) get(f, j);
#pragma unroll
    for (int j = 0; j < (WIDEN ? 8 : 0); ++j) widen(b[j], f, j);
    auto rest = [&](const f32x16& acc, int c) __attribute__((always_inline)) {   // the head sums of the last pass
#pragma unroll
      for (int e = 0; e < 16; ++e) head_term(acc, (RT - 1) * 16 + e);
      finish(own, c);
    };
    pass(No{}, Tile0{}, acc0, acc1, odd, c_first);
    if (RT == 2) pass(Yes{}, Tile1{}, acc1, acc0, odd, c_first);
    int c0 = c_first + 128;
    for (int i = 1;; i += 2, c0 += 256) {
      if (i >= steps) { rest(RT == 2 ? acc1 : acc0, c0 - 128); break; }
      if constexpr (RT == 2) {
        pass(Yes{}, Tile0{}, acc0, acc1, even, c0);
        pass(Yes{}, Tile1{}, acc1, acc0, even, c0);
      } else {
        pass(Yes{}, Tile0{}, acc1, acc0, even, c0);
      }
      if (i + 1 >= steps) { rest(acc1, c0); break; }
      pass(Yes{}, Tile0{}, acc0, acc1, odd, c0 + 128);
      if constexpr (RT == 2) pass(Yes{}, Tile1{}, acc1, acc0, odd, c0 + 128);
    }
  }
  if constexpr (FUSED) {
    static_assert(sizeof(SmallRowLds) <= sizeof(s_rows), "the top-k works in the rows' LDS");
    __syncthreads();                // all scores of the row are in LDS, the rows' LDS is free
    small_row_topk(s_cand, k_cand, k, crow, idx + qrow * k, val ? val + qrow * k : nullptr,
                   *reinterpret_cast<SmallRowLds*>(&s_rows[0][0]));
  }
}

template <int KDT, int QDT>
static hipError_t launch_generic(const Prob& p, const void* Q, const float* W, const int* heads,
                                 const void* K, const float* kscale, const int* cand, int k_cand,
                                 float* out, hipStream_t st) {
  const int row_len = cand ? k_cand : p.L;
  const int hpad = ((heads ? p.h : p.H) + 7) & ~7;
  const int lds = hpad * (kD + 1) * (int)sizeof(float);
  // 64 keys per workgroup where the chip takes all of those at once (eight per CU by registers, five with fp32 keys, four
  // by LDS with 64 heads), else 128 share the set-up, and 256 where there are many turns of them
  // (us, lane per key / this: one query of 8 heads x 4096 fp32 keys 6.6 / 3.8, 2 x 120 x 554 11.6 / 8.9,
  // 500 x 890 bf16 keys 22.3 / 17.0, 96 x 2951 fp8 candidates of 64 heads 181 / 136; 256 keys and room for 64 heads in every
  // workgroup: 14.2 for 2 x 120 x 554, 23.0 for 500 x 890, 175; 128 against 256 keys: 32 x 21 x 12143 fp32 keys 538 / 497)
  const int at_once = 256 * std::min(KDT == MISA_F32 ? 5 : 8, 160 * 1024 / lds);
  const long long most = (long long)((row_len + 63) / 64) * p.n_q * p.n_seq;
  const int groups = most <= at_once ? 1 : most <= 16 * at_once ? 2 : 4;
  const dim3 grid((row_len + 64 * groups - 1) / (64 * groups), p.n_q, p.n_seq);
  score_generic_kernel<KDT, QDT><<<grid, 256, lds, st>>>(p, Q, W, heads, K, kscale, cand, k_cand, groups, out);
  return hipGetLastError();
}

template <int KDT>
static hipError_t launch_stream(const Prob& p, const void* Q, const float* W, const int* heads,
                                const void* K, const float* kscale, float* S, hipStream_t st) {
  const int hc = heads ? p.h : p.H;
  const int nt = (hc + 15) / 16;
  // bf16 keys: 4 pipeline steps of one 64-key group per wavefront, 1024 keys (256 KB) per
  // workgroup.  fp8 keys with up to 16 heads: one step, 256 keys (32 KB) per workgroup -
  // every wavefront loads its 8 KB, computes and retires, and latency is hidden by the
  // other resident wavefronts alone (4 per SIMD).  Measured best of 256 .. 4096 keys per
  // workgroup on MI355X for each type (fp8: 96 us against 102 us with 1024 keys; bf16: 94 us
  // against 97 us with 256 keys); with more head tiles fewer wavefronts fit a SIMD and the
  // pipelined form is faster again (32 heads, fp8: 105 us against 134 us).
  const uint16_t* q = static_cast<const uint16_t*>(Q);
#define GO(NT, STEPS, MQ)                                                                         \
  do {                                                                                            \
    constexpr int KPW = 256 * (STEPS), NQ = (MQ) ? (NT) * (MQ) : 1;                               \
    const dim3 grid((p.L + KPW - 1) / KPW, (p.n_q + NQ - 1) / NQ, p.n_seq);                       \
    if (p.page_table)                                                                             \
      score_stream_kernel<KDT, NT, STEPS, 1, true, MQ><<<grid, 256, 0, st>>>(p, q, W, heads, K, kscale, S);  \
    else                                                                                          \
      score_stream_kernel<KDT, NT, STEPS, 1, false, MQ><<<grid, 256, 0, st>>>(p, q, W, heads, K, kscale, S); \
    return hipGetLastError();                                                                     \
  } while (0)
  // Several queries per read of the keys, where a workgroup per query and 1024 keys would be more than one per CU
  // (us, a query each / together: 7 queries of 8 heads, bf16, 32768 keys 9.9 / 13.2; 2 queries of 131072 10.4 / 10.8,
  // 3 of them 17.4 / 11.8; fp8 9.5 / 10.9, 4 queries of 131072 12.8 / 9.0).  Together a workgroup takes 1024 keys for
  // fp8 as well: the sums of the queries bound it, not the wavefronts in flight.
  const bool together = (long long)p.n_q * p.n_seq * ((p.L + 1023) / 1024) > 256;
  if (p.n_q > 1 && hc <= 16 && together) {
    if (hc <= 8) {
      if (p.n_q == 2) GO(1, 4, 2);
      if (p.n_q <= 4) GO(2, 4, 2);
      if (p.n_q <= 6) GO(3, 4, 2);
      GO(4, 4, 2);
    }
    if (p.n_q == 2) GO(2, 4, 1);
    if (p.n_q == 3) GO(3, 4, 1);
    GO(4, 4, 1);                 // (n_q 5 .. 7: two workgroups per key range)
  }
  switch (nt) {
    case 1:
      if (KDT == MISA_FP8_E4M3) GO(1, 1, 0);
      GO(1, 4, 0);
    case 2: GO(2, 4, 0);
    case 3: GO(3, 4, 0);
    default: GO(4, 4, 0);
  }
#undef GO
}

// q8: the store-mode geometry of fp8 query codes (the wider query tile)
int tile_queries_per_wg(const Prob& p, bool routed, bool q8) {
  const int hc = routed ? p.h : p.H;
  return hc <= 8 ? (q8 ? 64 : 32) : (hc <= 16 ? 16 : 8);
}

int tile_key_ranges(const Prob& p, bool routed, bool q8, int mode, int* keys_per_wg) {
  const int qwg = tile_queries_per_wg(p, routed, q8 && mode == kTileStore);
  const int q_tiles = (p.n_q + qwg - 1) / qwg;
  const int lt = mode == kTileSample ? p.L / kSampleStride : p.L;  // keys in tile space
  // Key ranges: a multiple of 8 (one set per XCD), enough workgroups to fill
  // the chip several times, at least 1024 keys each.
  int splits = 8;
  while (splits < 64 && (long long)splits * q_tiles * p.n_seq < 2048 && lt / (splits * 2) >= 1024) splits *= 2;
  // Where that leaves CUs without a workgroup, ranges of down to four tiles, while all of them run at once (two per
  // CU; us, 1024 keys / this: 333 queries x 10007 keys 26.3 / 16.1, 32 x 10007 20.5 / 9.9, 8 x 4096 13.0 / 9.6,
  // 1000 x 10007 30.2 / 27.8; past two per CU, 400 x 20000 in ranges of 313 keys 31.9, of 625 25.5).  One per CU where a
  // workgroup has 512 head rows to prepare, or two of 256 run no faster (one / two per CU: 160 queries of 64 heads x 4200 keys
  // 20.7 / 26.7, x 8300 33.6 / 39.2; 704 of 8 heads, fp8 codes, x 16500 38.0 / 42.0; 160 of 32 heads x 4200 13.6 / 14.3).
  const int hc = routed ? p.h : p.H;
  const int most = hc > 16 || (hc <= 8 && q8 && mode == kTileStore) ? 256 : 512;
  while (splits < 64 && 2ll * splits * q_tiles * p.n_seq <= most && lt / (splits * 2) >= 256) splits *= 2;
  *keys_per_wg = ((lt + splits - 1) / splits + kKT - 1) / kKT * kKT;
  return (lt + *keys_per_wg - 1) / *keys_per_wg;
}

template <int KDT, int MODE, bool Q8>
static hipError_t launch_tile(const Prob& p, const void* Q, const float* W, const int* heads,
                              const void* K, const float* kscale, float* S, const TileAux& aux,
                              hipStream_t st) {
  const int hc = heads ? p.h : p.H;
  const int hs = hc <= 8 ? 8 : (hc <= 16 ? 16 : (hc <= 32 ? 32 : 64));
  const int qwg = tile_queries_per_wg(p, heads != nullptr, Q8 && MODE == kTileStore);
  const int q_tiles = (p.n_q + qwg - 1) / qwg;
  int keys_per_wg = 0;
  const int ranges = tile_key_ranges(p, heads != nullptr, Q8, MODE, &keys_per_wg);
  dim3 grid(ranges, q_tiles, p.n_seq);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
  if (MODE == kTileStore && aux.run) {
    // about one resident set of workgroups, each striding over the query tiles
    grid.y = (unsigned)std::max(1, std::min(q_tiles, (int)(512 / ((long long)grid.x * p.n_seq))));
#define GO(HS)                                                                                                      \
  if (p.page_table)                                                                                                 \
    score_tile_repair_kernel<KDT, HS, true, Q8><<<grid, 256, 0, st>>>(p, keys_per_wg, q_tiles, q, W, heads, K, kscale, S, aux); \
  else                                                                                                              \
    score_tile_repair_kernel<KDT, HS, false, Q8><<<grid, 256, 0, st>>>(p, keys_per_wg, q_tiles, q, W, heads, K, kscale, S, aux)
    switch (hs) {
      case 8: GO(8); break;
      case 16: GO(16); break;
      case 32: GO(32); break;
      default: GO(64); break;
    }
#undef GO
    return hipGetLastError();
  }
#define GO(HS)                                                                                               \
  if (p.page_table)                                                                                          \
    score_tile_kernel<KDT, HS, MODE, true, Q8><<<grid, 256, 0, st>>>(p, keys_per_wg, q, W, heads, K, kscale, S, aux); \
  else                                                                                                       \
    score_tile_kernel<KDT, HS, MODE, false, Q8><<<grid, 256, 0, st>>>(p, keys_per_wg, q, W, heads, K, kscale, S, aux)
  switch (hs) {
    case 8: GO(8); break;
    case 16: GO(16); break;
    case 32: GO(32); break;
    default: GO(64); break;
  }
#undef GO
  return hipGetLastError();
}

// The matrix-core tile kernel takes bf16 queries with bf16 or fp8 keys, and fp8 query codes with
// fp8 keys (both operands then stay fp8).
bool tile_path(const Prob& p, int k_dtype, int q_dtype) {
  const bool types = (q_dtype == MISA_BF16 && k_dtype != MISA_F32) ||
                     (q_dtype == MISA_FP8_E4M3 && k_dtype == MISA_FP8_E4M3);
  return types && p.n_q >= kTileMinQueries;
}

hipError_t launch_tile_mode(const Prob& p, int k_dtype, int q_dtype, int mode, const TileAux& aux,
                            const void* Q, const float* W, const int* heads, const void* K,
                            const float* kscale, float* S, hipStream_t st) {
#define GO(KD, Q8)                                                                                      \
  switch (mode) {                                                                                       \
    case kTileSample: return launch_tile<KD, kTileSample, Q8>(p, Q, W, heads, K, kscale, S, aux, st);   \
    case kTileFilter: return launch_tile<KD, kTileFilter, Q8>(p, Q, W, heads, K, kscale, S, aux, st);   \
    default: return launch_tile<KD, kTileStore, Q8>(p, Q, W, heads, K, kscale, S, aux, st);             \
  }
  if (q_dtype == MISA_FP8_E4M3) GO(MISA_FP8_E4M3, true)
  if (k_dtype == MISA_BF16) GO(MISA_BF16, false)
  GO(MISA_FP8_E4M3, false)
#undef GO
}

template <int KDT, bool Q8>
static hipError_t launch_gather(const Prob& p, const void* Q, const float* W, const void* K,
                                const float* kscale, const int* cand, int k_cand, float* out,
                                hipStream_t st) {
  // pieces of 512 .. kGatherChunk candidates (a step of the four wavefronts covers 128 or 256): halved
  // while fewer than 1024 workgroups would result
  int chunk = kGatherChunk;
  const long long rows = (long long)p.n_q * p.n_seq;
  while (chunk > 512 && rows * ((k_cand + chunk - 1) / chunk) < 1024) chunk /= 2;
  const dim3 grid((k_cand + chunk - 1) / chunk, p.n_q, p.n_seq);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
#define GO(RT, PAGED) score_gather_kernel<KDT, RT, Q8, PAGED, false><<<grid, 256, 0, st>>>(p, q, W, K, kscale, cand, k_cand, chunk, out, 0, nullptr, nullptr)
  if (p.H <= 32) {
    if (p.page_table) GO(1, true); else GO(1, false);
  } else {
    if (p.page_table) GO(2, true); else GO(2, false);
  }
#undef GO
  return hipGetLastError();
}

// Re-rank with the top-k inside the gather kernel: for many queries with candidate lists from which
// the top-k is sampled (one workgroup per query fills the chip, the list fits LDS) and the types the
// gather kernel takes.
bool rerank_fused_path(const Prob& p, int k_dtype, int q_dtype, int k_cand) {
  const bool types = (q_dtype == MISA_BF16 && k_dtype != MISA_F32) ||
                     (q_dtype == MISA_FP8_E4M3 && k_dtype == MISA_FP8_E4M3);
  return types && k_cand >= kRerankFusedMinList && k_cand <= kSmallTopkMax &&
         (long long)p.n_q * p.n_seq >= kRerankFusedMinRows;
}

template <int KDT, bool Q8>
static hipError_t launch_gather_topk(const Prob& p, const void* Q, const float* W, const void* K,
                                     const float* kscale, const int* cand, int k_cand, int k, int* idx,
                                     float* val, hipStream_t st) {
  const int chunk = (k_cand + 255) / 256 * 256;
  const dim3 grid(1, p.n_q, p.n_seq);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
#define GO(RT, PAGED) score_gather_kernel<KDT, RT, Q8, PAGED, true><<<grid, 256, 0, st>>>(p, q, W, K, kscale, cand, k_cand, chunk, nullptr, k, idx, val)
  if (p.H <= 32) {
    if (p.page_table) GO(1, true); else GO(1, false);
  } else {
    if (p.page_table) GO(2, true); else GO(2, false);
  }
#undef GO
  return hipGetLastError();
}

hipError_t launch_rerank_fused(const Prob& p, int k_dtype, int q_dtype, const void* Q, const float* W,
                               const void* K, const float* kscale, const int* cand, int k_cand, int k,
                               int* idx, float* val, hipStream_t st) {
  if (!rerank_fused_path(p, k_dtype, q_dtype, k_cand)) return hipErrorInvalidValue;
  if (q_dtype == MISA_FP8_E4M3) return launch_gather_topk<MISA_FP8_E4M3, true>(p, Q, W, K, kscale, cand, k_cand, k, idx, val, st);
  if (k_dtype == MISA_BF16) return launch_gather_topk<MISA_BF16, false>(p, Q, W, K, kscale, cand, k_cand, k, idx, val, st);
  return launch_gather_topk<MISA_FP8_E4M3, false>(p, Q, W, K, kscale, cand, k_cand, k, idx, val, st);
}

hipError_t launch_score(const Prob& p, int k_dtype, int q_dtype, const void* Q, const float* W,
                        const int* heads, const void* K, const float* kscale, const int* cand,
                        int k_cand, float* out, hipStream_t st) {
  if (cand && !heads && q_dtype == MISA_FP8_E4M3 && k_dtype == MISA_FP8_E4M3)
    return launch_gather<MISA_FP8_E4M3, true>(p, Q, W, K, kscale, cand, k_cand, out, st);
  if (cand && !heads && q_dtype == MISA_BF16 && k_dtype != MISA_F32) {
    if (k_dtype == MISA_BF16) return launch_gather<MISA_BF16, false>(p, Q, W, K, kscale, cand, k_cand, out, st);
    return launch_gather<MISA_FP8_E4M3, false>(p, Q, W, K, kscale, cand, k_cand, out, st);
  }
  if (!cand && tile_path(p, k_dtype, q_dtype))
    return launch_tile_mode(p, k_dtype, q_dtype, kTileStore, TileAux{}, Q, W, heads, K, kscale, out, st);
  if (q_dtype == MISA_FP8_E4M3) return hipErrorInvalidValue;   // fp8 codes reach only the tile kernel
  const bool mfma_ok = !cand && q_dtype == MISA_BF16 && k_dtype != MISA_F32;
  if (mfma_ok) {
    if (k_dtype == MISA_BF16) return launch_stream<MISA_BF16>(p, Q, W, heads, K, kscale, out, st);
    return launch_stream<MISA_FP8_E4M3>(p, Q, W, heads, K, kscale, out, st);
  }
#define GEN(KD, QD) return launch_generic<KD, QD>(p, Q, W, heads, K, kscale, cand, k_cand, out, st)
  if (q_dtype == MISA_F32) {
    if (k_dtype == MISA_F32) GEN(MISA_F32, MISA_F32);
    if (k_dtype == MISA_BF16) GEN(MISA_BF16, MISA_F32);
    GEN(MISA_FP8_E4M3, MISA_F32);
  }
  if (k_dtype == MISA_F32) GEN(MISA_F32, MISA_BF16);
  if (k_dtype == MISA_BF16) GEN(MISA_BF16, MISA_BF16);
  GEN(MISA_FP8_E4M3, MISA_BF16);
#undef GEN
}

}  // namespace misa
