// Comparison indexers assembled from the library's own stages: HISA (preliminaries,
// "Indexer in HISA": Eq. block_score, Eq. final_topk) and the MoBA-style Block-Sparse
// selector (Experimental results, "Baselines").
//
//   block scores  J[t,b] = sum over ALL heads of w_j ReLU(q_j . k~_b) for the complete
//                 blocks inside the query's visible prefix (block_score_tile_kernel on the
//                 matrix core; block_score_kernel, fp32 FMA, for fp32 queries);
//   block choice  the first and the last block always, the best other blocks up to m in
//                 all: both get score +inf and the row top-k kernel takes m;
//   HISA          the tokens of those blocks are the candidate list of the dense fine
//                 stage (the re-rank kernels of misa_rerank);
//   Block-Sparse  the tokens of those blocks are the selection.
#include <algorithm>

#include "kernels.h"

namespace misa {

// One thread per pooled block of one query; the query's head rows sit in LDS as floats.
// Only complete blocks strictly inside the prefix are scored, from Kp: the first block
// and the last one (the only one that can be partial) are always kept, so their scores
// are never compared and are set to +inf; blocks past the prefix get -inf.
__global__ __launch_bounds__(256) void block_score_kernel(Prob p, const void* __restrict__ Q,
                                                          const float* __restrict__ W,
                                                          const float* __restrict__ Kp,
                                                          float* __restrict__ J) {
  __shared__ float qs[kMaxH][kD];
  __shared__ float wsm[kMaxH];
  using QV = Vec16<MISA_F32>;
  const int t = blockIdx.y, seq = blockIdx.z, tid = threadIdx.x;
  const int n = visible(p, seq, t);
  const int Mn = (int)(((long long)n + p.B - 1) / p.B);
  const size_t qrow = (size_t)seq * p.n_q + t;
  const int b = blockIdx.x * 256 + tid;

  for (int i = tid; i < p.H * (kD / QV::N); i += 256) {
    const int j = i / (kD / QV::N), c = i % (kD / QV::N);
    float v[QV::N];
    QV::load(static_cast<const char*>(Q) + ((qrow * p.H + j) * kD + c * QV::N) * (QV::ROW_BYTES / kD), v);
#pragma unroll
    for (int e = 0; e < QV::N; ++e) qs[j][c * QV::N + e] = v[e];
  }
  for (int j = tid; j < p.H; j += 256) wsm[j] = W[qrow * p.H + j];
  __syncthreads();
  if (b >= p.M) return;
  float out = -INFINITY;
  if (b < Mn) {
    if (b == 0 || b == Mn - 1) {
      out = INFINITY;  // always kept
    } else {
      float kv[kD];
      const float* src = Kp + ((size_t)seq * p.M + b) * kD;
#pragma unroll
      for (int c = 0; c < kD; c += 4) {
        const float4 v = *reinterpret_cast<const float4*>(src + c);
        kv[c] = v.x; kv[c + 1] = v.y; kv[c + 2] = v.z; kv[c + 3] = v.w;
      }
      float total = 0.f;
      for (int j = 0; j < p.H; ++j) {
        float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
#pragma unroll
        for (int c = 0; c < kD; c += 4) {
          d0 = fmaf(qs[j][c], kv[c], d0);
          d1 = fmaf(qs[j][c + 1], kv[c + 1], d1);
          d2 = fmaf(qs[j][c + 2], kv[c + 2], d2);
          d3 = fmaf(qs[j][c + 3], kv[c + 3], d3);
        }
        total = fmaf(wsm[j], relu((d0 + d1) + (d2 + d3)), total);
      }
      out = total;
    }
  }
  J[qrow * p.M + b] = out;
}

// bf16 queries.  The products run on the matrix core with the fp32 pooled keys as three bf16 pieces (the
// nearest bf16, the nearest to the remainder, and to what remains of that: all 24 bits), so nothing of
// a key is lost; products are exact and added in fp32.  A wavefront keeps the pieces of 32 blocks in
// registers (96) and the head rows of the queries pass through LDS, double buffered, shared by the four
// wavefronts of the workgroup: a step is 64 (query, head) rows, HS = 64 or 32 head slots per query.
// The pieces of an infinite (or larger than bf16) component are not numbers, an infinity times a zero
// piece or a zero head slot is none either, and of a product above the largest fp32 the pieces' products may
// be infinities of both signs: blocks with such a key and queries with such a component, found
// from the exponents of the operands, are scored by themselves in fp32, in the order of block_score_kernel.
// Bound: 3 x 2 H 128 flop per (query, block).  1024 queries x 512 blocks x 64 heads: 33 us, 155 us with one
// thread per block on the vector units; error of the scores against 64 bits 1.3e-7 (1.5e-7 before).
union BFrag {
  bf16x8 v;
  uint4 u;
  uint32_t w[4];
};

__device__ __forceinline__ void split_three(float x0, float x1, uint32_t& a, uint32_t& b, uint32_t& c) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  union P { b2 v; uint32_t u; } h, m, l;
  f2 x = {x0, x1};
  h.v = __builtin_convertvector(x, b2);
  x = f2{x0 - __uint_as_float(h.u << 16), x1 - __uint_as_float(h.u & 0xFFFF0000u)};
  m.v = __builtin_convertvector(x, b2);
  x = f2{x[0] - __uint_as_float(m.u << 16), x[1] - __uint_as_float(m.u & 0xFFFF0000u)};
  l.v = __builtin_convertvector(x, b2);
  a = h.u;
  b = m.u;
  c = l.u;
}

// Whether one of the two bf16 values of a word is 2^63 or more, infinite or not a number (in bits 15 and 31).
// Products of smaller ones stay below 2^126 and those of the second and third piece, 128 of them added, too.
__device__ __forceinline__ uint32_t exponents_large(uint32_t w) {
  return ((w & 0x7F807F80u) + 0x21002100u) & 0x80008000u;
}

// The score of one block by itself: heads rows of a query in LDS, `slots` 16-byte pieces apart.
__device__ __forceinline__ float block_score_plain(const uint4* rows, int slots, const float* gate, int heads,
                                                const float* __restrict__ key) {
  float total = 0.f;
  for (int j = 0; j < heads; ++j) {
    float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
    for (int c = 0; c < 16; ++c) {
      const uint4 q = rows[j * slots + c];
      const float4 x = *reinterpret_cast<const float4*>(key + 8 * c), y = *reinterpret_cast<const float4*>(key + 8 * c + 4);
      d0 = fmaf(__uint_as_float(q.x << 16), x.x, d0);
      d1 = fmaf(__uint_as_float(q.x & 0xFFFF0000u), x.y, d1);
      d2 = fmaf(__uint_as_float(q.y << 16), x.z, d2);
      d3 = fmaf(__uint_as_float(q.y & 0xFFFF0000u), x.w, d3);
      d0 = fmaf(__uint_as_float(q.z << 16), y.x, d0);
      d1 = fmaf(__uint_as_float(q.z & 0xFFFF0000u), y.y, d1);
      d2 = fmaf(__uint_as_float(q.w << 16), y.z, d2);
      d3 = fmaf(__uint_as_float(q.w & 0xFFFF0000u), y.w, d3);
    }
    total = fmaf(gate[j], relu((d0 + d1) + (d2 + d3)), total);
  }
  return total;
}

template <int HS>
__global__ __launch_bounds__(256) void block_score_tile_kernel(Prob p, int steps, const uint16_t* __restrict__ Q,
                                                               const float* __restrict__ W,
                                                               const float* __restrict__ Kp,
                                                               float* __restrict__ J) {
  constexpr int QPS = 64 / HS;                  // queries per step
  constexpr int SLOTS = 17;                     // 16-byte slots per row in LDS: 16 and one of padding
  __shared__ uint4 rows[2][64 * SLOTS];
  __shared__ __align__(16) float gate[2][64];
  __shared__ int blocks_of[2][QPS];             // blocks in a query's prefix
  __shared__ int odd_step[2];                   // the step itself (from 1) if a query component is not finite
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, hf = lane >> 5, seq = blockIdx.z;
  const int q_first = blockIdx.y * steps * QPS;
  const int n_steps = min(steps, (p.n_q - q_first + QPS - 1) / QPS);
  const int b = (blockIdx.x * 4 + wave) * 32 + col;   // this lane's block

  if (tid < 2) odd_step[tid] = 0;
  BFrag piece[3][8];
  uint32_t odd_key = 0;                         // a component of this lane's block has no three pieces
  {
    const float* src = Kp + ((size_t)seq * p.M + min(b, p.M - 1)) * kD + hf * 8;
    float4 x[8][2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      x[ks][0] = *reinterpret_cast<const float4*>(src + ks * 16);
      x[ks][1] = *reinterpret_cast<const float4*>(src + ks * 16 + 4);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const float v[8] = {x[ks][0].x, x[ks][0].y, x[ks][0].z, x[ks][0].w, x[ks][1].x, x[ks][1].y, x[ks][1].z, x[ks][1].w};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        split_three(v[2 * j], v[2 * j + 1], piece[0][ks].w[j], piece[1][ks].w[j], piece[2][ks].w[j]);
#pragma unroll
      for (int j = 0; j < 4; ++j) odd_key |= exponents_large(piece[0][ks].w[j]);
    }
    odd_key |= (uint32_t)__shfl_xor((int)odd_key, 32);
  }

  uint4 stage[4];
  float stage_gate = 0.f;
  int stage_blocks = 0, stage_step = 0;
  auto load = [&](int step) {                   // rows of a step; missing queries and heads are zeros
    const int q0 = q_first + step * QPS;
    stage_step = step + 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i, row = e >> 4, q = q0 + row / HS, head = row % HS;
      const size_t at = (((size_t)seq * p.n_q + min(q, p.n_q - 1)) * p.H + min(head, p.H - 1)) * kD + (e & 15) * 8;
      const uint4 v = *reinterpret_cast<const uint4*>(Q + at);
      stage[i] = q < p.n_q && head < p.H ? v : make_uint4(0, 0, 0, 0);
    }
    if (tid < 64) {
      const int q = q0 + tid / HS, head = tid % HS;
      stage_gate = q < p.n_q && head < p.H ? W[((size_t)seq * p.n_q + q) * p.H + head] : 0.f;
    }
    if (tid < QPS)
      stage_blocks = q0 + tid < p.n_q ? (int)(((long long)visible(p, seq, q0 + tid) + p.B - 1) / p.B) : 0;
  };
  auto store = [&](int buf) {
    uint32_t odd = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;
      rows[buf][(e >> 4) * SLOTS + (e & 15)] = stage[i];
      odd |= exponents_large(stage[i].x) | exponents_large(stage[i].y) | exponents_large(stage[i].z) | exponents_large(stage[i].w);
    }
    if (odd) odd_step[buf] = stage_step;
    if (tid < 64) gate[buf][tid] = stage_gate;
    if (tid < QPS) blocks_of[buf][tid] = stage_blocks;
  };

  load(0);
  __syncthreads();                              // (odd_step is clear)
  store(0);
  __syncthreads();
  for (int step = 0; step < n_steps; ++step) {
    const int buf = step & 1;
    load(min(step + 1, n_steps - 1));
    f32x16 acc[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        BFrag a;
        a.u = rows[buf][(rt * 32 + col) * SLOTS + 2 * ks + hf];
        // smallest pieces first
        acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, piece[2][ks].v, acc[rt], 0, 0, 0);
        acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, piece[1][ks].v, acc[rt], 0, 0, 0);
        acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, piece[0][ks].v, acc[rt], 0, 0, 0);
      }
    }
    float sum[2];                               // heads of row tile rt, block b
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      float part[2] = {0.f, 0.f};
#pragma unroll
      for (int g = 0; g < 4; ++g) {             // accumulator registers 4 g .. + 3: rows 8 g + 4 hf .. + 3
        const float4 w = *reinterpret_cast<const float4*>(&gate[buf][rt * 32 + 8 * g + 4 * hf]);
        part[g & 1] = fmaf(w.x, relu(acc[rt][4 * g]), part[g & 1]);
        part[g & 1] = fmaf(w.y, relu(acc[rt][4 * g + 1]), part[g & 1]);
        part[g & 1] = fmaf(w.z, relu(acc[rt][4 * g + 2]), part[g & 1]);
        part[g & 1] = fmaf(w.w, relu(acc[rt][4 * g + 3]), part[g & 1]);
      }
      sum[rt] = part[0] + part[1];
      sum[rt] += __shfl_xor(sum[rt], 32);
    }
    // HS = 64: both row tiles are one query's, the lower half-wave stores; HS = 32: half-wave hf stores
    // the query of row tile hf
    const int q = q_first + step * QPS + (HS == 32 ? hf : 0);
    float total = HS == 64 ? sum[0] + sum[1] : hf ? sum[1] : sum[0];
    const int Mn = blocks_of[buf][HS == 32 ? hf : 0];
    // (only blocks whose score is used: what lies behind a prefix may hold anything)
    const bool odd = (odd_key != 0 || odd_step[buf] == step + 1) && b > 0 && b < Mn - 1;
    if (__builtin_amdgcn_ballot_w64(odd)) {
      const int first = HS == 32 ? 32 * hf : 0;
      if (odd)
        total = block_score_plain(&rows[buf][first * SLOTS], SLOTS, &gate[buf][first], p.H,
                                  Kp + ((size_t)seq * p.M + min(b, p.M - 1)) * kD);
    }
    if ((HS == 32 || hf == 0) && q < p.n_q && b < p.M)
      J[((size_t)seq * p.n_q + q) * p.M + b] = b >= Mn ? -INFINITY : (b == 0 || b == Mn - 1) ? INFINITY : total;
    store(buf ^ 1);
    __syncthreads();
  }
}

// cand[row, i * B + o] = token o of the i-th selected block, -1 if the block slot is
// empty or the token is not visible.
// V: slots per thread, all of one block (4: 16-byte stores, 20 us with one slot per thread for 1024 x 8192).
template <int V>
__global__ __launch_bounds__(256) void expand_blocks_kernel(Prob p, int m, const int* __restrict__ blocks,
                                                            int* __restrict__ cand) {
  const int t = blockIdx.y, seq = blockIdx.z;
  const size_t row = (size_t)seq * p.n_q + t;
  const int n = visible(p, seq, t);
  const uint32_t slots = (uint32_t)m * (uint32_t)p.B;      // at most 16384
  const uint32_t slot = (blockIdx.x * 256 + threadIdx.x) * V;
  if (slot >= slots) return;
  const uint32_t i = slot / (uint32_t)p.B, o = slot % (uint32_t)p.B;
  const int b = blocks[row * m + i];
  int tok[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const long long at = (long long)b * p.B + o + v;
    tok[v] = b >= 0 && at < n ? (int)at : -1;
  }
  int* dst = cand + row * (size_t)slots + slot;
  if constexpr (V == 4) *reinterpret_cast<int4*>(dst) = make_int4(tok[0], tok[1], tok[2], tok[3]);
  else dst[0] = tok[0];
}

namespace {
size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
}

size_t hisa_ws_bytes(const Prob& p, int m) {
  if (m < 2) return 0;
  const size_t rows = (size_t)p.n_seq * p.n_q, kc = (size_t)m * p.B;
  return up256(rows * p.M * sizeof(float)) + up256(rows * m * sizeof(int)) + up256(rows * kc * sizeof(int)) +
         up256(rows * kc * sizeof(float));
}

// k == 0: Block-Sparse (idx receives the m * B candidate tokens); otherwise HISA.
hipError_t launch_hisa(const Prob& p, int k_dtype, int q_dtype, const void* Q, const float* W,
                       const float* Kp, const void* K, const float* kscale, int m, int k, int* blocks,
                       int* idx, float* val, void* ws, hipStream_t st) {
  const size_t rows = (size_t)p.n_seq * p.n_q, kc = (size_t)m * p.B;
  char* base = static_cast<char*>(ws);
  float* J = reinterpret_cast<float*>(base);
  int* C = reinterpret_cast<int*>(base + up256(rows * p.M * sizeof(float)));
  int* cand = reinterpret_cast<int*>(reinterpret_cast<char*>(C) + up256(rows * m * sizeof(int)));
  float* dense = reinterpret_cast<float*>(reinterpret_cast<char*>(cand) + up256(rows * kc * sizeof(int)));
  if (blocks) C = blocks;
  if (k == 0) cand = idx;

  const dim3 g1((p.M + 255) / 256, p.n_q, p.n_seq);
  if (q_dtype == MISA_F32) block_score_kernel<<<g1, 256, 0, st>>>(p, Q, W, Kp, J);
  else {
    // steps per workgroup: as many as leave about two resident sets of workgroups (the pieces of a
    // workgroup's blocks are made once), at most 16
    const int qps = p.H > 32 ? 1 : 2, tiles = (p.M + 127) / 128, all = (p.n_q + qps - 1) / qps;
    const int steps = (int)std::min(16ll, std::max(1ll, (long long)all * tiles * p.n_seq / 1024));
    const dim3 g(tiles, (all + steps - 1) / steps, p.n_seq);
    const uint16_t* q = static_cast<const uint16_t*>(Q);
    if (qps == 1) block_score_tile_kernel<64><<<g, 256, 0, st>>>(p, steps, q, W, Kp, J);
    else block_score_tile_kernel<32><<<g, 256, 0, st>>>(p, steps, q, W, Kp, J);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the m best blocks of every row of J (all M slots are scanned, -inf slots never chosen)
  e = launch_topk(p, J, p.M, m, nullptr, C, nullptr, nullptr, st, nullptr, true);
  if (e != hipSuccess) return e;
  const bool by_four = p.B % 4 == 0 && (reinterpret_cast<uintptr_t>(cand) & 15) == 0;
  const dim3 g3((unsigned)((kc + (by_four ? 1023 : 255)) / (by_four ? 1024 : 256)), p.n_q, p.n_seq);
  if (by_four) expand_blocks_kernel<4><<<g3, 256, 0, st>>>(p, m, C, cand);
  else expand_blocks_kernel<1><<<g3, 256, 0, st>>>(p, m, C, cand);
  if ((e = hipGetLastError()) != hipSuccess || k == 0) return e;
  // many queries: dense scores and their top-k in one kernel, as in misa_rerank
  if (rerank_fused_path(p, k_dtype, q_dtype, (int)kc))
    return launch_rerank_fused(p, k_dtype, q_dtype, Q, W, K, kscale, cand, (int)kc, k, idx, val, st);
  e = launch_score(p, k_dtype, q_dtype, Q, W, nullptr, K, kscale, cand, (int)kc, dense, st);
  if (e != hipSuccess) return e;
  return launch_topk(p, dense, (int)kc, k, cand, idx, val, nullptr, st);
}

}  // namespace misa
