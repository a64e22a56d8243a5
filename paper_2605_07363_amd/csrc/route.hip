// Stage 2: block-pooled head router (Eq. misa_route_score, Eq. misa_route).
//
// route_tile_kernel (bf16 queries): the [queries x heads, 128] x [128, blocks]
// product runs on the matrix core.  Query-head rows are the stationary operand
// (registers); the fp32 pooled keys stream through LDS as two bf16 tiles, the
// bf16 nearest to each value and the bf16 nearest to the exact remainder, and
// both are multiplied, so the products carry the pooled key to 2^-17 relative.  ReLU, the causal
// block mask and the sum over blocks stay in accumulator lanes until the end
// of the block range, when they are added by lane shifts and go through LDS to one
// lane per row, which writes the partial sum to the workspace.  (333 queries of 64
// heads, 157 blocks, with the finalisation: 26.9 us with 160 lane exchanges and a
// division per row and lane, tiles requested after the causal limits were known, and a
// finalisation of dependent rounds; 14.5 us now.)
// route_partial_kernel (fp32 queries): lane = head.  Each lane keeps its query head in
// registers; the pooled key of the block being visited is the same for the
// whole wavefront, so it is fetched with wave-uniform (scalar) loads and every
// FMA takes one scalar and one vector operand.  The four wavefronts of a
// workgroup stride over the blocks of one split of the prefix; partial sums of
// ReLU(q.k~) go to the workspace.
// route_finalize_kernel: adds the causal tail block (mean of the raw keys of
// the last, partial block of a query that does not sit at the end of the
// cache), scales by |w| / M_n and selects the top-h heads by rank counting.
#include <algorithm>

#include "kernels.h"

namespace misa {

template <int QDT>
__device__ __forceinline__ void load_query_head(const void* Q, size_t head_index, float* qv) {
  using V = Vec16<QDT>;
  const char* src = static_cast<const char*>(Q) + head_index * V::ROW_BYTES;
#pragma unroll
  for (int c = 0; c < kD / V::N; ++c) V::load(src + c * 16, qv + c * V::N);
}

// Two fp32 values -> two packed bf16 pairs whose sums represent them to 2^-17 relative: hi is
// the bf16 nearest to the value, lo the bf16 nearest to the (exactly computed) remainder.
// Element 0 sits in the low half of each word.
typedef __bf16 bf16x2_r __attribute__((ext_vector_type(2)));
typedef float f32x2_r __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  union { bf16x2_r b; uint32_t u; } h, l;
  const f32x2_r v = {x0, x1};
  h.b = __builtin_convertvector(v, bf16x2_r);
  const f32x2_r r = {x0 - __uint_as_float(h.u << 16), x1 - __uint_as_float(h.u & 0xFFFF0000u)};
  l.b = __builtin_convertvector(r, bf16x2_r);
  hi = h.u;
  lo = l.u;
}

// Blocks whose pooled key in Kp is valid for a query with prefix n: all
// ceil(n/B) when the query sits at the end of the cache (the partial block in
// Kp then holds exactly its tokens), else only the complete ones.
__device__ __forceinline__ int pooled_blocks(int n, int len, int B) {
  const int full = n / B;
  return full + ((n == len && full * B != n) ? 1 : 0);
}

template <int QDT>
__global__ __launch_bounds__(256) void route_partial_kernel(Prob p, int splits,
                                                            const void* __restrict__ Q,
                                                            const float* __restrict__ Kp,
                                                            float* __restrict__ part) {
  __shared__ float red[4][kWave];
  const int split = blockIdx.x, t = blockIdx.y, seq = blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = visible(p, seq, t), len = seq_length(p, seq);
  const int nb = pooled_blocks(n, len, p.B);
  const int per = (p.M + splits - 1) / splits;
  const int b_lo = split * per, b_hi = min(b_lo + per, nb);

  // the query's rows are read whole, in thread order, and go through LDS to the lanes (rows padded by 16 bytes; 6.8 -> 4.4 us
  // for one query of 64 heads and 64 blocks, where every lane of every wavefront read its row by itself)
  using QV = Vec16<QDT>;
  constexpr int CPH = kD / QV::N, PITCH = CPH + 1;
  __shared__ u32x4 s_q[kWave * PITCH];
  float qv[kD];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const char*>(Q) + ((size_t)seq * p.n_q + t) * p.H * QV::ROW_BYTES);
    u32x4 v[kWave * CPH / 256];
#pragma unroll
    for (int i = 0; i < kWave * CPH / 256; ++i) v[i] = src[min((int)threadIdx.x + 256 * i, p.H * CPH - 1)];
#pragma unroll
    for (int i = 0; i < kWave * CPH / 256; ++i) {
      const int e = threadIdx.x + 256 * i;
      s_q[(e / CPH) * PITCH + e % CPH] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPH; ++c) QV::unpack(s_q[lane * PITCH + c], qv + c * QV::N);
  }

  float acc = 0.f;
  for (int b = b_lo + wave; b < b_hi; b += 4) {
    const float* __restrict__ kp = Kp + ((size_t)seq * p.M + b) * kD;  // wave-uniform
    float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
#pragma unroll
    for (int c = 0; c < kD; c += 4) {
      d0 = fmaf(qv[c], kp[c], d0);
      d1 = fmaf(qv[c + 1], kp[c + 1], d1);
      d2 = fmaf(qv[c + 2], kp[c + 2], d2);
      d3 = fmaf(qv[c + 3], kp[c + 3], d3);
    }
    acc += fmaxf((d0 + d1) + (d2 + d3), 0.f);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    const float s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    part[(((size_t)seq * p.n_q + t) * splits + split) * kWave + lane] = s;
  }
}

constexpr int kRouteKT = 32;  // pooled blocks per LDS tile

// Sum over each row of 16 lanes, in its lane 15 (all lanes of the wavefront active).
__device__ __forceinline__ float row16_sum(float v) {
#define MISA_DPP_ADD(ctrl) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true))
  MISA_DPP_ADD(0x111);  // row_shr:1
  MISA_DPP_ADD(0x112);  // row_shr:2
  MISA_DPP_ADD(0x114);  // row_shr:4
  MISA_DPP_ADD(0x118);  // row_shr:8
#undef MISA_DPP_ADD
  return v;
}

// Sum over each half of the wavefront, in its last lane (all lanes active).
__device__ __forceinline__ float half_sum(float v) {
  v = row16_sum(v);
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));   // row_bcast:15
}

union RFrag {
  bf16x8 v;
  uint4 u;
  u32x4 x;
};

// RG wavefronts of a workgroup own different 64-row groups; the other 4 / RG
// "phases" take every (4 / RG)-th block tile of the same rows.
template <int RG>
__global__ __launch_bounds__(256) void route_tile_kernel(Prob p, int splits,
                                                         const uint16_t* __restrict__ Q,
                                                         const float* __restrict__ Kp,
                                                         float* __restrict__ part) {
  constexpr int CP = 4 / RG;
  __shared__ uint2 tile[2][2][kRouteKT * 32];  // [buffer][hi | lo][block row * 32 + 8-byte slot]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, hf = lane >> 5;
  const int split = blockIdx.x, seq = blockIdx.z;
  const int rg = wave % RG, phase = wave / RG;
  const int rows_per_seq = p.n_q * p.H;
  const int row0 = (blockIdx.y * RG + rg) * 64;  // first (query, head) row of this wavefront
  const int len = seq_length(p, seq);

  const int per = (p.M + splits - 1) / splits;
  const int b_lo = split * per, b_hi = min(b_lo + per, p.M);

  // (the first tiles are requested before anything else: with a few tiles per workgroup the kernel is their latency)
  const float* kp_seq = Kp + (size_t)seq * p.M * kD;
  float4 stage[2][4];  // two sets: with CP == 1 tiles are requested two iterations ahead
  auto load_tile = [&](int b0, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;               // float4 index inside the 32 x 128 tile
      const int row = e >> 5;
      stage[SET][i] = *reinterpret_cast<const float4*>(kp_seq + (size_t)min(b0 + row, p.M - 1) * kD + (e & 31) * 4);
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  load_tile(b_lo, Set1{});
  if (CP == 1) load_tile(b_lo + kRouteKT, Set0{});  // staged during the first iteration

  // stationary operand
  RFrag a[2][8];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const int row = row0 + rt * 32 + col;
    const uint16_t* src = Q + ((size_t)seq * rows_per_seq + min(row, rows_per_seq - 1)) * kD + hf * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint4 v = *reinterpret_cast<const uint4*>(src + ks * 16);
      a[rt][ks].u = row < rows_per_seq ? v : make_uint4(0, 0, 0, 0);
    }
  }
  // per row of the wavefront, the number of pooled blocks it may use (its own prefix, cut at
  // the end of this split); kept in LDS because only tiles on the causal edge need it
  __shared__ int s_nb[4][64];
  int nb_lane = 0;
  {
    const int rr = row0 + lane;
    if (rr < rows_per_seq) nb_lane = min(pooled_blocks(visible(p, seq, rr / p.H), len, p.B), b_hi);
    s_nb[wave][lane] = nb_lane;
  }
  int nb_max = nb_lane, nb_min = nb_lane;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    nb_max = max(nb_max, __shfl_xor(nb_max, o));
    nb_min = min(nb_min, __shfl_xor(nb_min, o));
  }
  // tiles that end at or before this limit are visible in full to every row of the wavefront
  const int b_full = __builtin_amdgcn_readfirstlane(nb_min);
  // the block range this workgroup must visit: up to the largest count of any of its rows
  __shared__ int s_stop;
  if (tid == 0) s_stop = 0;
  __syncthreads();
  if (lane == 0) atomicMax(&s_stop, nb_max);
  __syncthreads();
  const int b_stop = s_stop;

  auto store_tile = [&](int buf, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;
      const int row = e >> 5, c4 = e & 31;        // c4: group of 4 components
      const float x[4] = {stage[SET][i].x, stage[SET][i].y, stage[SET][i].z, stage[SET][i].w};
      uint32_t hi[2], lo[2];
      split_pair(x[0], x[1], hi[0], lo[0]);
      split_pair(x[2], x[3], hi[1], lo[1]);
      // 16-byte chunk c4 / 2 of the row, XOR-swizzled by the row; 8-byte half c4 & 1
      const int slot = row * 32 + (((c4 >> 1) ^ (row & 15)) << 1) + (c4 & 1);
      tile[buf][0][slot] = make_uint2(hi[0], hi[1]);
      tile[buf][1][slot] = make_uint2(lo[0], lo[1]);
    }
  };

  float sum[2][16];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[rt][r] = 0.f;

  int buf = 0;
  if (b_lo < b_stop) store_tile(0, Set1{});
  __builtin_amdgcn_s_waitcnt(0);  // prologue loads have landed; in-loop waits concern only loop loads
  __syncthreads();
  int it = 0;
  // One iteration.  CP == 1: the set named by set_tag holds the next tile (requested an iteration
  // ago) and is staged between the matrix instructions, the tile after it is requested into the
  // other set.  Otherwise one set is loaded at the top and staged at the bottom.  Tiles past the
  // last are requested and staged too, with clamped addresses (never read): the body stays one
  // scheduling region.
  auto iteration = [&](int b0, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
    if (CP == 1) load_tile(b0 + 2 * kRouteKT, std::integral_constant<int, SET ^ 1>{});
    else load_tile(b0 + kRouteKT, Set0{});
    if (it % CP == phase) {
      f32x16 acc[2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[rt][r] = 0.f;
      const uint4* hi_t = reinterpret_cast<const uint4*>(tile[buf][0]);
      const uint4* lo_t = reinterpret_cast<const uint4*>(tile[buf][1]);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        RFrag bh, bl;
        const int idx = col * 16 + ((ks * 2 + hf) ^ (col & 15));
        bh.u = hi_t[idx];
        bl.u = lo_t[idx];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[rt][ks].v, bh.v, acc[rt], 0, 0, 0);
          acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[rt][ks].v, bl.v, acc[rt], 0, 0, 0);
        }
      }
      if (CP == 1) {
        // staging the next tile (split into pieces, LDS writes) needs nothing from these matrix
        // instructions and its data arrived an iteration ago: it sits in the same scheduling
        // region, ahead of the sums that have to wait for them
        store_tile(buf ^ 1, set_tag);
      }
      if (b0 + kRouteKT <= b_full) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[rt][r] += relu(acc[rt][r]);
      } else {
        const int b = b0 + col;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int4 nb = *reinterpret_cast<const int4*>(&s_nb[wave][rt * 32 + 8 * g + 4 * hf]);
            sum[rt][4 * g + 0] += b < nb.x ? relu(acc[rt][4 * g + 0]) : 0.f;
            sum[rt][4 * g + 1] += b < nb.y ? relu(acc[rt][4 * g + 1]) : 0.f;
            sum[rt][4 * g + 2] += b < nb.z ? relu(acc[rt][4 * g + 2]) : 0.f;
            sum[rt][4 * g + 3] += b < nb.w ? relu(acc[rt][4 * g + 3]) : 0.f;
          }
      }
    }
    if (CP != 1) store_tile(buf ^ 1, Set0{});
    __syncthreads();
    buf ^= 1;
    ++it;
  };
  for (int b0 = b_lo; b0 < b_stop;) {
    iteration(b0, Set0{});
    b0 += kRouteKT;
    if (b0 >= b_stop) break;
    if (CP == 1) iteration(b0, Set1{}); else iteration(b0, Set0{});
    b0 += kRouteKT;
  }

  // sum over the 32 block columns of each half-wave; the sums go through LDS of the wavefront to one lane per row
  __shared__ __align__(16) float s_sum[4][64];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 v = make_float4(half_sum(sum[rt][4 * g]), half_sum(sum[rt][4 * g + 1]), half_sum(sum[rt][4 * g + 2]),
                                   half_sum(sum[rt][4 * g + 3]));
      if (col == 31) *reinterpret_cast<float4*>(&s_sum[wave][rt * 32 + 8 * g + 4 * hf]) = v;
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int rr = row0 + lane;
  if (rr < rows_per_seq) {
    const int t = rr / p.H, j = rr - t * p.H;
    part[(((size_t)seq * p.n_q + t) * (splits * CP) + split * CP + phase) * kWave + j] = s_sum[wave][lane];
  }
}

// Few query-head rows (decode: n_q * H <= 64 in one workgroup; up to 7 queries of any head count: blockIdx.z
// is the query): a wavefront takes 16 pooled blocks at a time as the columns
// of v_mfma_f32_16x16x32_bf16, loads them straight into matrix fragments (a lane reads 32 contiguous bytes
// of a pooled key per k-step) and splits them into two bf16 pieces in registers; RT 16-row tiles of head
// rows are the other operand.  The sums over a wavefront's columns are four shifted adds inside rows of 16
// lanes, the four wavefronts of a workgroup add theirs through LDS: one partial sum per row and 64 blocks.
// Bound by latency: one round of loads, few instructions.  (32 blocks per wavefront on the 32x32 instruction,
// the columns added by lane exchanges, a partial sum per wavefront: 14-15 us
// for 64 heads against 6-8 us; four queries of 64 heads on the tile kernel 19 us.)
template <int RT>
__global__ __launch_bounds__(256) void route_few_kernel(Prob p, int tiles_per_wave, int n_parts,
                                                        const uint16_t* __restrict__ Q,
                                                        const float* __restrict__ Kp,
                                                        float* __restrict__ part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int seq = blockIdx.y;
  const int t0 = blockIdx.z, rows = gridDim.z > 1 ? p.H : p.n_q * p.H;   // first query, its (and the others') rows
  __shared__ __align__(16) int s_nb[kWave];     // pooled blocks a row may use
  __shared__ float s_sum[4][kWave];
  __shared__ u32x4 s_q[RT * 16 * 17];           // query rows, padded by one 16-byte slot

  // The rows are read whole and in thread order: fragments loaded by the lanes that need them touch 64 cache lines per
  // instruction, in every wavefront, and the texture addresser takes a clock for each (64 heads: 5.9 -> 4.3 us for one
  // query, 9.4 -> 7.5 us for 64 sequences, 9.7 -> 7.6 us for 16 sequences of four).
  u32x4 q[RT];
  {
    const u32x4* src = reinterpret_cast<const u32x4*>(Q + ((size_t)seq * p.n_q + t0) * p.H * kD);
#pragma unroll
    for (int i = 0; i < RT; ++i) q[i] = src[min(tid + 256 * i, rows * 16 - 1)];
  }
  const float* kp_seq = Kp + (size_t)seq * p.M * kD;
  float4 x[4][2];
  auto load = [&](int b0) {
    const float* src = kp_seq + (size_t)min(b0 + c, p.M - 1) * kD + g * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      x[ks][0] = *reinterpret_cast<const float4*>(src + ks * 32);
      x[ks][1] = *reinterpret_cast<const float4*>(src + ks * 32 + 4);
    }
  };
  const int first = ((int)blockIdx.x * 4 + wave) * tiles_per_wave * 16;
  load(first);
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int e = tid + 256 * i;
    s_q[(e >> 4) * 17 + (e & 15)] = q[i];
  }
  if (tid < kWave)
    s_nb[tid] = tid < rows ? min(pooled_blocks(visible(p, seq, t0 + tid / p.H), seq_length(p, seq), p.B), p.M) : 0;
  __syncthreads();
  RFrag a[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[rt][ks].x = s_q[(rt * 16 + c) * 17 + 4 * ks + g];
  float sum[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int j = 0; j < 4; ++j) sum[rt][j] = 0.f;

  for (int tl = 0; tl < tiles_per_wave; ++tl) {
    const int b0 = first + tl * 16;
    f32x4 acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const float v[8] = {x[ks][0].x, x[ks][0].y, x[ks][0].z, x[ks][0].w,
                          x[ks][1].x, x[ks][1].y, x[ks][1].z, x[ks][1].w};
      uint32_t hi[4], lo[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) split_pair(v[2 * j], v[2 * j + 1], hi[j], lo[j]);
      RFrag bh, bl;
      bh.u = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      bl.u = make_uint4(lo[0], lo[1], lo[2], lo[3]);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rt][ks].v, bh.v, acc[rt], 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rt][ks].v, bl.v, acc[rt], 0, 0, 0);
    }
    if (tl + 1 < tiles_per_wave) load(b0 + 16);
    // the accumulator of lane (c, g) holds rows 16 rt + 4 g + j of column c
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int4 nb = *reinterpret_cast<const int4*>(&s_nb[16 * rt + 4 * g]);
      sum[rt][0] += b0 + c < nb.x ? relu(acc[rt][0]) : 0.f;
      sum[rt][1] += b0 + c < nb.y ? relu(acc[rt][1]) : 0.f;
      sum[rt][2] += b0 + c < nb.z ? relu(acc[rt][2]) : 0.f;
      sum[rt][3] += b0 + c < nb.w ? relu(acc[rt][3]) : 0.f;
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = row16_sum(sum[rt][j]);    // in lane 15 of the 16
      if (c == 15) s_sum[wave][16 * rt + 4 * g + j] = v;
    }
  __syncthreads();
  if (tid < rows) {
    const int t = tid / p.H, j = tid - t * p.H;
    part[(((size_t)seq * p.n_q + t0 + t) * n_parts + blockIdx.x) * kWave + j] =
        (s_sum[0][tid] + s_sum[1][tid]) + (s_sum[2][tid] + s_sum[3][tid]);
  }
}

// Bound by latency for few queries (a chain of a few rounds of loads: what does not depend on another is requested
// first) and by reading the queries again for many: 4096 of 64 heads 23.6 -> 16.9 us, 333 of them 11.2 -> 5.9 us.
template <int KDT, int QDT>
__global__ __launch_bounds__(128) void route_finalize_kernel(
    Prob p, int splits, const void* __restrict__ Q, const float* __restrict__ W,
    const void* __restrict__ K, const float* __restrict__ kscale, const float* __restrict__ part,
    int* __restrict__ heads, float* __restrict__ E) {
  __shared__ __align__(16) float tailk[kD];
  __shared__ __align__(16) float tsum[128 / (kD / Vec16<KDT>::N)][kD];
  __shared__ __align__(16) float Es[kMaxH];
  __shared__ float sred[4][kMaxH];
  __shared__ float sdot[kMaxH];
  using KV = Vec16<KDT>;
  const int t = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x;
  const int n = visible(p, seq, t), len = seq_length(p, seq);
  const int nfull = n / p.B, r = n - nfull * p.B;
  const int Mn = nfull + (r > 0 ? 1 : 0);
  const bool tail = r > 0 && n < len;
  const size_t q_head = ((size_t)seq * p.n_q + t) * p.H + min(tid, p.H - 1);
  const float gate = W[q_head];   // (requested before the chain of round trips that it ends)

  // The query's H rows are one contiguous piece, read in 16-byte chunks in thread order; the first eight of a thread are
  // requested before the tail block, whose mean they wait for.
  using QV = Vec16<QDT>;
  constexpr int CPH = kD / QV::N;  // chunks per head row: 32 (fp32) or 16 (bf16)
  constexpr int QU = 8;
  const char* qrow = static_cast<const char*>(Q) + ((size_t)seq * p.n_q + t) * p.H * QV::ROW_BYTES;
  const int q_chunks = p.H * CPH;
  u32x4 qraw[QU];
  auto request_queries = [&](int base) {
#pragma unroll
    for (int u = 0; u < QU; ++u)
      qraw[u] = *reinterpret_cast<const u32x4*>(qrow + (size_t)min(base + 128 * u + tid, q_chunks - 1) * 16);
  };
  if (tail) {  // mean of keys nfull*B .. n-1
    // LPR consecutive lanes read a row, the workgroup RPI rows with one load each; eight loads in flight (the
    // workgroup's run time is the latency of these rounds)
    constexpr int LPR = kD / KV::N, RPI = 128 / LPR, U = 8;
    const int lr = tid / LPR, lp = tid % LPR;
    request_queries(0);
    float acc[KV::N];
#pragma unroll
    for (int e = 0; e < KV::N; ++e) acc[e] = 0.f;
    for (int row = nfull * p.B + lr; row < n; row += RPI * U) {
      float v[U][KV::N], scale[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const size_t slot = key_slot(p, seq, min(row + RPI * u, n - 1));
        KV::load(static_cast<const char*>(K) + slot * KV::ROW_BYTES + lp * 16, v[u]);
        scale[u] = KDT == MISA_FP8_E4M3 ? kscale[slot] : 1.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (row + RPI * u < n) {
#pragma unroll
          for (int e = 0; e < KV::N; ++e) acc[e] = KDT == MISA_FP8_E4M3 ? fmaf(v[u][e], scale[u], acc[e]) : acc[e] + v[u][e];
        }
    }
#pragma unroll
    for (int e = 0; e < KV::N; ++e) tsum[lr][lp * KV::N + e] = acc[e];
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < RPI; ++i) s += tsum[i][tid];
    tailk[tid] = s / (float)r;
  }
  // Partial sums of the block tiles: the 128 threads form 4 (H <= 32) or 2 groups of one thread
  // per head; group g adds the slots g, g + G, ... in order, eight loads in flight at a time,
  // and the groups' sums are added in group order below.
  {
    const int hp = p.H <= 32 ? 32 : 64, G = 128 / hp, g = tid / hp, j = tid % hp;
    float s = 0.f;
    if (j < p.H) {
      const float* ps = part + ((size_t)seq * p.n_q + t) * splits * kWave + j;
      for (int sp = g; sp < splits; sp += 8 * G) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = sp + u * G < splits ? ps[(size_t)(sp + u * G) * kWave] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
      }
    }
    sred[g][j] = s;
  }
  __syncthreads();

  if (tail) {
    // q_j . (tail mean) for all heads: the CPH consecutive lanes that hold a head's chunks add
    // their partial products, and the last of them keeps the sum.
    const int part_of = tid % CPH;
    float tk[QV::N];
#pragma unroll
    for (int e = 0; e < QV::N; ++e) tk[e] = tailk[part_of * QV::N + e];
    for (int base = 0; base < q_chunks; base += 128 * QU) {
      if (base > 0) request_queries(base);
#pragma unroll
      for (int u = 0; u < QU; ++u) {
        const int c = base + 128 * u + tid;
        float v[QV::N], d = 0.f;
        QV::unpack(qraw[u], v);
#pragma unroll
        for (int e = 0; e < QV::N; ++e) d = fmaf(v[e], tk[e], d);
        d = CPH == 32 ? half_sum(d) : row16_sum(d);
        if (part_of == CPH - 1 && c < q_chunks) sdot[c / CPH] = d;
      }
    }
    __syncthreads();
  }

  if (tid < kMaxH) {   // one wavefront
    float e = -INFINITY;
    if (tid < p.H) {
      float s = sred[0][tid] + sred[1][tid];
      if (p.H <= 32) s += sred[2][tid] + sred[3][tid];
      if (tail) s += fmaxf(sdot[tid], 0.f);
      e = Mn > 0 ? fabsf(gate) * s / (float)Mn : 0.f;
      if (E) E[q_head] = e;
    }
    Es[tid] = e;
    __builtin_amdgcn_wave_barrier();   // (the wavefront's own writes: LDS keeps their order)
    int rank = 0;
#pragma unroll 4
    for (int i = 0; i < kMaxH; i += 4) {   // (rows past H hold -inf and rank behind every head)
      const float4 o = *reinterpret_cast<const float4*>(&Es[i]);
      rank += (o.x > e || (o.x == e && i < tid)) ? 1 : 0;
      rank += (o.y > e || (o.y == e && i + 1 < tid)) ? 1 : 0;
      rank += (o.z > e || (o.z == e && i + 2 < tid)) ? 1 : 0;
      rank += (o.w > e || (o.w == e && i + 3 < tid)) ? 1 : 0;
    }
    const bool chosen = tid < p.H && rank < p.h;
    const unsigned long long mask = __ballot(chosen);
    const int pos = __popcll(mask & ((1ull << tid) - 1ull));
    if (chosen && pos < p.h) heads[((size_t)seq * p.n_q + t) * p.h + pos] = tid;   // (NaN scores rank first together)
  }
}

// Content-free router scores of the routing-score ablation (appendix "Ablation: routing
// score"): kind 1: E_j = w_j, the gate itself; kind 2: E_j = ||q_j||_2.  Same top-h rule.
// One wavefront per query, lane = head.
template <int QDT>
__global__ __launch_bounds__(64) void route_proxy_kernel(Prob p, int kind, const void* __restrict__ Q,
                                                         const float* __restrict__ W,
                                                         int* __restrict__ heads,
                                                         float* __restrict__ E) {
  __shared__ float Es[kWave];
  __shared__ int sel[kWave];
  const int t = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x;
  const size_t qi = ((size_t)seq * p.n_q + t) * p.H + tid;
  float e = -INFINITY;
  if (tid < p.H) {
    if (kind == MISA_ROUTER_GATE) {
      e = W[qi];
    } else {
      float qv[kD];
      load_query_head<QDT>(Q, qi, qv);
      float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
      for (int c = 0; c < kD; c += 4) {
        s0 = fmaf(qv[c], qv[c], s0);
        s1 = fmaf(qv[c + 1], qv[c + 1], s1);
        s2 = fmaf(qv[c + 2], qv[c + 2], s2);
        s3 = fmaf(qv[c + 3], qv[c + 3], s3);
      }
      e = sqrtf((s0 + s1) + (s2 + s3));
    }
    if (E) E[qi] = e;
  }
  if (e == 0.f) e = 0.f;  // -0.0 ties with +0.0
  Es[tid] = e;
  __syncthreads();
  int rank = 0;
  for (int i = 0; i < p.H; ++i) {
    const float o = Es[i];
    rank += (o > e || (o == e && i < tid)) ? 1 : 0;
  }
  sel[tid] = (tid < p.H && rank < p.h) ? 1 : 0;
  __syncthreads();
  if (sel[tid]) {
    int pos = 0;
    for (int i = 0; i < tid; ++i) pos += sel[i];
    heads[((size_t)seq * p.n_q + t) * p.h + pos] = tid;
  }
}

hipError_t launch_route_proxy(const Prob& p, int q_dtype, int kind, const void* Q, const float* W,
                              int* heads, float* E, hipStream_t st) {
  const dim3 grid(p.n_q, p.n_seq);
  if (q_dtype == MISA_F32) route_proxy_kernel<MISA_F32><<<grid, 64, 0, st>>>(p, kind, Q, W, heads, E);
  else if (q_dtype == MISA_BF16) route_proxy_kernel<MISA_BF16><<<grid, 64, 0, st>>>(p, kind, Q, W, heads, E);
  else route_proxy_kernel<MISA_FP8_E4M3><<<grid, 64, 0, st>>>(p, kind, Q, W, heads, E);
  return hipGetLastError();
}

// Row groups (of 64 query-head rows) per workgroup of the tiled kernel.
static int route_row_groups(const Prob& p) {
  const long long groups = ((long long)p.n_q * p.H + 63) / 64;
  return groups >= 4 ? 4 : (groups >= 2 ? 2 : 1);
}

int route_splits(const Prob& p) {
  // Enough workgroups to cover the chip, but at least 4 block tiles (128 blocks) per split.
  const long long wgs = (long long)p.n_seq * (((long long)p.n_q * p.H + 255) / 256);
  long long s = (512 + wgs - 1) / wgs;
  const long long cap = (p.M + 127) / 128;
  if (s > cap) s = cap;
  if (s > 16) s = 16;
  if (s < 1) s = 1;
  return (int)s;
}

// Whether all (query, head) rows of a sequence fit one wavefront.
static bool route_few_rows(const Prob& p) { return (long long)p.n_q * p.H <= 64; }

// 16-block tiles per wavefront and partial sums (workgroups) per query of route_few_kernel: one tile each
// up to the partial sums there is room for, more tiles per wavefront beyond.
static void route_few_shape(const Prob& p, int* tiles_per_wave, int* n_parts) {
  const int groups = (p.M + 63) / 64, most = route_few_rows(p) ? 64 : 4 * route_splits(p);
  *tiles_per_wave = (groups + most - 1) / most;
  *n_parts = (groups + *tiles_per_wave - 1) / *tiles_per_wave;
}

size_t route_ws_bytes(const Prob& p) {
  // partial sums [n_seq, n_q, parts, 64]; the tiled kernel needs room for every column phase
  // (splits * 4), the kernels for few rows for their (at most 64) parts
  size_t parts = (size_t)route_splits(p) * 4;
  if (route_few_rows(p)) parts = std::max<size_t>(parts, 64);
  return (size_t)p.n_seq * p.n_q * parts * kWave * sizeof(float);
}

hipError_t launch_route(const Prob& p, int k_dtype, int q_dtype, const void* Q, const float* W,
                        const float* Kp, const void* K, const float* kscale, int* heads, float* E,
                        void* ws, hipStream_t st) {
  const int splits = route_splits(p);
  float* part = static_cast<float*>(ws);
  int total_splits = splits;
  // A query of route_few_kernel reads all pooled blocks by itself.  Where the rows of a sequence are more than one
  // wavefront's that pays until the workgroups of all queries fill the chip (64 heads, us, tile kernel / this one:
  // 3 queries of 64 x 512 blocks 33 / 30, 4 of them 31 / 35; 4 of 256 x 64 blocks 34 / 30; 7 of 64 x 2048 59 / 113).
  const bool few_queries = p.n_q < 8 && (long long)p.n_seq * p.n_q * ((p.M + 63) / 64) <= 1536;
  if (q_dtype == MISA_BF16 && (route_few_rows(p) || few_queries)) {
    int tpw, parts;
    route_few_shape(p, &tpw, &parts);
    total_splits = parts;
    const bool together = route_few_rows(p);
    const dim3 g1(parts, p.n_seq, together ? 1 : p.n_q);
    const uint16_t* q = static_cast<const uint16_t*>(Q);
    const int rows = together ? p.n_q * p.H : p.H;
    if (rows <= 16) route_few_kernel<1><<<g1, 256, 0, st>>>(p, tpw, parts, q, Kp, part);
    else if (rows <= 32) route_few_kernel<2><<<g1, 256, 0, st>>>(p, tpw, parts, q, Kp, part);
    else route_few_kernel<4><<<g1, 256, 0, st>>>(p, tpw, parts, q, Kp, part);
  } else if (q_dtype == MISA_BF16) {
    const int rg = route_row_groups(p);
    const int rows = p.n_q * p.H, groups = (rows + 64 * rg - 1) / (64 * rg);
    // where CUs are left without a workgroup, down to one tile of 32 blocks per split, as far as there is room for the
    // partial sums (us, 128 blocks / this: 8 queries of 64 x 64 blocks 13.4 / 12.7, 100 of 32 x 512 15.5 / 12.8; not past one
    // workgroup per CU: 700 of 64 x 64 blocks 14.5 / 16.2 in two)
    const long long most = std::min<long long>(std::min((p.M + kRouteKT - 1) / kRouteKT, splits * rg), 256 / ((long long)groups * p.n_seq));
    const int s = std::max<int>(splits, (int)most);
    total_splits = s * (4 / rg);
    const dim3 g1(s, groups, p.n_seq);
    const uint16_t* q = static_cast<const uint16_t*>(Q);
    if (rg == 4) route_tile_kernel<4><<<g1, 256, 0, st>>>(p, s, q, Kp, part);
    else route_tile_kernel<2><<<g1, 256, 0, st>>>(p, s, q, Kp, part);   // (one group: few rows)
  } else {
    // few rows: a block per wavefront while that makes at most 64 partial sums (64 blocks: 6.8 us; 25 us in
    // one workgroup, whose wavefronts then take 16 blocks each one after the other), and no more workgroups
    // than two per CU (256 sequences of 64 blocks: 19 us; 64 us with a workgroup for 4 blocks; one per CU: 64 x 256
    // blocks of 32 heads 19 us instead of 16)
    const long long most = std::min<long long>(std::min(64, (p.M + 3) / 4), 512 / ((long long)p.n_seq * p.n_q));
    while (route_few_rows(p) && 2 * total_splits <= most) total_splits *= 2;
    const dim3 g1(total_splits, p.n_q, p.n_seq);
    route_partial_kernel<MISA_F32><<<g1, 256, 0, st>>>(p, total_splits, Q, Kp, part);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 g2(p.n_q, p.n_seq);
#define FIN(KD, QD) \
  route_finalize_kernel<KD, QD><<<g2, 128, 0, st>>>(p, total_splits, Q, W, K, kscale, part, heads, E)
  if (q_dtype == MISA_F32) {
    if (k_dtype == MISA_F32) FIN(MISA_F32, MISA_F32);
    else if (k_dtype == MISA_BF16) FIN(MISA_BF16, MISA_F32);
    else FIN(MISA_FP8_E4M3, MISA_F32);
  } else {
    if (k_dtype == MISA_F32) FIN(MISA_F32, MISA_BF16);
    else if (k_dtype == MISA_BF16) FIN(MISA_BF16, MISA_BF16);
    else FIN(MISA_FP8_E4M3, MISA_BF16);
  }
#undef FIN
  return hipGetLastError();
}

}  // namespace misa
