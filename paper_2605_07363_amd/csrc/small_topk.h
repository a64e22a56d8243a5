// Exact top-k of one short row (at most 8192 scores) that already sits in LDS, by the 256
// threads of a workgroup: the tail of the fused re-rank kernel (Eq. misa_final_topk), where the
// dense scores of a query's candidates never leave the workgroup that computed them.
//
// Same result as topk_kernel in map mode, bit for bit: -inf (skipped candidates) is never
// selected, the k largest of the rest are, ties go to the lower position, positions come out in
// ascending order and unused output slots hold -1 / -inf.
//
// Method: pick_row, from a sampled bracket; small_row_by_digits for rows that the bracket does not fit.  (Rows below 2048
// scores have no such bracket and do not come here.)
#pragma once

#include "kernels.h"
#include "radix.h"

namespace misa {

constexpr int kSmallTopkThreads = 256;
constexpr int kSmallTopkMax = 8192;                                  // scores per row
constexpr int kSmallTopkEpt = kSmallTopkMax / kSmallTopkThreads;     // 32 per thread
constexpr int kSmallTopkWords = kSmallTopkMax / 32;                  // bitmap words: one per thread
constexpr int kSmallTopkFew = 64;    // brute-force ranking up to here (256 measured 20 us slower on 2048 rows of 8192)

struct SmallTopkLds {
  int hist[kBins];
  uint32_t sel[kSmallTopkWords];
  uint32_t eq[kSmallTopkWords];
  int wpre[kSmallTopkWords];         // selected positions in the bitmap words before a word
  uint2 few[kSmallTopkFew];          // (key, position) of the entries of the threshold bin
  int few_rank[kSmallTopkFew];       // entries of that list that rank before an entry
  int scan[32];
  int thr[4];
  uint32_t red[3 * 4];
  int few_len;
};

// The digits of the keys: thread t owns positions t, t + 256, ... (32 of them) and keeps their keys
// (order-preserving integer images) in registers.  One
// 2047-bin digit, linear in the key over [lo, max] (keys below lo share bin 0 and are counted in
// registers), is counted in LDS; everything above the bin that holds the k-th largest is
// selected, everything below it dropped, and the bin itself is either taken whole, ranked by
// brute force (at most 64 entries), or refined by the next pass over its own key range.  lo
// starts four binades below the row maximum, which is where the k-th largest of a few thousand
// scores normally lies; after two passes that ended in the catch-all bin lo is the row minimum,
// and from there the range shrinks 2048-fold per pass until all live keys are equal (ties: the
// lowest positions win, by a bitmap walk).  The loops over a thread's elements are free of
// branches, so that their LDS reads and atomics are issued back to back.
//
// sc[0 .. n): the bit patterns of the row's scores in LDS (complete: the caller has passed a
// barrier); n <= 8192.
// map[0 .. n): global; out_idx[j] = map[position] for the selected positions in ascending order.
// All 256 threads call this; it contains barriers.
__device__ __forceinline__ void small_row_by_digits(const int* sc, int n, int k, const int* __restrict__ map,
                                               int* __restrict__ out_idx, float* __restrict__ out_val,
                                               SmallTopkLds& L) {
  constexpr int NT = kSmallTopkThreads, EPT = kSmallTopkEpt;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  uint32_t key[EPT];
  uint32_t act = 0;        // bit u: element tid + NT u can still be selected and is undecided
  uint32_t kmax = 0, kmin = 0xFFFFFFFFu;
#pragma unroll
  for (int u = 0; u < EPT; ++u) key[u] = order_key(__int_as_float(sc[min(tid + NT * u, n - 1)]));
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const bool ok = tid + NT * u < n && key[u] > kKeyNegInf;
    act |= ok ? 1u << u : 0u;
    kmax = max(kmax, ok ? key[u] : 0u);
    kmin = min(kmin, ok ? key[u] : 0xFFFFFFFFu);
  }
  int selectable = __popc(act);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    selectable += __shfl_xor(selectable, off);
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off));
  }
  if (lane == 0) { L.red[wave] = (uint32_t)selectable; L.red[4 + wave] = kmax; L.red[8 + wave] = kmin; }
  if (tid == 0) L.few_len = 0;
  if (tid < kSmallTopkFew) {
    L.few[tid] = make_uint2(0u, 0u);   // padding of the brute-force list: key 0 ranks below every live key
    L.few_rank[tid] = 0;
  }
  __syncthreads();
  selectable = (int)(L.red[0] + L.red[1] + L.red[2] + L.red[3]);
  kmax = max(max(L.red[4], L.red[5]), max(L.red[6], L.red[7]));
  kmin = min(min(L.red[8], L.red[9]), min(L.red[10], L.red[11]));

  const int k_eff = min(k, selectable);
  for (int i = k_eff + tid; i < k; i += NT) {
    out_idx[i] = -1;
    if (out_val) out_val[i] = -INFINITY;
  }
  if (k_eff == 0) return;

  enum { kDone, kBrute, kTies };
  int mode = kDone;
  int need = k_eff, nb = selectable;   // nb: live elements
  uint32_t chosen = 0;
  if (k_eff == selectable) {
    chosen = act;
  } else {
    for (int pass = 0;; ++pass) {      // every quantity that steers the loop is uniform over the block
      if (nb <= kSmallTopkFew) { mode = kBrute; break; }
      if (kmax == kmin) { mode = kTies; break; }               // all live keys are equal
      const uint32_t lo = (pass < 2 && kmax - kmin > (1u << 25)) ? kmax - (1u << 25) : kmin;
      const uint32_t span = kmax - lo;
      int shift = max(0, 32 - __clz((int)span) - 11);
      if ((span >> shift) > (uint32_t)(kBins - 2)) ++shift;      // bins 1 .. 2047 cover [lo, kmax]
      zero_hist_n<NT>(L.hist);
      int below = 0;                   // live elements under lo: counted in registers, not by LDS atomics
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        const bool live = (act >> u) & 1u;
        const bool in = live && key[u] >= lo;
        below += (int)live - (int)in;
        if (in) atomicAdd(&L.hist[(int)((key[u] - lo) >> shift) + 1], 1);
      }
      below = wave_inclusive_scan(below);
      if (lane == 63 && below) atomicAdd(&L.hist[0], below);
      __syncthreads();
      find_threshold_bin_n<NT>(L.hist, need, L.scan, L.thr);
      const int b = L.thr[0];
      need = L.thr[1];
      nb = L.thr[2];
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        const int d = key[u] < lo ? 0 : (int)((key[u] - lo) >> shift) + 1;
        const uint32_t bit = act & (1u << u);
        chosen |= d > b ? bit : 0u;
        act &= d == b ? ~0u : ~bit;
      }
      if (nb == need) { chosen |= act; break; }
      if (b > 0) {
        kmin = lo + ((uint32_t)(b - 1) << shift);
        kmax = min(kmax, kmin + ((1u << shift) - 1u));
      } else {
        kmax = lo - 1u;                                         // (lo > kmin here: bin 0 was not empty)
      }
      __syncthreads();                                          // thr is rewritten by the next pass
    }
  }

  // ---- the selected positions as a bitmap: element tid + NT u is bit (tid & 31) of word 2 wave + 8 u (+ 1)
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const unsigned long long m = __ballot((chosen >> u) & 1u);
    if (lane == 0) {
      L.sel[2 * wave + 8 * u] = (uint32_t)m;
      L.sel[2 * wave + 8 * u + 1] = (uint32_t)(m >> 32);
    }
    if (mode == kTies) {
      const unsigned long long e = __ballot((act >> u) & 1u);
      if (lane == 0) {
        L.eq[2 * wave + 8 * u] = (uint32_t)e;
        L.eq[2 * wave + 8 * u + 1] = (uint32_t)(e >> 32);
      }
    }
  }
  if (mode == kBrute) {
    // the (at most 64) live entries, listed by the few threads that own one
    for (uint32_t a = act; a; a &= a - 1) {
      const int i = tid + NT * (__ffs(a) - 1);
      const int slot = atomicAdd(&L.few_len, 1);
      if (slot < kSmallTopkFew) L.few[slot] = make_uint2(order_key(__int_as_float(sc[i])), (uint32_t)i);
    }
  }
  __syncthreads();
  if (mode == kBrute) {
    // the nb entries of the threshold bin, ranked by score, then position: all pairs, thread t
    // comparing entry t % 64 with a quarter of the list (padded with entries that rank below all)
    {
      constexpr int JP = kSmallTopkFew / (NT / 64);
      const int i = tid & 63, j0 = (tid >> 6) * JP;
      const uint2 mine = L.few[i];
      int part = 0;
#pragma unroll
      for (int j = j0; j < j0 + JP; ++j) {
        const uint2 o = L.few[j];
        part += (o.x > mine.x || (o.x == mine.x && o.y < mine.y)) ? 1 : 0;
      }
      if (part) atomicAdd(&L.few_rank[i], part);
    }
    __syncthreads();
    if (tid < nb && L.few_rank[tid] < need) {
      const uint32_t e = L.few[tid].y;
      atomicOr(&L.sel[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
  } else if (mode == kTies) {
    // more equal scores than places: the `need` lowest positions among them
    const uint32_t bits0 = L.eq[tid];
    int total;
    int before = block_exclusive_scan(__popc(bits0), L.scan, &total);
    uint32_t bits = bits0, kept = 0;
    while (bits && before < need) {
      const uint32_t low = bits & (0u - bits);
      kept |= low;
      bits ^= low;
      ++before;
    }
    L.sel[tid] |= kept;          // a word is owned by one thread here
    __syncthreads();
  }

  // ---- output in position order: slot of a selected position = selected positions before it
  //      = those of the bitmap words before its word (prefix sums, one word per thread) + the lower
  //      bits of its word.  Every thread goes back to its own positions t, t + 256, ..., so that the
  //      map entries are read coalesced and all at once.
  int mapped[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) mapped[u] = map[min(tid + NT * u, n - 1)];
  {
    int total;
    const int before = block_exclusive_scan(__popc(L.sel[tid]), L.scan, &total);
    L.wpre[tid] = before;
  }
  __syncthreads();
  const uint32_t below = (1u << (tid & 31)) - 1u;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int w = (tid >> 5) + 8 * u;
    const uint32_t word = L.sel[w];
    const int pos = L.wpre[w] + __popc(word & below);
    if (((word >> (tid & 31)) & 1u) && pos < k) {   // pos < k: always true when the selection is consistent
      out_idx[pos] = mapped[u];
      if (out_val) out_val[pos] = __int_as_float(sc[tid + NT * u]);
    }
  }
}

// The usual row: 1024 of its scores bracket the k-th largest, one walk over the row marks what lies above the
// bracket and lists what lies inside, and a histogram of the list finds the bin of the k-th, whose few entries are
// ranked directly.  The counts prove the bracket right or wrong, so the result does not depend on the sample; false
// (for all threads; nothing written) where it is wrong, the list does not fit, or a NaN is seen: small_row_by_digits then.
// Workgroups reach the end of their rows together, so this is not hidden behind the matrix work of others: a chain of
// barriers, the map's loads (requested first) and about 30 vector instructions per score and thread (86 with every
// score's key in registers).  2048 rows of 8192, beside the kernel's scores: 22 - 33 us against 50 - 70 us.
constexpr int kPickBins = 1024;
constexpr int kPickSamples = 1024;
constexpr int kPickSeg = 640;        // list entries of a wavefront, behind them 64 of slack
static_assert(kRerankFusedMinList >= 2 * kPickSamples, "shorter lists are left to the two kernels");

struct PickLds {
  int hist[kPickBins];
  uint16_t list[4][kPickSeg + 64];   // positions inside the bracket
  alignas(8) uint32_t sel[kSmallTopkWords];   // bitmap of the selected positions
  int wpre[kSmallTopkWords];
  uint2 few[kSmallTopkFew];          // (key, position) of the entries of the k-th largest's bin
  int few_rank[kSmallTopkFew];
  int scan[32];
  int at_lo[3], at_hi[3];            // of the sample: bin, rank inside it, its count
  float red[8];
  int sure[4], listed[4];
  int few_len, nan_seen;
};

// The bin that holds the r-th (and r2-th) largest of the histogram's entries, the rank inside it and its count.
__device__ __forceinline__ void pick_bin(const int* hist, int* scan, int r, int* out, int r2, int* out2) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int top = kPickBins - 1 - 4 * tid;
  const int4 v = *reinterpret_cast<const int4*>(&hist[top - 3]);
  const int h[4] = {v.w, v.z, v.y, v.x};
  const int sum = (h[0] + h[1]) + (h[2] + h[3]);
  const int inc = wave_inclusive_scan(sum);
  if (lane == 63) scan[wave] = inc;
  __syncthreads();
  int total;
  int above = waves_before(scan, 4, &total) + inc - sum;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (above < r && r <= above + h[i]) { out[0] = top - i; out[1] = r - above; out[2] = h[i]; }
    if (above < r2 && r2 <= above + h[i]) { out2[0] = top - i; out2[1] = r2 - above; out2[2] = h[i]; }
    above += h[i];
  }
  __syncthreads();
}

__device__ __forceinline__ bool pick_row(int* sc, int n, int k, const int* __restrict__ map,
                                         int* __restrict__ out_idx, float* __restrict__ out_val, PickLds& L) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float kf = (float)k * (float)kPickSamples / (float)n, margin = 4.f * sqrtf(kf) + 8.f;
  const int r_lo = (int)ceilf(kf + margin), r_hi = (int)floorf(kf - margin);
  if (r_lo > kPickSamples) return false;
  const float* scf = reinterpret_cast<const float*>(sc);
  int mapped[kSmallTopkEpt];           // requested here, used at the end (in four rounds there: 8 us of a row's 14)
#pragma unroll
  for (int u = 0; u < kSmallTopkEpt; ++u) mapped[u] = map[min(256 * u + tid, n - 1)];

  // ---- sample: one score of every n / 1024, at a hashed place among them
  float smp[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = tid + 256 * i, from = (j * n) >> 10, to = ((j + 1) * n) >> 10;
    smp[i] = scf[from + (int)((((uint32_t)j * 2654435761u >> 16) * (uint32_t)(to - from)) >> 16)];
  }
  float lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (fabsf(smp[i]) < 1e30f) { lo = fminf(lo, smp[i]); hi = fmaxf(hi, smp[i]); }
  lo = -wave_max_f32(-lo);
  hi = wave_max_f32(hi);
  if (lane == 0) { L.red[wave] = lo; L.red[4 + wave] = hi; }
  reinterpret_cast<int4*>(L.hist)[tid] = make_int4(0, 0, 0, 0);
  L.sel[tid] = 0;
  if (tid < kSmallTopkFew) {
    L.few[tid] = make_uint2(0u, 0u);
    L.few_rank[tid] = 0;
  }
  if (tid == 0) { L.few_len = 0; L.nan_seen = 0; L.at_lo[2] = 0; L.at_hi[2] = 0; }
  if ((n & 255) && tid >= (n & 255)) sc[(n & ~255) + tid] = (int)0xFF800000u;   // the walk takes 256 at a time
  __syncthreads();
  lo = fminf(fminf(L.red[0], L.red[1]), fminf(L.red[2], L.red[3]));
  hi = fmaxf(fmaxf(L.red[4], L.red[5]), fmaxf(L.red[6], L.red[7]));
  const float width = (hi - lo) * (1.f / kPickBins), per = (float)kPickBins / (hi - lo);
  if (!(width > 0.f) || !(per < 3e38f)) return false;
  auto bin_of = [](float x, float from, float scale) {
    return (int)__builtin_amdgcn_fmed3f((x - from) * scale, 0.f, (float)(kPickBins - 1));
  };
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (smp[i] >= lo) atomicAdd(&L.hist[bin_of(smp[i], lo, per)], 1);
  __syncthreads();
  pick_bin(L.hist, L.scan, r_lo, L.at_lo, max(r_hi, 1), L.at_hi);
  if (L.at_lo[2] == 0) return false;
  // the bracket's ends, rounded outwards: of a bin 1024 x 2^-22, and what the values have lost by their size
  const float slack = 0.001f * width + 2.5e-7f * fmaxf(fabsf(lo), fabsf(hi));
  const float b_lo = fmaxf(lo + (float)L.at_lo[0] * width - slack, -3.402823466e38f);
  const float edge = lo + (float)(L.at_hi[0] + 1) * width + slack;
  const float b_hi = r_hi >= 1 && L.at_hi[0] < kPickBins - 1 ? edge : INFINITY;
  reinterpret_cast<int4*>(L.hist)[tid] = make_int4(0, 0, 0, 0);

  // ---- walk: the wavefront takes positions 256 u + 64 wave .. + 63
  const int slabs = (n + 255) >> 8;
  int sure = 0, fill = 0;
#pragma unroll 8
  for (int u = 0; u < slabs; ++u) {
    const float x = scf[256 * u + tid];
    const unsigned long long above = __builtin_amdgcn_ballot_w64(x >= b_hi);
    const unsigned long long in = __builtin_amdgcn_ballot_w64(!(x < b_lo)) & ~above;    // (and NaN)
    if (lane == 0) *reinterpret_cast<uint2*>(&L.sel[8 * u + 2 * wave]) = make_uint2((uint32_t)above, (uint32_t)(above >> 32));
    sure += __popcll(above);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0));
    if (__builtin_amdgcn_inverse_ballot_w64(in)) L.list[wave][min(fill, kPickSeg) + at] = (uint16_t)(256 * u + tid);
    fill += __popcll(in);
  }
  if (lane == 0) { L.sure[wave] = sure; L.listed[wave] = fill; }
  __syncthreads();
  sure = (L.sure[0] + L.sure[1]) + (L.sure[2] + L.sure[3]);
  const int listed = (L.listed[0] + L.listed[1]) + (L.listed[2] + L.listed[3]);
  const int most = max(max(L.listed[0], L.listed[1]), max(L.listed[2], L.listed[3]));
  if (sure > k || sure + listed < k || most > kPickSeg) return false;

  // ---- the listed ones: a wavefront looks at those that it has listed (also where none of them is wanted: a NaN ranks by its
  // sign, above or below all others)
  int need = k - sure;
  const float fine = fminf(fmaxf((float)kPickBins / (edge - b_lo), 1e-35f), 3e38f);
  bool nan = false;
  for (int j = lane; j < fill; j += 64) {
    const float x = scf[L.list[wave][j]];
    nan |= x != x;
    atomicAdd(&L.hist[bin_of(x, b_lo, fine)], 1);
  }
  if (nan) L.nan_seen = 1;
  __syncthreads();
  if (L.nan_seen) return false;
  if (need > 0) {
    pick_bin(L.hist, L.scan, need, L.at_lo, need, L.at_hi);
    const int b = L.at_lo[0], few = L.at_lo[2];
    need = L.at_lo[1];
    if (few > kSmallTopkFew) return false;
    for (int j = lane; j < fill; j += 64) {
      const int e = L.list[wave][j];
      const float x = scf[e];
      const int d = bin_of(x, b_lo, fine);
      if (d > b) atomicOr(&L.sel[e >> 5], 1u << (e & 31));
      if (d == b) L.few[atomicAdd(&L.few_len, 1)] = make_uint2(order_key(x), (uint32_t)e);
    }
    __syncthreads();
    {
      // ranked by score, then position: all pairs, thread t comparing entry t % 64 with a quarter of the list (padded
      // with entries that rank below all)
      constexpr int JP = kSmallTopkFew / 4;
      const uint2 mine = L.few[lane];
      int part = 0;
#pragma unroll
      for (int j = wave * JP; j < wave * JP + JP; ++j) {
        const uint2 o = L.few[j];
        part += (o.x > mine.x || (o.x == mine.x && o.y < mine.y)) ? 1 : 0;
      }
      if (part) atomicAdd(&L.few_rank[lane], part);
    }
    __syncthreads();
    if (tid < few && L.few_rank[tid] < need) {
      const uint32_t e = L.few[tid].y;
      atomicOr(&L.sel[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
  }

  // ---- output in position order
  {
    int total;
    L.wpre[tid] = block_exclusive_scan(__popc(L.sel[tid]), L.scan, &total);
  }
  __syncthreads();
  const int my_word = 8 * (lane >> 1) + 2 * wave + (lane & 1);   // lane 2 u + h: word h of the wavefront's positions of u
  const uint32_t word = L.sel[my_word];
  const int before = L.wpre[my_word];
#pragma unroll
  for (int u = 0; u < kSmallTopkEpt; ++u) {
    if (u >= slabs) break;
    const uint32_t m_lo = __builtin_amdgcn_readlane(word, 2 * u), m_hi = __builtin_amdgcn_readlane(word, 2 * u + 1);
    const int pos = __builtin_amdgcn_mbcnt_hi(m_hi, __builtin_amdgcn_mbcnt_lo(m_lo, (uint32_t)__builtin_amdgcn_readlane(before, 2 * u)));
    if (__builtin_amdgcn_inverse_ballot_w64((unsigned long long)m_hi << 32 | m_lo) && pos < k) {   // pos < k: always true when the selection is consistent
      out_idx[pos] = mapped[u];
      if (out_val) out_val[pos] = scf[256 * u + tid];
    }
  }
  return true;
}

// The row's top-k (see the head of this file).  sc[n .. n rounded up to 256) is scratch.
union SmallRowLds {
  PickLds pick;
  SmallTopkLds digits;
};
__device__ __forceinline__ void small_row_topk(int* sc, int n, int k, const int* __restrict__ map,
                                               int* __restrict__ out_idx, float* __restrict__ out_val, SmallRowLds& L) {
  if (pick_row(sc, n, k, map, out_idx, out_val, L.pick)) return;
  __syncthreads();
  small_row_by_digits(sc, n, k, map, out_idx, out_val, L.digits);
}

}  // namespace misa
