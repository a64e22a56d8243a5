// Stages 3 + 4 in one call for many-query (prefill) problems: the indices of the
// k best-scoring visible keys of every query (Eq. misa_score followed by Eq.
// misa_topk; with all heads Eq. dsa_score / Eq. dsa_topk) without writing the
// [rows, L] score matrix to memory and reading it back.
//
//   1. sample    The tile scoring kernel scores one key of every group of 16
//                (1/16 of the work) into a small matrix.
//   2. threshold Per row, the r-th largest sampled score tau is found (radix
//                select, rounded down).  r is a little above k/16, so that with
//                overwhelming probability at least k of all scores reach tau
//                while only about 16 r do.  Rows with few visible keys get
//                tau = -inf (everything is a candidate).
//   3. filter    The tile scoring kernel runs over all keys and writes the
//                (key, score) pairs with score >= tau to per-row lists.  A row's
//                list is cut into one segment per key range of that launch,
//                sized in step 2 from the range's own sampled scores, so every
//                segment has exactly one writer and needs no atomics.  Segments
//                are filled in ascending key order: step 4 takes an entry's place
//                in the list for its rank by index.
//   4. select    Per row, the exact top-k of the list (ties: lower index) is
//                written in ascending index order: from a bracket that a sample
//                of the entries gives and the counts prove (select_sampled), or,
//                where the list or k is short or the bracket wrong, from
//                the digits of the keys.  Since every score >= tau is in the
//                list, the result equals the top-k of the full row whenever the
//                list holds at least k entries and did not overflow.
//   5. repair    Rows for which that does not hold are flagged; the plain path
//                (dense scores of their query tiles, then the row top-k) runs
//                for them only.  Without flagged rows these two launches exit
//                at once.  The result is therefore always exact; the sampling
//                only decides how much work it takes.
//
// Everything is stream-ordered device work: no host read-back, so the call can
// be captured in a HIP graph.
#include <algorithm>
#include <cmath>

#include "kernels.h"
#include "radix.h"

namespace misa {

constexpr int kFusedMaxK = 8192;          // the candidate list of a row is held in registers
constexpr int kFusedMinL = 4096;

// Rank of the sampled threshold: mean k/16 sampled scores lie among the top k; the
// margin covers the sampling noise of that count (more than five standard deviations).
static int sample_rank(int k) {
  const double mu = (double)k / kSampleStride;
  return (int)std::ceil(mu + 6.0 * std::sqrt(mu) + 8.0);
}

// Length of the list segment of a key range in which c sampled scores reached the threshold.
// Exactly one key of every group of 16 is sampled, so with n keys of the range at or above
// the threshold the count of sampled ones has mean n / 16 and variance below n / 16; the
// segment holds 16 c plus six standard deviations of 16 (c - n / 16) at n = 16 (c + 1), plus
// room for a range none of whose ~200 hits was sampled (probability (15/16)^200 < 3e-6) and
// for the unsampled tail group.  Device and host use the same integer formula.
__host__ __device__ inline int segment_length(int c) {
  int root = 0;                                     // ceil(sqrt(c + 1))
  while (root * root < c + 1) ++root;
  return kSampleStride * c + 6 * kSampleStride * root + 128;
}

// At most this many sampled scores may reach the threshold of a row (r do by construction,
// more only through ties at the threshold value); rows with more are left to the repair pass.
static int max_sample_hits(int k) { return sample_rank(k) + sample_rank(k) / 4 + 16; }

// List capacity of a row: the segment lengths add up to at most this (the square roots are
// largest when the sampled hits are spread evenly over the ranges), in units of 256.
static int list_capacity(int k, int ranges) {
  const int hits = max_sample_hits(k);
  const int per = (hits + ranges - 1) / ranges;
  long long c = 0;
  for (int r = 0; r < ranges; ++r) c += segment_length(per) + 6 * kSampleStride;   // (+ one more root: the roots are rounded up)
  return (int)((c + 255) / 256 * 256);
}

// Room for entries that the row selection has to have: a row's entries have mean 16 r and variance 240 r (r hits among
// samples of one key in 16), of which 5.5 standard deviations are covered, as sample_rank does at the other end; and the
// last chunk of every key range may hold a single entry.  (Chunks of 64 instead, a wavefront-wide load each,
// lose up to 63 per range, and do where most ranges hold a few entries: 4 of 232 rows of k = 942 in 63 ranges needed more
// than 5120 places for 2000 entries.)
constexpr int kChunk = 16;                // entries of one key range that 16 lanes take together (128 bytes of the list)
static int row_room(int k, int ranges) {
  const double r = sample_rank(k);
  return (int)std::ceil(kSampleStride * r + 5.5 * std::sqrt(240.0 * r)) + (kChunk - 1) * ranges;
}

static size_t select_lds_bytes(const Prob& p) {
  const size_t nwords = ((size_t)p.L + 31) / 32;
  return nwords * 8;  // selection bitmap and per-word prefix counts
}

// With one or two active heads a quarter or half of all keys score exactly 0 (every active head
// negative); the k-th largest then often lies on that plateau of ties, whose rows the threshold
// filter has to hand to the repair pass, and the two calls are faster (measured with h = 2 on the
// 131072-key prefill: 1.89 ms against 0.97 ms).
static bool fused(const Prob& p, int k_dtype, int q_dtype, int k) {
  return tile_path(p, k_dtype, q_dtype) && k <= kFusedMaxK && p.L >= kFusedMinL && p.h > 2;
}

__device__ __forceinline__ float key_to_float(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// ---------------------------------------------------------------- threshold
// One workgroup of 256 threads per row: tau[row] = a value at or just below the r-th largest of
// the row's visible sampled scores (the lower edge of its 22-bit radix bin, i.e. within 2^-13
// relative), so at least r samples reach it.  upper[row]: the top key of the first radix digit
// that holds the sampled score of rank r / 4, a robust upper end of the interval in which the
// k-th largest score lies (select_rows_kernel spreads its first digit over [tau, upper]).  The
// first 16 samples of every thread (4096 per row) stay in registers for both digit passes, all
// their loads in flight together; longer rows read the rest again in the second pass.  Also
// clears the row's repair flags and lays out the row's candidate list: seg[row][r] is the offset
// of the segment of key range r (seg[row][ranges] the total), its length segment_length(samples
// of the range that reach tau), cut to the visible keys of the range.  A row whose sampled hits
// exceed max_hits (ties at the threshold value) gets empty segments and so falls to the repair
// pass.  A row all of whose visible keys fit the list keeps every key (tau = -inf, segments =
// the visible keys of each range).
constexpr int kThrThreads = 256;
constexpr int kThrHeld = 16;
__global__ __launch_bounds__(kThrThreads) void select_threshold_kernel(
    Prob p, const float* __restrict__ Ss, int m, int r, int cap, int keep_all, int qwg, int q_tiles, int ranges,
    int keys_per_range, int max_hits, float* __restrict__ tau, uint32_t* __restrict__ upper,
    int* __restrict__ seg, int* __restrict__ row_flag, int* __restrict__ tile_flag) {
  __shared__ int hist[kBins];
  __shared__ int range_hits[64];
  __shared__ int hist2[kBins];
  __shared__ int scan_scratch[32];
  __shared__ int thr[3];
  __shared__ int thr_up[3];
  const int tid = threadIdx.x;
  const int row = blockIdx.x;
  const int seq = row / p.n_q, t = row % p.n_q;
  const int n = visible(p, seq, t);
  if (tid == 0) {
    row_flag[row] = 0;
    if (t % qwg == 0) tile_flag[seq * q_tiles + t / qwg] = 0;
  }
  int* row_seg = seg + (size_t)row * (ranges + 1);
  if (n <= keep_all) {  // every visible key fits into the list (and into the registers of the row
                        // selection): a range's segment holds its visible keys
    if (tid == 0) { tau[row] = -INFINITY; upper[row] = 0xFFFFFFFFu; }
    if (tid <= ranges) row_seg[tid] = (int)min((long long)n, (long long)tid * keys_per_range);
    return;
  }
  const int ns = n / kSampleStride;  // visible samples; ns > keep_all / 16 >= r
  const float* s = Ss + (size_t)row * m;
  float held[kThrHeld];
#pragma unroll
  for (int u = 0; u < kThrHeld; ++u) {
    const int i = u * kThrThreads + tid;
    held[u] = i < ns ? s[i] : 0.f;
  }
  for (int i = tid; i < kBins; i += kThrThreads) { hist[i] = 0; hist2[i] = 0; }
  __syncthreads();
  auto scan = [&](auto f) {
#pragma unroll
    for (int u = 0; u < kThrHeld; ++u)
      if (u * kThrThreads + tid < ns) f(order_key(held[u]));
    for (int base = kThrHeld * kThrThreads; base < ns; base += 8 * kThrThreads) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = base + u * kThrThreads + tid;
        v[u] = i < ns ? s[i] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (base + u * kThrThreads + tid < ns) f(order_key(v[u]));
    }
  };
  scan([&](uint32_t key) { atomicAdd(&hist[key >> 21], 1); });
  __syncthreads();
  find_threshold_bin_n<kThrThreads>(hist, r, scan_scratch, thr, max(r / 4, 1), thr_up);
  const uint32_t d1 = (uint32_t)thr[0];
  const int need = thr[1];
  scan([&](uint32_t key) {
    if ((key >> 21) == d1) atomicAdd(&hist2[(key >> 10) & 0x7FF], 1);
  });
  __syncthreads();
  find_threshold_bin_n<kThrThreads>(hist2, need, scan_scratch, thr);
  const float tau_row = key_to_float((d1 << 21) | ((uint32_t)thr[0] << 10));
  if (tid == 0) {
    tau[row] = tau_row;
    upper[row] = ((uint32_t)thr_up[0] << 21) | 0x1FFFFFu;
  }
  // sampled scores of every key range that reach the threshold (sample i stands for the keys
  // 16 i .. 16 i + 15, and a range is a whole number of such groups)
  if (tid < 64) range_hits[tid] = 0;
  __syncthreads();
  const int groups_per_range = keys_per_range / kSampleStride;
  auto tally = [&](float v, int i) {
    if (v >= tau_row) atomicAdd(&range_hits[i / groups_per_range], 1);
  };
#pragma unroll
  for (int u = 0; u < kThrHeld; ++u)
    if (u * kThrThreads + tid < ns) tally(held[u], u * kThrThreads + tid);
  for (int i = kThrHeld * kThrThreads + tid; i < ns; i += kThrThreads) tally(s[i], i);
  __syncthreads();
  if (tid < 64) {  // one wavefront: segment lengths, their prefix sums
    const int hits = tid < ranges ? range_hits[tid] : 0;
    int total_hits = hits;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) total_hits += __shfl_xor(total_hits, o);
    const long long first_key = (long long)tid * keys_per_range;
    const int visible_here = (int)max(0ll, min((long long)n - first_key, (long long)keys_per_range));
    int len = tid < ranges ? min(segment_length(hits), visible_here) : 0;
    if (total_hits > max_hits) len = 0;          // ties at the threshold: the repair pass takes the row
    int end = wave_inclusive_scan(len);
    if (__shfl(end, 63) > cap) { len = 0; end = 0; }   // cannot happen below max_hits; never lay out past the list
    if (tid < ranges) row_seg[tid] = end - len;
    if (tid == ranges - 1) row_seg[ranges] = end;
  }
}

// ---------------------------------------------------------------- select
// The passes over a thread's entries are unrolled in three parts, and a row takes those that its chunks reach into (a
// branch per entry would keep the loads and LDS accesses of a pass from being issued together; us, one part / these: 4096
// rows of 5760 entries 130 / 114, 4000 of 670 40.5 / 35.8).
template <int NT>
constexpr int kPart1 = NT == 512 ? 3 : 5;
template <int NT>
constexpr int kPart2 = NT == 512 ? 6 : 8;
template <int NT, int EPT, class F>
__device__ __forceinline__ void for_entries(int slabs, F f) {
#pragma unroll
  for (int u = 0; u < kPart1<NT>; ++u) f(u);
  if (slabs > kPart1<NT>) {
#pragma unroll
    for (int u = kPart1<NT>; u < kPart2<NT>; ++u) f(u);
    if (slabs > kPart2<NT>) {
#pragma unroll
      for (int u = kPart2<NT>; u < EPT; ++u) f(u);
    }
  }
}

// The usual row: one entry per thread brackets the k-th largest between two thresholds, a walk over the registers marks what lies above
// the bracket and lists what lies inside, a histogram of the list finds the bin of the k-th, whose few entries are ranked
// directly.  The entries are in index order, so the output place of one is the number of selected ones
// before it, from the ballots.  The counts prove the bracket right or wrong; false (for all threads; nothing
// written) where it is wrong or does not fit.
// For shorter lists the chain of barriers of the digits is shorter (us, sampled / digits: 250 rows of 320 entries
// 18.9 / 12.2, 1000 of 980 19.1 / 13.8, of 1630 17.4 / 14.3, of 1920 18.7 / 18.9, of 3260 20.7 / 22.2), and rows that are listed
// whole, whose digits are coarse, have few entries in that of a small k (8817 rows of 4691: k = 20 116 / 93, k = 300 119 / 125).
constexpr int kSampledMin = 2048, kSampledMinK = 128;
constexpr int kRowSeg = 288;        // list entries of a wavefront, behind them 64 of slack
template <int NT, int EPT>
struct EntryLds {
  uint2 word[EPT * (NT / 64)];      // selected entries: word u NW + wave holds u NT + 64 wave ..
  int before[EPT * (NT / 64)];      // selected entries of the words before a word
  uint2 few[64];                    // (key, entry)
  int few_rank[64];
  int sure[16], listed[16], valid[16];
  int at_lo[3], at_hi[3];
  float low[16], high[16];
  int few_len, unlike;
  uint32_t same;
};
template <int NT>
constexpr size_t row_list_bytes() { return (size_t)(NT / 64) * (kRowSeg + 64) * 8; }

template <int NT, int EPT>
__device__ __forceinline__ bool select_sampled(const int (&ei)[EPT], const float (&ev)[EPT], int c, int slabs, int k, float tau, float top,
                                               int* hist, int* scan_scratch, uint32_t* dyn, EntryLds<NT, EPT>& L,
                                               int* __restrict__ out_idx, float* __restrict__ out_val) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint2* const list = reinterpret_cast<uint2*>(dyn) + wave * (kRowSeg + 64);
  auto bin_of = [](float v, float from, float scale) {
    return (int)__builtin_amdgcn_fmed3f((v - from) * scale, 0.f, (float)(kBins - 1));
  };

  // ---- sample: one entry of every thread (hist is cleared, a barrier passed)
  float width;
  {
    const int us = (int)((((uint32_t)tid * 2654435761u >> 16) * (uint32_t)slabs) >> 16);
    uint32_t bits = 0;          // (a chain of selects would become an indexed load, and the entries scratch memory)
    bool valid = false;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      bits |= us == u ? __float_as_uint(ev[u]) : 0u;
      valid |= us == u && ei[u] >= 0;
    }
    const float smp = __uint_as_float(bits);
    if (!(fabsf(tau) < 1e30f) || !(fabsf(top) < 1e30f)) {   // (the list is the whole row: the sample's own range)
      const bool finite = valid && fabsf(smp) < 1e30f;
      const float low = -wave_max_f32(finite ? -smp : -INFINITY), high = wave_max_f32(finite ? smp : -INFINITY);
      if (lane == 0) { L.low[wave] = low; L.high[wave] = high; }
      __syncthreads();
      tau = -wave_max_f32(-L.low[lane & (NW - 1)]);
      top = wave_max_f32(L.high[lane & (NW - 1)]);
    }
    width = (top - tau) * (1.f / kBins);
    const float per = (float)kBins / (top - tau);
    if (!(width > 0.f) || !(per < 3e38f)) return false;
    if (valid && smp >= tau) atomicAdd(&hist[bin_of(smp, tau, per)], 1);
    const int n_valid = __popcll(__builtin_amdgcn_ballot_w64(valid));
    if (lane == 0) L.valid[wave] = n_valid;
  }
  if (tid < 64) {
    L.few[tid] = make_uint2(0u, 0u);      // (key 0 ranks below every entry)
    L.few_rank[tid] = 0;
  }
  if (tid == 0) { L.few_len = 0; L.at_lo[2] = 0; L.at_hi[2] = 0; L.unlike = 0; }
  __syncthreads();
  int m;
  waves_before(L.valid, NW, &m);
  const float part = (float)k / (float)c, kf = part * (float)m, margin = 5.f * sqrtf(kf * (1.f - part)) + 8.f;
  const int r_lo = min((int)ceilf(kf + margin), m), r_hi = (int)floorf(kf - margin);
  find_threshold_bin_n<NT>(hist, r_lo, scan_scratch, L.at_lo, max(r_hi, 1), L.at_hi);
  if (L.at_lo[2] == 0) return false;
  // the bracket's ends, rounded outwards: of the bins 2048 x 2^-22 of one, and what the values have lost by their size
  const float slack = 0.001f * width + 2.5e-7f * fmaxf(fabsf(tau), fabsf(top));
  const float from = kf + margin > (float)m ? tau : tau + (float)L.at_lo[0] * width - slack;   // (no lower end in the sample: all)
  const float edge = tau + (float)(L.at_hi[0] + 1) * width + slack;
  const float upto = r_hi >= 1 && L.at_hi[0] < kBins - 1 ? edge : INFINITY;
  const float fine = fminf((float)kBins / (edge - from), 3e38f);

  for (int i = tid; i < kBins; i += NT) hist[i] = 0;

  // ---- walk
  int sure = 0, fill = 0;
  for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
    const bool live = ei[u] >= 0;
    const unsigned long long above = __builtin_amdgcn_ballot_w64(live && ev[u] >= upto);
    const unsigned long long in = __builtin_amdgcn_ballot_w64(live && ev[u] >= from) & ~above;
    if (lane == 0) L.word[u * NW + wave] = make_uint2((uint32_t)above, (uint32_t)(above >> 32));
    sure += __popcll(above);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0));
    if (__builtin_amdgcn_inverse_ballot_w64(in)) list[min(fill, kRowSeg) + at] = make_uint2(__float_as_uint(ev[u]), (uint32_t)(u * NT + tid));
    fill += __popcll(in);
  });
  if (lane >= slabs && lane < EPT) L.word[lane * NW + wave] = make_uint2(0u, 0u);   // (parts left out)
  __syncthreads();     // (the histogram is clear)
  for (int j = lane; j < min(fill, kRowSeg); j += 64) atomicAdd(&hist[bin_of(__uint_as_float(list[j].x), from, fine)], 1);
  if (lane == 0) { L.sure[wave] = sure; L.listed[wave] = fill; }
  __syncthreads();
  int all_sure, all_listed;
  waves_before(L.sure, NW, &all_sure);
  waves_before(L.listed, NW, &all_listed);
  const bool over = lane < NW && L.listed[lane & (NW - 1)] > kRowSeg;
  int need = k - all_sure;
  if (__builtin_amdgcn_ballot_w64(over) != 0 || need < 0 || all_listed < need) return false;
  auto mark = [&](uint32_t e) {
    atomicOr(reinterpret_cast<uint32_t*>(&L.word[e >> 6]) + ((e >> 5) & 1), 1u << (e & 31));   // (entry u NT + 64 wave + lane)
  };
  if (need > 0) {
    find_threshold_bin_n<NT>(hist, need, scan_scratch, L.at_lo);
    const int b = L.at_lo[0];
    int few = L.at_lo[2], b2 = -1;
    need = L.at_lo[1];
    const float from2 = from + (float)b / fine, fine2 = fminf(fine * (float)kBins, 3e38f);
    if (few > 64) {             // a crowded bin (scores that pile up: a query whose gates are all negative) is cut once more
      for (int i = tid; i < kBins; i += NT) hist[i] = 0;
      __syncthreads();
      for (int j = lane; j < fill; j += 64) {
        const float v = __uint_as_float(list[j].x);
        if (bin_of(v, from, fine) == b) atomicAdd(&hist[bin_of(v, from2, fine2)], 1);
      }
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, L.at_lo);
      b2 = L.at_lo[0];
      few = L.at_lo[2];
      need = L.at_lo[1];
    }
    for (int j = lane; j < fill; j += 64) {
      const uint2 e = list[j];
      int d = bin_of(__uint_as_float(e.x), from, fine) - b;
      if (d == 0 && b2 >= 0) d = bin_of(__uint_as_float(e.x), from2, fine2) - b2;
      if (d > 0) mark(e.y);
      if (d == 0) {
        if (few <= 64) L.few[atomicAdd(&L.few_len, 1)] = make_uint2(order_key(__uint_as_float(e.x)), e.y);
        else L.same = e.x;
      }
    }
    __syncthreads();
    if (few > 64) {
      // as a rule equal scores (the zeros of keys that no active head likes): the first of them
      const float same = __uint_as_float(L.same);
      bool unlike = false;
      for (int j = lane; j < fill; j += 64) {
        const float v = __uint_as_float(list[j].x);
        unlike |= bin_of(v, from, fine) == b && bin_of(v, from2, fine2) == b2 && v != same;
      }
      if (unlike) L.unlike = 1;
      uint2* const eq = reinterpret_cast<uint2*>(hist);      // (searched before the last barrier)
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        const unsigned long long m_eq = __builtin_amdgcn_ballot_w64(ei[u] >= 0 && ev[u] == same);
        if (lane == 0) eq[u * NW + wave] = make_uint2((uint32_t)m_eq, (uint32_t)(m_eq >> 32));
      }
      __syncthreads();
      if (L.unlike) return false;
      const uint2 w = tid < EPT * NW ? eq[tid] : make_uint2(0u, 0u);
      const int n_w = __popc(w.x) + __popc(w.y);
      int total;
      int left = need - block_exclusive_scan(n_w, scan_scratch, &total);
      if (tid < EPT * NW && left > 0) {
        unsigned long long bits = (unsigned long long)w.y << 32 | w.x, kept = bits;
        if (left < n_w) {
          kept = 0;
          for (; left > 0; --left) {
            kept |= bits & (0ull - bits);
            bits &= bits - 1;
          }
        }
        L.word[tid].x |= (uint32_t)kept;
        L.word[tid].y |= (uint32_t)(kept >> 32);
      }
      __syncthreads();
    } else {
    {
      // ranked by score, then index: all pairs, a wavefront comparing each entry with its share of the others
      constexpr int JP = 64 / NW;
      const uint2 own = L.few[lane];
      int rank = 0;
#pragma unroll
      for (int j = 0; j < JP; ++j) {
        const uint2 o = L.few[wave * JP + j];
        rank += (o.x > own.x || (o.x == own.x && o.y < own.y)) ? 1 : 0;
      }
      if (rank) atomicAdd(&L.few_rank[lane], rank);
    }
    __syncthreads();
    if (tid < few && L.few_rank[tid] < need) mark(L.few[tid].y);
    __syncthreads();
    }
  }

  // ---- output in entry order, which is index order
  {
    const uint2 w = tid < EPT * NW ? L.word[tid] : make_uint2(0u, 0u);
    int total;
    const int before = block_exclusive_scan(__popc(w.x) + __popc(w.y), scan_scratch, &total);
    if (tid < EPT * NW) L.before[tid] = before;
  }
  __syncthreads();
  const uint2 word = lane < EPT ? L.word[lane * NW + wave] : make_uint2(0u, 0u);
  const int before = lane < EPT ? L.before[lane * NW + wave] : 0;
  for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
    const uint32_t m_lo = __builtin_amdgcn_readlane(word.x, u), m_hi = __builtin_amdgcn_readlane(word.y, u);
    const int pos = __builtin_amdgcn_mbcnt_hi(m_hi, __builtin_amdgcn_mbcnt_lo(m_lo, (uint32_t)__builtin_amdgcn_readlane(before, u)));
    if (__builtin_amdgcn_inverse_ballot_w64((unsigned long long)m_hi << 32 | m_lo) && pos < k) {   // pos < k: always true when the selection is consistent
      out_idx[pos] = ei[u];
      if (out_val) out_val[pos] = ev[u];
    }
  });
  return true;
}

// One workgroup of NT threads per row: exact top-k of the row's candidate list.
// A thread keeps its (at most EPT) list entries in registers for all passes; index and score without their keys fit 64
// registers, so that two workgroups of 1024 threads share a CU.  Bound by the chain of barriers and loads of a row, which
// all workgroups go through in step, then by reading the lists (2048 rows of about 10500 entries: 95 us with the place of
// every entry searched by its thread and all of them counted, 82 now, 48 at the rate of a large copy; chunks found by
// ballots of every wavefront: 92).
template <int NT, int EPT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void select_rows_kernel(
    Prob p, const int2* __restrict__ cand, const int* __restrict__ seg, const int* __restrict__ seg_count,
    int ranges, const float* __restrict__ tau, const uint32_t* __restrict__ upper, int cap, int k, int qwg,
    int q_tiles, int* __restrict__ idx, float* __restrict__ val, int* __restrict__ row_flag,
    int* __restrict__ tile_flag) {
  extern __shared__ __align__(16) uint32_t dyn[];  // the sampled selection's lists; or the selection bitmap, then the prefix count of every bitmap word
  __shared__ __align__(16) int hist[kBins];   // (also the marks of equal scores, in words of 8 bytes: select_sampled)
  __shared__ int scan_scratch[32];
  __shared__ int thr[3];
  __shared__ uint32_t bkey[64];
  __shared__ int bidx[64];
  __shared__ int b_len;
  __shared__ int brank[64];       // entries of the boundary list that rank before an entry
  constexpr int NW = NT / 64, kSlab = NT / kChunk;
  const int t = blockIdx.x, seq = blockIdx.y, tid = threadIdx.x;
  const size_t row = (size_t)seq * p.n_q + t;
  const int n = visible(p, seq, t);
  const int k_eff = min(k, n);
  int* out_idx = idx + row * k;
  float* out_val = val ? val + row * k : nullptr;
  for (int i = k_eff + tid; i < k; i += NT) {
    out_idx[i] = -1;
    if (out_val) out_val[i] = -INFINITY;
  }
  if (k_eff == 0) return;
  // The row's entries: range r holds seg_count[r] of them from seg[r] on; a count above the segment's length means that
  // hits were dropped.  They are taken in chunks of kChunk of one range, one after another by 16 lanes each, in slabs of NT;
  // lane r of every wavefront looks after range r, and the wavefronts together write down where the chunks are.
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int cnt = 0, len = 0, first_entry = 0;
  if (lane < ranges) {
    first_entry = seg[row * (ranges + 1) + lane];
    len = seg[row * (ranges + 1) + lane + 1] - first_entry;
    cnt = seg_count[row * ranges + lane];
  }
  const bool dropped = __builtin_amdgcn_ballot_w64(cnt > len) != 0;
  const int mine = (cnt + kChunk - 1) / kChunk;
  const int chunk_end = wave_inclusive_scan(mine), chunks = __builtin_amdgcn_readlane(chunk_end, 63);
  const int entry_end = wave_inclusive_scan(cnt), c = __builtin_amdgcn_readlane(entry_end, 63);
  if (dropped || chunks > kSlab * EPT || c < k_eff) {  // a segment overflowed, more entries than this kernel holds, or threshold too high: leave the row to the repair pass
    if (tid == 0) {
      row_flag[row] = 1;
      tile_flag[seq * q_tiles + t / qwg] = 1;
    }
    return;
  }
  const int nwords = (n + 31) / 32;
  uint32_t* sel = dyn;
  int* wpre = reinterpret_cast<int*>(dyn + (p.L + 31) / 32);
  // this thread's entries: index (-1 = none) and score; the order-preserving key is made again in every
  // pass, so that two workgroups of 1024 threads fit a CU (64 registers)
  int ei[EPT];
  float ev[EPT];
  const int2* src = cand + row * (size_t)cap;
  __shared__ int2 s_chunk[kSlab * EPT];   // place of a chunk's first entry in the row's list; its number in the row and, in 8 bits, the chunk's entries
  for (int q = wave; __builtin_amdgcn_ballot_w64(q < mine) != 0; q += NW)
    if (q < mine)
      s_chunk[chunk_end - mine + q] = make_int2(first_entry + kChunk * q, (entry_end - cnt + kChunk * q) << 8 | min(cnt - kChunk * q, kChunk));
  for (int j = chunks + tid; j < kSlab * EPT; j += NT) s_chunk[j] = make_int2(0, 0);
  for (int i = tid; i < kBins; i += NT) hist[i] = 0;
  __syncthreads();
  const int slabs = (chunks + kSlab - 1) / kSlab;
#pragma unroll
  for (int u = kPart1<NT>; u < EPT; ++u) { ei[u] = -1; ev[u] = 0.f; }
  for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
    const int2 chunk = s_chunk[u * kSlab + tid / kChunk];
    const int in_chunk = tid % kChunk;
    const bool live = in_chunk < (chunk.y & 0xFF);
    const int2 e = src[live ? chunk.x + in_chunk : 0];
    ei[u] = live ? e.x : -1;
    ev[u] = __int_as_float(e.y);
  });
  if (c == k_eff) {       // every entry, in index order
#pragma unroll
    for (int u = 0; u < EPT; ++u)
      if (ei[u] >= 0) {
        const int at = (s_chunk[u * kSlab + tid / kChunk].y >> 8) + tid % kChunk;
        out_idx[at] = ei[u];
        if (out_val) out_val[at] = ev[u];
      }
    return;
  }
  __shared__ EntryLds<NT, EPT> entry_lds;
  if (c >= kSampledMin && k_eff >= kSampledMinK && select_sampled<NT, EPT>(ei, ev, c, slabs, k_eff, tau[row], key_to_float(upper[row]), hist, scan_scratch, dyn, entry_lds, out_idx, out_val)) return;
  // the digits of the keys instead
  __syncthreads();
  auto key_of = [&](int u) { return order_key(ev[u]); };
  for (int i = tid; i < nwords; i += NT) sel[i] = 0;
  if (tid == 0) b_len = 0;
  if (tid < 64) brank[tid] = 0;
  zero_hist_n<NT>(hist);
  auto mark = [&](int e) { atomicOr(&sel[e >> 5], 1u << (e & 31)); };

  // Lists below kSampledMin and k below kSampledMinK, as a rule: one digit of key - key(tau), scaled so that [tau, upper]
  // fills the 2047 lower values of the digit (larger keys share 2047).  The list entries then spread over the whole
  // histogram instead of piling up in the few bins a raw key prefix gives them; entries above
  // the digit of the k-th largest are selected and the few inside it ranked against each other
  // (score descending, index ascending).  More than 64 entries in that digit, or the catch-all
  // digit: the three raw key digits below decide instead.
  bool done = false;
  {
    const uint32_t klo = order_key(tau[row]);
    const uint32_t up = upper[row];
    const uint32_t span = up > klo ? up - klo : 1u;
    const int sh = __clz(span);
    auto digit = [&](uint32_t key) {
      const uint32_t x = key > klo ? key - klo : 0u;
      return x > span ? (uint32_t)(kBins - 1) : (x << sh) >> 21;
    };
    for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
      if (ei[u] >= 0) atomicAdd(&hist[digit(key_of(u))], 1);
    });
    __syncthreads();
    find_threshold_bin_n<NT>(hist, k_eff, scan_scratch, thr);
    const uint32_t d1 = thr[0];
    const int need = thr[1], nb = thr[2];
    if (nb <= 64 && d1 != kBins - 1) {   // block-uniform
      // (digit > d1 and == d1 as compares of the shifted distance; d1 < 2047, and what lies past the span
      // shares 2047)
      const uint32_t from = d1 << 21, past = (d1 + 1) << 21;
      for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
        const uint32_t key = key_of(u), x = key > klo ? key - klo : 0u, y = x > span ? 0xFFFFFFFFu : x << sh;
        if (ei[u] >= 0 && y >= past) mark(ei[u]);
        const bool edge = ei[u] >= 0 && y >= from && y < past;
        if (__builtin_amdgcn_ballot_w64(edge)) {
          const int b = wave_append(edge, &b_len);
          if (b >= 0) { bkey[b] = key_of(u); bidx[b] = ei[u]; }
        }
      });
      __syncthreads();
      {
        // all pairs of the (at most 64) boundary entries, spread over the block: thread t compares
        // entry t % 64 with its share of the others
        constexpr int JP = 64 / (NT / 64);
        const int i = tid & 63, j0 = (tid >> 6) * JP;
        if (i < nb && j0 < nb) {
          const uint32_t key = bkey[i];
          const int e = bidx[i];
          int part = 0;
#pragma unroll
          for (int j = j0; j < j0 + JP; ++j)
            part += (j < nb && (bkey[j] > key || (bkey[j] == key && bidx[j] < e))) ? 1 : 0;
          if (part) atomicAdd(&brank[i], part);
        }
      }
      __syncthreads();
      if (tid < nb && brank[tid] < need) mark(bidx[tid]);
      done = true;
    } else {
      __syncthreads();
      zero_hist_n<NT>(hist);
    }
  }

  if (!done) {
    // most significant digit first: 11 + 11 + 10 bits of the key
#pragma unroll
    for (int u = 0; u < EPT; ++u)
      if (ei[u] >= 0) atomicAdd(&hist[key_of(u) >> 21], 1);
    __syncthreads();
    find_threshold_bin_n<NT>(hist, k_eff, scan_scratch, thr);
    const uint32_t d1 = thr[0];
    int need = thr[1];
    __syncthreads();
    zero_hist_n<NT>(hist);
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      if (ei[u] < 0) continue;
      const uint32_t a = key_of(u) >> 21;
      if (a > d1) mark(ei[u]);
      else if (a == d1) atomicAdd(&hist[(key_of(u) >> 10) & 0x7FF], 1);
    }
    __syncthreads();
    find_threshold_bin_n<NT>(hist, need, scan_scratch, thr);
    const uint32_t pre22 = (d1 << 11) | (uint32_t)thr[0];
    need = thr[1];
    __syncthreads();
    zero_hist_n<NT>(hist);
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      if (ei[u] < 0 || (key_of(u) >> 21) != d1) continue;
      if ((key_of(u) >> 10) > pre22) mark(ei[u]);
      else if ((key_of(u) >> 10) == pre22) atomicAdd(&hist[key_of(u) & 0x3FF], 1);
    }
    __syncthreads();
    find_threshold_bin_n<NT>(hist, need, scan_scratch, thr);
    const uint32_t tkey = (pre22 << 10) | (uint32_t)thr[0];
    need = thr[1];
    const int ties = thr[2];
    __syncthreads();
    if (ties == need) {
#pragma unroll
      for (int u = 0; u < EPT; ++u)
        if (ei[u] >= 0 && (key_of(u) >> 10) == pre22 && key_of(u) >= tkey) mark(ei[u]);
    } else {
      // More entries equal to the threshold value than places: the `need` lowest
      // indices among them win, found by the same digit search on the (high, low)
      // halves of the index with the bin order inverted.
      zero_hist_n<NT>(hist);
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        if (ei[u] < 0) continue;
        if ((key_of(u) >> 10) == pre22 && key_of(u) > tkey) mark(ei[u]);
        else if (key_of(u) == tkey) atomicAdd(&hist[kBins - 1 - (ei[u] >> 10)], 1);
      }
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr);
      const int hi_digit = kBins - 1 - thr[0];
      need = thr[1];
      __syncthreads();
      zero_hist_n<NT>(hist);
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        if (ei[u] < 0 || key_of(u) != tkey) continue;
        if ((ei[u] >> 10) < hi_digit) mark(ei[u]);
        else if ((ei[u] >> 10) == hi_digit) atomicAdd(&hist[kBins - 1 - (ei[u] & 0x3FF)], 1);
      }
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr);
      const int lo_digit = kBins - 1 - thr[0];
#pragma unroll
      for (int u = 0; u < EPT; ++u) {
        if (ei[u] < 0 || key_of(u) != tkey) continue;
        if ((ei[u] >> 10) == hi_digit && (ei[u] & 0x3FF) <= lo_digit) mark(ei[u]);
      }
    }
  }
  __syncthreads();

  // Output slot of a selected index = number of selected indices below it.
  const int wpt = (nwords + NT - 1) / NT;
  const int w_lo = min(tid * wpt, nwords), w_hi = min(w_lo + wpt, nwords);
  int selected = 0;
  for (int w = w_lo; w < w_hi; ++w) selected += __popc(sel[w]);
  int total;
  int pos = block_exclusive_scan(selected, scan_scratch, &total);
  for (int w = w_lo; w < w_hi; ++w) {
    wpre[w] = pos;
    pos += __popc(sel[w]);
  }
  __syncthreads();
  for_entries<NT, EPT>(slabs, [&](int u) __attribute__((always_inline)) {
    const int e = ei[u];
    if (e < 0) return;
    const uint32_t bits = sel[e >> 5], bit = 1u << (e & 31);
    if (!(bits & bit)) return;
    const int slot = wpre[e >> 5] + __popc(bits & (bit - 1u));
    if (slot < k) {  // always true when the selection is consistent
      out_idx[slot] = e;
      if (out_val) out_val[slot] = ev[u];
    }
  });
}

// ---------------------------------------------------------------- host side
namespace {

struct Layout {
  size_t S, sample, tau, upper, row_flag, tile_flag, seg, seg_count, cand, total;
  int m, cap, qwg, q_tiles, ranges, keys_per_range;
};

size_t up(size_t x) { return (x + 255) & ~(size_t)255; }

Layout layout(const Prob& p, bool routed, int k, bool q8 = false) {
  Layout l;
  const size_t rows = (size_t)p.n_seq * p.n_q;
  l.m = p.L / kSampleStride;
  l.ranges = tile_key_ranges(p, routed, q8, kTileFilter, &l.keys_per_range);
  l.cap = list_capacity(k, l.ranges);
  l.qwg = tile_queries_per_wg(p, routed, q8);
  l.q_tiles = (p.n_q + l.qwg - 1) / l.qwg;
  size_t o = 0;
  l.S = o;         o += up(rows * p.L * sizeof(float));
  l.sample = o;    o += up(rows * l.m * sizeof(float));
  l.tau = o;       o += up(rows * sizeof(float));
  l.upper = o;     o += up(rows * sizeof(uint32_t));
  l.row_flag = o;  o += up(rows * sizeof(int));
  l.tile_flag = o; o += up((size_t)p.n_seq * l.q_tiles * sizeof(int));
  l.seg = o;       o += up(rows * (l.ranges + 1) * sizeof(int));
  l.seg_count = o; o += up(rows * l.ranges * sizeof(int));
  l.cand = o;      o += up(rows * l.cap * sizeof(int2));
  l.total = o;
  return l;
}

}  // namespace

size_t select_ws_bytes(const Prob& p, int k_dtype, int q_dtype, int k) {
  if (k < 1) return 0;
  const size_t dense = up((size_t)p.n_seq * p.n_q * p.L * sizeof(float));
  if (!fused(p, k_dtype, q_dtype, k)) return dense + up(topk_ws_bytes(p, k));
  // the number of key ranges, hence the list capacity, and the number of query tiles depend
  // on the head count of the call: room for either kind
  return std::max(layout(p, false, k).total, layout(p, true, k).total);
}

long long select_row_flags_offset(const Prob& p, int k_dtype, int q_dtype, bool routed, int k) {
  if (k < 1 || !fused(p, k_dtype, q_dtype, k)) return -1;
  return (long long)layout(p, routed, k).row_flag;
}

hipError_t launch_select(const Prob& p, int k_dtype, int q_dtype, const void* Q, const float* W,
                         const int* heads, const void* K, const float* kscale, int k, int* idx,
                         float* val, void* ws, hipStream_t st) {
  char* base = static_cast<char*>(ws);
  if (!fused(p, k_dtype, q_dtype, k)) {
    float* S = reinterpret_cast<float*>(base);
    const size_t dense = up((size_t)p.n_seq * p.n_q * p.L * sizeof(float));
    hipError_t e = launch_score(p, k_dtype, q_dtype, Q, W, heads, K, kscale, nullptr, 0, S, st);
    if (e != hipSuccess) return e;
    return launch_topk(p, S, p.L, k, nullptr, idx, val, base + dense, st);
  }
  const Layout l = layout(p, heads != nullptr, k, q_dtype == MISA_FP8_E4M3);
  float* S = reinterpret_cast<float*>(base + l.S);
  float* Ss = reinterpret_cast<float*>(base + l.sample);
  float* tau = reinterpret_cast<float*>(base + l.tau);
  uint32_t* upper = reinterpret_cast<uint32_t*>(base + l.upper);
  int* seg = reinterpret_cast<int*>(base + l.seg);
  int* seg_count = reinterpret_cast<int*>(base + l.seg_count);
  int* row_flag = reinterpret_cast<int*>(base + l.row_flag);
  int* tile_flag = reinterpret_cast<int*>(base + l.tile_flag);
  int2* cand = reinterpret_cast<int2*>(base + l.cand);
  const dim3 rows(p.n_q, p.n_seq);

  // The row selection holds a row's entries in registers: 512 threads x 10 or 12 for up to 5120 expected entries (16 r and
  // six standard deviations of 16 sqrt(r)), 1024 x 13 or 14 above.  Rows all of whose visible keys are listed fill their
  // chunks (a key range is whole tiles of 64 keys).
  const double rr = sample_rank(k);
  const bool small_rows = kSampleStride * rr * (1.0 + 6.0 / std::sqrt(rr)) <= 5120.0;
  const int entry_limit = small_rows ? 512 * 10 : 1024 * 13;
  // Listed whole: rows of what a list in 8 key ranges has room for.  (A list in more ranges has more room, 450 entries per
  // range for k = 2, but a threshold costs less than entries that it would have kept away: 313 rows of up to 5139 keys, k = 2, 16 ranges
  // 48.8 us with rows of 5120 listed whole, 42.7 with 8 ranges.)
  const int keep_all = std::min(std::min(l.cap, list_capacity(k, 8)), entry_limit);

  hipError_t e = launch_tile_mode(p, k_dtype, q_dtype, kTileSample, TileAux{}, Q, W, heads, K, kscale, Ss, st);
  if (e != hipSuccess) return e;
  select_threshold_kernel<<<p.n_seq * p.n_q, kThrThreads, 0, st>>>(
      p, Ss, l.m, sample_rank(k), l.cap, keep_all, l.qwg, l.q_tiles, l.ranges, l.keys_per_range, max_sample_hits(k), tau,
      upper, seg, row_flag, tile_flag);
  if ((e = hipGetLastError()) != hipSuccess) return e;

  TileAux filter;
  filter.tau = tau;
  filter.cand = cand;
  filter.seg = seg;
  filter.seg_count = seg_count;
  filter.cap = l.cap;
  filter.ranges = l.ranges;
  e = launch_tile_mode(p, k_dtype, q_dtype, kTileFilter, filter, Q, W, heads, K, kscale, nullptr, st);
  if (e != hipSuccess) return e;

  const size_t lds = select_lds_bytes(p);  // at most 128 KB (L <= 524288)
#define GO(NT, EPT)                                                                                 \
  do {                                                                                              \
    static LdsSeen seen;                                                                            \
    const size_t dyn = std::max(lds, row_list_bytes<NT>());                                         \
    e = ensure_dynamic_lds(reinterpret_cast<const void*>(select_rows_kernel<NT, EPT>), dyn, seen);  \
    if (e != hipSuccess) return e;                                                                  \
    select_rows_kernel<NT, EPT><<<rows, NT, dyn, st>>>(p, cand, seg, seg_count, l.ranges, tau, upper, l.cap, k, \
                                                       l.qwg, l.q_tiles, idx, val, row_flag, tile_flag); \
  } while (0)
  // the smallest room that is enough: without it a row goes to the repair pass, whatever the selection itself would take
  const int room = row_room(k, l.ranges);      // at most 5914 for small rows, 13639 for k = kFusedMaxK (64 ranges)
  if (small_rows) {
    if (room <= 512 * 10) GO(512, 10);
    else GO(512, 12);
  } else {
    if (room <= 1024 * 13) GO(1024, 13);
    else GO(1024, 14);
  }
#undef GO
  if ((e = hipGetLastError()) != hipSuccess) return e;

  // repair pass, a no-op unless rows were flagged
  TileAux repair;
  repair.run = tile_flag;
  e = launch_tile_mode(p, k_dtype, q_dtype, kTileStore, repair, Q, W, heads, K, kscale, S, st);
  if (e != hipSuccess) return e;
  return launch_topk(p, S, p.L, k, nullptr, idx, val, nullptr, st, row_flag);
}

}  // namespace misa
