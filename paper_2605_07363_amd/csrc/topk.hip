// Stage 4: exact per-row top-k (Eq. dsa_topk, Eq. misa_topk, Eq. misa_candidate).
//
// The k-th largest value of a row is found by a most-significant-digit-first
// radix select (11 + 11 + 10 bits) on an order-preserving integer image of the
// fp32 scores.  Selected elements are marked in an LDS bitmap of the row and
// the result is expanded from the bitmap in index order with one block-wide
// prefix sum, so the output is ascending and bit-reproducible without a sort.
//
// Usual case (sampled path): the row is read once.  A sample of the row brackets the k-th largest
// value between two thresholds; while the row streams through registers the elements above the
// lower one are listed, and the list is selected from exactly.  The counts found on the way prove
// the bracket right or wrong, so the result never depends on the sample: a row whose list is too short
// or too long gets another bracket from the count of the first, a row whose k-th largest lies on a plateau
// of equal values is marked in one more pass, and what is left (NaN, further wrong brackets) is redone
// by the radix select on the row itself, which reads it twice or four times.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "radix.h"

namespace misa {

constexpr int kFew = 64;             // entries around the k-th largest that are ranked directly
constexpr int kListTarget = 6000;    // boundary list entries of the two-pass path, where LDS is cheap

// How a block of NT threads takes a row.  A short row of at most 16 (256 threads) or 8 elements per
// thread stays in registers and is its own sample.  Otherwise the row is streamed and at most eight
// elements per thread are sampled.
constexpr int kHeldLong = 8;
constexpr int kAttempts = 4;         // further brackets tried on a row
__host__ __device__ constexpr int held_hard(int nt) { return nt == 256 ? 16 : 8; }
__host__ __device__ constexpr int held_short(int nt) { return nt == 256 ? 16 : 8; }

template <int NT>
__device__ __forceinline__ void clear_hist(int* hist) {
  for (int i = this_thread(); i < kBins; i += NT) hist[i] = 0;
  __syncthreads();
}

// Visits elements lo..hi-1 of a row with all threads of the block.  Eight
// coalesced loads per thread are in flight before the first one is used.  f is
// called by every thread of every wavefront in each round (in == false past
// the end), so it may contain wavefront-wide operations.
template <int NT, int U = 8, typename F>
__device__ __forceinline__ void scan_row(const float* __restrict__ s, int lo, int hi, F f) {
  const int tid = this_thread();
  for (int base = lo; base < hi; base += NT * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * NT + tid;
      v[u] = i < hi ? s[i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * NT + tid;
      f(i, v[u], i < hi);
    }
  }
}

// Sampled 16-element lines of the n visible elements of a long row of row_len: about 4096 elements, 8192 for
// large k and where rows may be very long (they narrow the bracket, whose width in elements grows with
// sqrt(k n / samples)).  row_len decides and not n: the list is sized for a row of row_len elements, and a
// shorter one may not be sampled more coarsely.
__host__ __device__ inline int sample_lines(int n, int row_len, int k, int nt) {
  return nt == kTopkThreads && (n <= 8192 || k > 4096 || row_len > 131072) ? 512 : 256;
}

// LDS words of the bitmap of a row, which a histogram has to fit as well; even, because the list behind
// it has 8-byte entries.
__host__ __device__ inline int sel_words(int row_len) { return (max((row_len + 31) / 32, kBins) + 1) & ~1; }

// ---------------------------------------------------------------- sampled path
//
//   sample   16-element lines, one of every `ls` at a hashed place (the short rows of the smaller
//            blocks are their own sample and stay in registers).  The k-th largest of the row lies
//            between the sample elements of rank r_hi and r_lo = k m/n -+ (6 sqrt(k m/n) + 8): the
//            number of the top k in the sample has mean k m/n and, if the elements of a line are
//            independent, no larger variance (lines of like elements: up to 16 times; see "again").
//            Both are found by a histogram that is linear between the smallest and the largest
//            sample and rounded outwards to the values lo and hi of the bracket.  Where outliers leave
//            the bin of lo too coarse it is repeated inside that bin, then (hard_row) cut by digits of
//            the key until few samples are left in it, or one value.
//   stream   Elements >= lo (and NaN) go to the list, at places counted from the ballots of the
//            compares; a wavefront claims the places of eight ballots with one atomic: five vector
//            instructions per 64 elements.  (At the 6 TB/s of the memory a CU has time for that many
//            and no more; with the bitmap marked here from a second compare, and a list of only the
//            elements in between, the same rows took 1.3 times as long.)  A register is requested
//            again as soon as its elements have been looked at.
//            A list segment per wavefront instead of the claims overflows where the large values lie
//            in stretches.
//   select   Entries >= hi are sure and only counted; need = k - sure of the others are found by a
//            histogram that is linear over [lo, hi), and a second one inside a crowded bin; the few
//            entries in the bin of the need-th are ranked against each other, or, if there are many
//            (repeated values), resolved by the digits of key and index.
//
//   again    (hard_row)  If sure > k, the row is sampled and streamed again without an upper end; if fewer than
//            k or more than the list holds pass, with the rank r_lo scaled by what the last count says of it.
//            One value: what lies above it and the first of it are marked.
// A NaN leaves the row to the two-pass path.  Candidate rows never select -inf: it lies below the bracket.
// The histograms share their LDS with the bitmap, which is cleared once the last of them has been read.
//
// Measured: 4096 rows of 65536, k = 2048: 212 us = 5.1 TB/s (two passes over each row: 402 us; sample and
// stream alone, nothing selected: 190 us); 64 rows of 32768: 14.6 us (17.3 us in two launches).  Few rows
// are a chain of barrier-separated phases of one workgroup.
struct Bracket {
  float lo, hi;
  float edge;   // upper end of the histogram: hi where it is finite
};
enum Found { kNoBracket, kBracket, kPlateau };   // kPlateau: the lower end is one value that repeats

// What the phases of a block share.
template <int NT>
struct TopkLds {
  int scan_scratch[32];
  int thr[3], thr_up[3];
  int list_fill, few_len, nan_seen;
  int wave_sure[NT / 64], wave_more[NT / 64];
  float wave_min[NT / 64], wave_max[NT / 64];
  uint32_t fkey[kFew];
  int fidx[kFew];
  int frank[kFew];   // entries of the few that rank before an entry
};

// values at or above `from`, in bins of 1 / scale; all others in bin 0, values past the end in the last
__device__ __forceinline__ int linear_bin(float v, float from, float scale) {
  return (int)__builtin_amdgcn_fmed3f((v - from) * scale, 0.f, (float)(kBins - 1));
}

// Value of a key (the inverse of order_key; a key between those of -0 and +0 gives -0).
__device__ __forceinline__ float key_value(uint32_t key) {
  return __uint_as_float(key & 0x80000000u ? key ^ 0x80000000u : ~key);
}
constexpr uint32_t kKeyPosInf = 0xFF800000u;

// Counts bins in an LDS histogram: U of each lane (all active; bin_of(u) < 0: none).  LDS adds of a wavefront to
// one address go one after the other, so where the first lane's bin is that of a quarter of the lanes (far outliers,
// plateaus) its count is taken from ballots and added once.
template <int U, typename F>
__device__ __forceinline__ void count_bins(int* hist, F bin_of) {
  const int first = __builtin_amdgcn_readfirstlane(bin_of(0));
  if (__popcll(__builtin_amdgcn_ballot_w64(bin_of(0) == first)) >= 16 && first >= 0) {   // wavefront-uniform
    int same = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int bin = bin_of(u);
      same += __popcll(__builtin_amdgcn_ballot_w64(bin == first));
      if (bin >= 0 && bin != first) atomicAdd(&hist[bin], 1);
    }
    if ((this_thread() & 63) == 0) atomicAdd(&hist[first], same);
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int bin = bin_of(u);
      if (bin >= 0) atomicAdd(&hist[bin], 1);
    }
  }
}

// The sample of a row of n elements: of every ls lines one, HELD elements per thread (-inf where there is none).
struct Sample {
  int m, ls;          // sample elements; lines per sampled line
  int r_lo, r_hi;     // ranks of the bracket's ends in the sample
  int rank_up;        // rank of the upper end of the histogram of the list
};
template <int NT, bool SHORT, int HELD, typename F>
__device__ __forceinline__ Sample take_sample(const float* __restrict__ s, int n, int row_len, int k, int tid,
                                              float (&held)[HELD], F also) {
  Sample sm;
  const int lines = (n + 15) >> 4, max_lines = SHORT ? lines : sample_lines(n, row_len, k, NT);
  const int ls = (lines + max_lines - 1) / max_lines;
  const int groups = lines / ls;       // >= 1
  // (16-bit hash and ls <= 128: 24-bit products)
  auto line_of = [&](uint32_t g) { return (int)(__umul24(g, ls) + (__umul24((g * 2654435761u) >> 16, ls) >> 16)); };
  bool in[HELD];
#pragma unroll
  for (int u = 0; u < HELD; ++u) {
    const int smp = tid + u * NT, g = smp >> 4;
    const int i = SHORT ? smp : line_of(g) * 16 + (smp & 15);
    in[u] = (SHORT || g < groups) && i < n;
    held[u] = s[in[u] ? i : 0];
  }
  also();
  // number of samples: 16 per sampled line, less what the row's last line lacks if it is one
  int m = 16 * groups;
  {
    const int last = lines - 1, g = last / ls;
    if (g < groups && line_of(g) == last) m -= 16 * lines - n;
  }
  sm.m = m;
  sm.ls = ls;
  sm.r_lo = sm.r_hi = k;
  if (ls > 1) {
    const float kf = (float)k * (float)m / (float)n, margin = 6.f * sqrtf(kf) + 8.f;
    sm.r_lo = (int)ceilf(kf + margin);
    sm.r_hi = (int)floorf(kf - margin);
  }
  sm.rank_up = sm.r_hi >= 1 ? sm.r_hi : max(sm.r_lo / 16, 1);   // (hi open: the histogram ends above most of the top k)
#pragma unroll
  for (int u = 0; u < HELD; ++u) held[u] = in[u] ? held[u] : -INFINITY;
  return sm;
}

// The bracket of a row's k-th largest of n > k elements (block-uniform) from a histogram of the sample that is
// linear between the smallest and the largest one, masks and the like left out (below they are not counted, above
// they share the last bin), and while that is too coarse (far outliers, heavy tails) from a second and a third one
// inside the r_lo-th sample's bin; false if the third is, too.  The lowest bin is not counted: it holds nearly all
// samples of a row with heavy tails, and LDS adds to one address go one after the other.  `also` is called once the
// sample's loads have been issued.  Leaves hist cleared if there is a bracket.
template <int NT, bool SHORT, int HELD, typename F>
__device__ __forceinline__ bool sample_bracket(const float* __restrict__ s, int n, int row_len, int k, float (&held)[HELD],
                                               int* hist, TopkLds<NT>& L, Bracket& br, F also) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Sample sm = take_sample<NT, SHORT>(s, n, row_len, k, tid, held, [&] {
    also();
    for (int i = tid; i < kBins; i += NT) hist[i] = 0;
    if (tid == 0) { L.few_len = 0; L.nan_seen = 0; L.list_fill = 0; L.thr[2] = 0; L.thr_up[2] = 0; }
    if (tid < kFew) L.frank[tid] = 0;
  });
  if (sm.r_lo > sm.m) return false;
  float lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int u = 0; u < HELD; ++u)
    if (fabsf(held[u]) < 1e30f) { lo = fminf(lo, held[u]); hi = fmaxf(hi, held[u]); }
  lo = -wave_max_f32(-lo);
  hi = wave_max_f32(hi);
  if (lane == 0) { L.wave_min[wave] = lo; L.wave_max[wave] = hi; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) { lo = fminf(lo, L.wave_min[w]); hi = fmaxf(hi, L.wave_max[w]); }
  br.edge = INFINITY;
  for (int pass = 0;; ++pass) {
    const float width = (hi - lo) * (1.f / kBins), per = (float)kBins / (hi - lo);
    if (!(width > 0.f) || !(per < 3e38f)) return false;
    const float counted = lo + width;
    if constexpr (SHORT) {   // (a whole row; for 4096 samples the test costs 0.1 to 0.6 us and a shared bin 1.7 us)
      count_bins<HELD>(hist, [&](int u) { return held[u] >= counted ? linear_bin(held[u], lo, per) : -1; });
    } else {
#pragma unroll
      for (int u = 0; u < HELD; ++u)
        if (held[u] >= counted) atomicAdd(&hist[linear_bin(held[u], lo, per)], 1);
    }
    __syncthreads();
    find_threshold_bin_n<NT>(hist, sm.r_lo, L.scan_scratch, L.thr, sm.rank_up, L.thr_up, this_thread());
    const int crowd = L.thr[2], b_lo = crowd ? L.thr[0] : 0, b_hi = L.thr_up[0];   // (crowd 0: not among the counted)
    // rounding of the bins: 2048 x 2^-22 of one, and what lo and hi have lost by their size
    const float slack = 0.001f * width + 2.5e-7f * fmaxf(fabsf(lo), fabsf(hi));
    br.lo = fmaxf(lo + (float)b_lo * width - slack, -FLT_MAX);   // (never -inf, which pads the list appends)
    if (L.thr_up[2] != 0 && (b_hi < kBins - 1 || br.edge == INFINITY)) br.edge = lo + (float)(b_hi + 1) * width + slack;
    for (int i = tid; i < kBins; i += NT) hist[i] = 0;   // (read by everybody: find_threshold_bin ends with a barrier)
    __syncthreads();
    if (crowd != 0 && crowd <= 64) {
      br.hi = sm.r_hi >= 1 ? br.edge : INFINITY;
      return true;
    }
    if (pass == 2) return false;
    hi = lo + (float)(b_lo + 1) * width + slack;
    lo = br.lo;
    if (tid == 0) { L.thr[2] = 0; L.thr_up[2] = 0; }
  }
}

// The same by digits of the key, 11 bits each time until few samples are left beside the r_lo-th, or one value.
template <int NT, int HELD>
__device__ __forceinline__ Found key_bracket(int cap, const Sample& sm, const float (&held)[HELD], int* hist,
                                             TopkLds<NT>& L, Bracket& br) {
  constexpr int NW = NT / 64;
  const int tid = this_thread(), lane = tid & 63, wave = tid >> 6;
  if (sm.r_lo > sm.m) return kNoBracket;
  // samples past the r_lo-th that the list has room for
  const int spare = sm.ls == 1 ? max(cap - sm.r_lo, 0) : (int)(3.f * sqrtf((float)sm.r_lo));
  __syncthreads();
  clear_hist<NT>(hist);
  uint32_t key_lo = order_key(-FLT_MAX), key_hi = kKeyPosInf;   // key range of the r_lo-th sample
  br.hi = br.edge = INFINITY;
#pragma unroll 1
  for (;;) {
    const int sh = max(21 - (int)__clz(key_hi - key_lo), 0);
    auto digit = [&](uint32_t key) { return key >= key_lo && key <= key_hi ? (int)((key - key_lo) >> sh) : -1; };
    int above = 0;
#pragma unroll
    for (int u = 0; u < HELD; ++u) above += order_key(held[u]) > key_hi ? 1 : 0;
    count_bins<HELD>(hist, [&](int u) { return digit(order_key(held[u])); });
    above = wave_inclusive_scan(above);
    if (lane == 63) L.wave_sure[wave] = above;
    if (tid == 0) L.thr[2] = 0;
    __syncthreads();
    waves_before(L.wave_sure, NW, &above);
    const int r = sm.r_lo - above;
    find_threshold_bin_n<NT>(hist, r, L.scan_scratch, L.thr, sm.rank_up - above, L.thr_up, this_thread());
    const int b_lo = L.thr[0], crowd = L.thr[2], rest = crowd - L.thr[1];
    if (r < 1 || crowd == 0) return kNoBracket;   // the r_lo-th sample is infinite
    if (sm.rank_up - above >= 1) {
      br.edge = key_value(min(key_lo + ((uint32_t)(L.thr_up[0] + 1) << sh), kKeyPosInf));
      br.hi = sm.r_hi >= 1 ? br.edge : INFINITY;
    }
    key_lo += (uint32_t)b_lo << sh;
    key_hi = min(key_hi, key_lo + ((1u << sh) - 1u));
    br.lo = key_value(key_lo);
    if (key_lo == kKeyPosInf) return kPlateau;
    br.edge = fmaxf(br.edge, key_value(key_lo + 1));
    for (int i = tid; i < kBins; i += NT) hist[i] = 0;
    __syncthreads();
    if (rest <= spare) return kBracket;
    if (sh == 0) return kPlateau;
  }
}

// The elements of a stretch of the row that reach `lo` go to the list (`cap` entries and 64 of slack,
// its fill in *fill, which counts on past cap); indices are counted from `first`.  The eight values of a
// lane: the compares, one claim of list places for all that pass, the places, the stores.
template <typename INDEX>
__device__ __forceinline__ void list_append(const float (&x)[8], float lo, uint2* list, int cap, int* fill, INDEX index) {
  unsigned long long pass[8];
  int total = 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    pass[c] = __builtin_amdgcn_ballot_w64(!(x[c] < lo));
    total += __popcll(pass[c]);
  }
  int base = 0;
  if ((threadIdx.x & 63) == 0) base = atomicAdd(fill, total);
  base = __builtin_amdgcn_readfirstlane(base);
  uint32_t* at[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(pass[c] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pass[c], 0));
    at[c] = reinterpret_cast<uint32_t*>(list + min(base, cap)) + 2 * below;
    base += __popcll(pass[c]);
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    if (__builtin_amdgcn_inverse_ballot_w64(pass[c])) {
      at[c][0] = __float_as_uint(x[c]);
      at[c][1] = (uint32_t)index(c);
    }
  }
}

// A stretch of n elements: vectors of four elements per thread in blocks of 4 NT elements, the rest one
// by one.  begin() requests the first vectors.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // (16-byte loads need 4-byte alignment only)
template <int NT, int AHEAD>
struct Stream {
  const float* s;
  int n, blocks, tid;
  f32x4_u v[AHEAD];

  __device__ __forceinline__ f32x4_u request(int block) const {
    return reinterpret_cast<const f32x4_u*>(s + min(block, blocks - 1) * 4 * NT)[tid];
  }
  __device__ __forceinline__ void begin(const float* s_, int n_, int tid_) {
    s = s_;
    n = n_;
    tid = tid_;
    blocks = n / (4 * NT);
    if (blocks == 0) return;
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = request(u);
  }
  __device__ __forceinline__ void filter(float lo, int first, uint2* list, int cap, int* fill) {
    const int rest0 = blocks * 4 * NT;
    float rest[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) rest[u] = s[min(rest0 + u * NT + tid, n - 1)];
    auto two_blocks = [&](const f32x4_u& p, const f32x4_u& q, int block) {
      const float x[8] = {p[0], p[1], p[2], p[3], q[0], q[1], q[2], q[3]};
      const int i = first + (block * NT + tid) * 4;
      list_append(x, lo, list, cap, fill, [&](int c) { return i + (c >> 2) * 4 * NT + (c & 3); });
    };
    int block = 0;
    for (; block + AHEAD <= blocks; block += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; u += 2) {
        two_blocks(v[u], v[u + 1], block + u);
        v[u] = request(block + u + AHEAD);
        v[u + 1] = request(block + u + 1 + AHEAD);
      }
    }
    const f32x4_u none = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int u = 0; u < AHEAD - 1; u += 2)
      if (block + u < blocks) two_blocks(v[u], block + u + 1 < blocks ? v[u + 1] : none, block + u);
    if (rest0 < n) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        x[u] = rest0 + u * NT + tid < n ? rest[u] : -INFINITY;
        x[4 + u] = -INFINITY;
      }
      list_append(x, lo, list, cap, fill, [&](int u) { return first + rest0 + u * NT + tid; });
    }
  }
};

// The top k of a row of n elements from the list of those that reach br.lo into the bitmap sel (whose
// LDS is hist, cleared, before).  false: see above.
template <int NT>
__device__ __forceinline__ bool select_listed(const uint2* list, int listed, int cap, int n, int k, const Bracket& br,
                                              uint32_t* sel, TopkLds<NT>& L, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  int* hist = reinterpret_cast<int*>(sel);
  auto mark = [&](int e) { atomicOr(&sel[e >> 5], 1u << (e & 31)); };
  const float fine = fminf(fmaxf((float)kBins / (br.edge - br.lo), 1e-35f), 3e38f);   // entries above share the last bin
  if (listed < k || listed > cap) return false;
  int sure = 0;
  bool nan = false;
  for (int j0 = 0; j0 < listed; j0 += NT) {
    const int j = j0 + tid;
    const bool live = j < listed;
    const float x = live ? __uint_as_float(list[j].x) : 0.f;
    nan |= x != x;
    sure += __popcll(__builtin_amdgcn_ballot_w64(live && x >= br.hi));
    if (live && x < br.hi) atomicAdd(&hist[linear_bin(x, br.lo, fine)], 1);
  }
  if (nan) L.nan_seen = 1;
  if (lane == 0) L.wave_sure[wave] = sure;
  __syncthreads();
  if (L.nan_seen) return false;
  int total_sure;
  waves_before(L.wave_sure, NT / 64, &total_sure);
  int need = k - total_sure;
  if (need < 0) return false;
  find_threshold_bin_n<NT>(hist, max(need, 1), L.scan_scratch, L.thr, this_thread());
  const int b = need > 0 ? L.thr[0] : kBins;             // need == 0: the sure ones are all
  int few = need > 0 ? L.thr[2] : 0;
  // A crowded bin (the bracket of a row with far outliers is wide) is cut into 2048 finer ones.  rank of an
  // entry against the need-th: 2 above, 1 undecided, 0 below.
  const float from2 = br.lo + (float)b / fine, fine2 = fminf(fine * (float)kBins, 3e38f);
  int b2 = -1;
  auto side = [&](float x) {
    const int d = x >= br.hi ? kBins + 1 : linear_bin(x, br.lo, fine);
    if (d != b || b2 < 0) return d > b ? 2 : d == b ? 1 : 0;
    const int d2 = linear_bin(x, from2, fine2);
    return d2 > b2 ? 2 : d2 == b2 ? 1 : 0;
  };
  if (few > kFew) {
    need = L.thr[1];
    __syncthreads();
    clear_hist<NT>(hist);
    for (int j = tid; j < listed; j += NT) {
      const float x = __uint_as_float(list[j].x);
      if (side(x) == 1) atomicAdd(&hist[linear_bin(x, from2, fine2)], 1);
    }
    __syncthreads();
    find_threshold_bin_n<NT>(hist, need, L.scan_scratch, L.thr, 0, nullptr, this_thread());
    b2 = L.thr[0];
    few = L.thr[2];
  }
  need = L.thr[1];
  if (few > kFew) {
    // digits of the key, most significant first, then of the index, inverted so that a lower index ranks higher
    uint64_t prefix = 0;
    auto rank_of = [&](uint2 e) {
      return ((uint64_t)order_key(__uint_as_float(e.x)) << 20) | (uint64_t)(0xFFFFFu - e.y);
    };
#pragma unroll 1
    for (int shift = 41; shift >= -3; shift -= 11) {     // 52 bits: 11 at 41, 30, 19, 8 and the last 8
      const int low = max(shift, 0), bits = shift < 0 ? 11 + shift : 11;
      __syncthreads();
      clear_hist<NT>(hist);
      for (int j = tid; j < listed; j += NT) {
        const uint64_t r = rank_of(list[j]);
        if (side(__uint_as_float(list[j].x)) != 1) continue;
        if (low + bits == 52 || (r >> (low + bits)) == prefix) atomicAdd(&hist[(int)(r >> low) & ((1 << bits) - 1)], 1);
      }
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, L.scan_scratch, L.thr, 0, nullptr, this_thread());
      prefix = (prefix << bits) | (uint64_t)L.thr[0];
      need = L.thr[1];
    }
    for (int i = tid; i < (n + 31) >> 5; i += NT) sel[i] = 0;
    __syncthreads();
    for (int j = tid; j < listed; j += NT) {
      const int where = side(__uint_as_float(list[j].x));
      if (where == 2 || (where == 1 && rank_of(list[j]) >= prefix)) mark((int)list[j].y);
    }
    __syncthreads();
    return true;
  }
  for (int i = tid; i < (n + 31) >> 5; i += NT) sel[i] = 0;
  __syncthreads();
  for (int j0 = 0; j0 < listed; j0 += NT) {
    const int j = j0 + tid;
    const uint2 e = list[min(j, listed - 1)];
    const float x = __uint_as_float(e.x);
    const int where = j < listed ? side(x) : 0;
    if (where == 2) mark((int)e.y);
    const int at = wave_append(where == 1, &L.few_len);
    if (at >= 0) { L.fkey[at] = order_key(x); L.fidx[at] = (int)e.y; }
  }
  __syncthreads();
  {
    // all pairs, spread over the block: a wavefront compares each of the (at most 64) entries with its
    // share of the others (one thread per entry and a loop over the others took up to 7 us)
    constexpr int JP = kFew / (NT / 64);
    const int j0 = wave * JP;
    if (lane < few && j0 < few) {
      const uint32_t key = L.fkey[lane];
      const int e = L.fidx[lane];
      int part = 0;
#pragma unroll
      for (int j = j0; j < j0 + JP; ++j)
        part += (j < few && (L.fkey[j] > key || (L.fkey[j] == key && L.fidx[j] < e))) ? 1 : 0;
      if (part) atomicAdd(&L.frank[lane], part);
    }
  }
  __syncthreads();
  if (tid < few && L.frank[tid] < need) mark(L.fidx[tid]);
  __syncthreads();
  return true;
}

// The selected entries of the list in index order: the place of one is the number of selected elements in
// the bitmap words before its own (before[], 16 bits: k <= 16384) and below it in its word.
template <int NT>
__device__ __forceinline__ void write_listed(const uint2* list, int listed, int n, int k, const uint32_t* sel,
                                             uint16_t* before, int* scan_scratch, const int* __restrict__ map,
                                             int* __restrict__ out_idx, float* __restrict__ out_val, int tid) {
  const int nwords = (n + 31) / 32;
  const int wpt = (nwords + NT - 1) / NT;
  const int w_lo = min(tid * wpt, nwords), w_hi = min(w_lo + wpt, nwords);
  int cnt = 0;
  for (int w = w_lo; w < w_hi; ++w) cnt += __popc(sel[w]);
  int total;
  int pos = block_exclusive_scan(cnt, scan_scratch, &total);
  for (int w = w_lo; w < w_hi; ++w) {
    before[w] = (uint16_t)pos;
    pos += __popc(sel[w]);
  }
  __syncthreads();
  for (int j = tid; j < listed; j += NT) {
    const uint2 e = list[j];
    const uint32_t word = sel[e.y >> 5], bit = 1u << (e.y & 31);
    const int at = before[e.y >> 5] + __popc(word & (bit - 1u));
    if ((word & bit) && at < k) {     // at < k: always true when the selection is consistent
      out_idx[at] = map ? map[e.y] : (int)e.y;
      if (out_val) out_val[at] = __uint_as_float(e.x);
    }
  }
}

// ---------------------------------------------------------------- few long rows
// One workgroup per row would leave most of the chip idle, and a single CU needs longer to read a long
// row than the rest of the work takes.  Workgroup (range, t, seq) of this
// kernel finds the row's bracket from the sample, as every workgroup of the row does, and lists the
// elements of its key range that reach it in the range's segment of the workspace; topk_kernel<LISTED>
// selects from the segments of a row.
constexpr int kMaxRanges = 16;      // key ranges (workgroups) per row
constexpr int kSegCap = 6936;       // entries of a segment, behind them 64 of slack
constexpr int kSegInts = 64 + 2 * (kSegCap + 64);   // header (fill, or -1: no bracket; bracket at 8 .. 10), then entries

// Length of the key ranges a row of L elements is cut into (at most kMaxRanges of them).
__host__ __device__ inline int range_len(int L) {
  const int per = (L + kMaxRanges - 1) / kMaxRanges;
  return max((per + 4095) & ~4095, 8192);
}

__global__ __launch_bounds__(kTopkThreads) void topk_prefilter_kernel(Prob p, const float* __restrict__ S, int k,
                                                                      int rlen, int* __restrict__ pre) {
  constexpr int NT = kTopkThreads;
  __shared__ int hist[kBins];
  __shared__ TopkLds<NT> L;
  const int range = blockIdx.x, t = blockIdx.y, seq = blockIdx.z;
  const size_t row = (size_t)seq * p.n_q + t;
  const int n = visible(p, seq, t);
  const int lo = range * rlen, hi = min(lo + rlen, n);
  if (lo >= hi || k >= n) return;       // nothing here / every element is selected anyway
  const float* s = S + row * p.L;
  int* seg = pre + (row * gridDim.x + range) * kSegInts;
  float held[kHeldLong];
  Bracket br = {0.f, 0.f, 0.f};
  Stream<NT, 2> st;
  const bool ok = sample_bracket<NT, false>(s, n, p.L, k, held, hist, L, br, [&] { st.begin(s + lo, hi - lo, threadIdx.x); });
  if (ok) st.filter(br.lo, lo, reinterpret_cast<uint2*>(seg + 64), kSegCap, &L.list_fill);
  __syncthreads();
  if (threadIdx.x == 0) {
    seg[0] = ok ? L.list_fill : -1;
    seg[8] = __float_as_int(br.lo);
    seg[9] = __float_as_int(br.hi);
    seg[10] = __float_as_int(br.edge);
  }
}

// The segments of a row's ranges into the list; returns how many elements passed, or -1 if there is no
// bracket.  whole: no segment overflowed, nor the list.  Wavefront w takes range w.
__device__ __forceinline__ int gather_segments(const int* __restrict__ segs, int ranges, uint2* list, int cap, Bracket& br,
                                               bool& whole) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int cnt = lane < ranges ? segs[(size_t)lane * kSegInts] : 0;
  br.lo = __int_as_float(segs[8]);
  br.hi = __int_as_float(segs[9]);
  br.edge = __int_as_float(segs[10]);
  const int end = row16_inclusive_scan(cnt);             // (kMaxRanges = 16 lanes matter)
  const int total = __builtin_amdgcn_readlane(end, 15);
  whole = __ballot(cnt < 0 || cnt > kSegCap) == 0 && total <= cap;
  if (__ballot(cnt < 0) != 0) return -1;
  if (!whole) return total;
  if (wave < ranges) {
    const int mine = __builtin_amdgcn_readlane(cnt, wave), at = __builtin_amdgcn_readlane(end, wave) - mine;
    const uint2* src = reinterpret_cast<const uint2*>(segs + (size_t)wave * kSegInts + 64);
    for (int j0 = lane; j0 < mine; j0 += 512) {
      uint2 e[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) e[u] = src[min(j0 + 64 * u, mine - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (j0 + 64 * u < mine) list[at + j0 + 64 * u] = e[u];
    }
  }
  return total;
}

// ---------------------------------------------------------------- per-row kernel
enum { kRowShort, kRowLong, kRowListed, kRowPlain };   // held in registers / streamed / listed by topk_prefilter_kernel / two passes

// The `need` lowest-index elements of the bitmap eq into sel (words are owned by one thread here).
template <int NT>
__device__ __forceinline__ void mark_lowest(const uint32_t* eq, uint32_t* sel, int nwords, int need, int* scan_scratch) {
  const int tid = this_thread();
  const int wpt = (nwords + NT - 1) / NT;
  const int w_lo = min(tid * wpt, nwords), w_hi = min(w_lo + wpt, nwords);
  int cnt = 0;
  for (int w = w_lo; w < w_hi; ++w) cnt += __popc(eq[w]);
  int total;
  int before = block_exclusive_scan(cnt, scan_scratch, &total);
  for (int w = w_lo; w < w_hi && before < need; ++w) {
    uint32_t bits = eq[w];
    const int c = __popc(bits);
    int take = min(c, need - before);
    before += c;
    uint32_t kept = 0;
    if (take == c) kept = bits;
    else
      while (take-- > 0) {
        const uint32_t low = bits & (0u - bits);
        kept |= low;
        bits ^= low;
      }
    sel[w] |= kept;
  }
  __syncthreads();
}

// The marked elements of a row in index order.
template <int NT>
__device__ __forceinline__ void write_marked(const float* __restrict__ s, int n, int k, const uint32_t* sel, int* scan_scratch,
                                             const int* __restrict__ map, int* __restrict__ out_idx, float* __restrict__ out_val) {
  const int tid = this_thread(), nwords = (n + 31) / 32;
  const int wpt = (nwords + NT - 1) / NT;
  const int w_lo = min(tid * wpt, nwords), w_hi = min(w_lo + wpt, nwords);
  int cnt = 0;
  for (int w = w_lo; w < w_hi; ++w) cnt += __popc(sel[w]);
  int total;
  int pos = block_exclusive_scan(cnt, scan_scratch, &total);
  for (int w = w_lo; w < w_hi; ++w) {
    uint32_t bits = sel[w];
    while (bits) {
      const int i = w * 32 + __ffs(bits) - 1;
      bits &= bits - 1;
      if (pos < k) {  // always true when the selection is consistent
        out_idx[pos] = map ? map[i] : i;
        if (out_val) out_val[pos] = s[i];
      }
      ++pos;
    }
  }
}

// The top k of a row by the radix select on the row itself.  skip_lowest: -inf is never selected.
template <int NT>
__device__ __forceinline__ void two_pass_row(const float* __restrict__ s, int n, int row_len, int k, const int* __restrict__ map,
                                             int* __restrict__ out_idx, float* __restrict__ out_val, int list_cap,
                                             bool skip_lowest, uint32_t* dyn, TopkLds<NT>& L) {
  // dyn: sel bitmap, histogram, then eq bitmap OR list (keys, idx)
  int* const scan_scratch = L.scan_scratch;
  int* const thr = L.thr;
  const int tid = this_thread();
  uint32_t* sel = dyn;
  uint32_t* region = dyn + sel_words(row_len);
  int* hist = reinterpret_cast<int*>(region);
  uint32_t* eq = region + kBins;
  uint32_t* lkey = region + kBins;       // (aliases eq)
  int* lidx = reinterpret_cast<int*>(lkey + list_cap);
  const int nwords = (n + 31) / 32;
  for (int i = tid; i < nwords; i += NT) sel[i] = 0;
  if (tid == 0) { L.list_fill = 0; L.few_len = 0; }
  clear_hist<NT>(hist);
  if (k < n || skip_lowest) {   // otherwise every element is selected
    // ---- pass 1: histogram of the top 11 bits
    scan_row<NT>(s, 0, n, [&](int, float v, bool in) {
      if (in) atomicAdd(&hist[order_key(v) >> 21], 1);
    });
    __syncthreads();
  }

  int selectable = n;
  if (skip_lowest) {  // never select -inf slots (skipped candidates): they live in bins <= 3
    selectable = n - (hist[0] + hist[1] + hist[2] + hist[3]);
  }
  const int k_eff = min(k, selectable);
  for (int i = k_eff + tid; i < k; i += NT) {
    out_idx[i] = -1;
    if (out_val) out_val[i] = -INFINITY;
  }
  if (k_eff == 0) return;

  if (k_eff == n) {
    for (int i = tid; i < nwords; i += NT) {
      const int rem = n - i * 32;
      sel[i] = rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
    }
    __syncthreads();
  } else {
    find_threshold_bin_n<NT>(hist, k_eff, scan_scratch, thr, 0, nullptr, this_thread());
    const uint32_t d1 = thr[0];
    int need = thr[1];
    const bool listed = thr[2] <= list_cap;
    __syncthreads();
    clear_hist<NT>(hist);

    if (listed) {
      // ---- pass 2: mark digit1 > d1, compact digit1 == d1 into the LDS list
      scan_row<NT>(s, 0, n, [&](int i, float v, bool in) {
        const uint32_t key = order_key(v), a = key >> 21;
        if (in && a > d1) atomicOr(&sel[i >> 5], 1u << (i & 31));
        const int b = wave_append(in && a == d1, &L.list_fill);
        if (b >= 0) { lkey[b] = key; lidx[b] = i; }
      });
      __syncthreads();
      const int len = L.list_fill;
      // ---- digits 2 and 3 on the list
      for (int i = tid; i < len; i += NT) atomicAdd(&hist[(lkey[i] >> 10) & 0x7FF], 1);
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
      const uint32_t p22 = (d1 << 11) | (uint32_t)thr[0];
      need = thr[1];
      const int nb = thr[2];
      if (nb <= kFew) {
        // ---- few list entries share the second threshold digit (the usual case): they are
        //      ranked against each other by score, then index, instead of a third digit pass
        for (int i = tid; i < len; i += NT) {
          const uint32_t key = lkey[i], kp = key >> 10;
          if (kp > p22) atomicOr(&sel[lidx[i] >> 5], 1u << (lidx[i] & 31));
          const int b = wave_append(kp == p22, &L.few_len);
          if (b >= 0) { L.fkey[b] = key; L.fidx[b] = lidx[i]; }
        }
        __syncthreads();
        if (tid < nb) {
          const uint32_t key = L.fkey[tid];
          const int e = L.fidx[tid];
          int rank = 0;
          for (int j = 0; j < nb; ++j) {
            const uint32_t kj = L.fkey[j];
            rank += (kj > key || (kj == key && L.fidx[j] < e)) ? 1 : 0;
          }
          if (rank < need) atomicOr(&sel[e >> 5], 1u << (e & 31));
        }
      } else {
      __syncthreads();
      clear_hist<NT>(hist);
      for (int i = tid; i < len; i += NT) {
        const uint32_t key = lkey[i], kp = key >> 10;
        if (kp > p22) atomicOr(&sel[lidx[i] >> 5], 1u << (lidx[i] & 31));
        else if (kp == p22) atomicAdd(&hist[key & 0x3FF], 1);
      }
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
      const uint32_t tkey = (p22 << 10) | (uint32_t)thr[0];
      need = thr[1];
      const int ties = thr[2];
      __syncthreads();
      clear_hist<NT>(hist);
      if (ties == need) {
        for (int i = tid; i < len; i += NT)
          if (lkey[i] >= tkey) atomicOr(&sel[lidx[i] >> 5], 1u << (lidx[i] & 31));
      } else {
        // More ties than places: take the `need` lowest indices among them, by the
        // same digit search on (high, low) halves of the index, inverted so that a
        // lower index ranks higher.  Indices are distinct, so this is exact.
        for (int i = tid; i < len; i += NT) {
          const uint32_t key = lkey[i];
          if (key > tkey) atomicOr(&sel[lidx[i] >> 5], 1u << (lidx[i] & 31));
          else if (key == tkey) atomicAdd(&hist[kBins - 1 - (lidx[i] >> 10)], 1);
        }
        __syncthreads();
        find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
        const int hi_digit = kBins - 1 - thr[0];
        need = thr[1];
        __syncthreads();
        clear_hist<NT>(hist);
        for (int i = tid; i < len; i += NT) {
          if (lkey[i] != tkey) continue;
          const int e = lidx[i];
          if ((e >> 10) < hi_digit) atomicOr(&sel[e >> 5], 1u << (e & 31));
          else if ((e >> 10) == hi_digit) atomicAdd(&hist[kBins - 1 - (e & 0x3FF)], 1);
        }
        __syncthreads();
        find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
        const int lo_digit = kBins - 1 - thr[0];
        for (int i = tid; i < len; i += NT) {
          if (lkey[i] != tkey) continue;
          const int e = lidx[i];
          if ((e >> 10) == hi_digit && (e & 0x3FF) <= lo_digit) atomicOr(&sel[e >> 5], 1u << (e & 31));
        }
      }
      }  // more than kFew entries in the second digit
      __syncthreads();
    } else {
      // ---- fallback: two more digit passes over the row, ties through a bitmap
      for (int i = tid; i < nwords; i += NT) eq[i] = 0;
      __syncthreads();
      scan_row<NT>(s, 0, n, [&](int i, float v, bool in) {
        const uint32_t key = order_key(v), a = key >> 21;
        if (!in) return;
        if (a > d1) atomicOr(&sel[i >> 5], 1u << (i & 31));
        else if (a == d1) atomicAdd(&hist[(key >> 10) & 0x7FF], 1);
      });
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
      const uint32_t d2 = thr[0];
      need = thr[1];
      __syncthreads();
      clear_hist<NT>(hist);
      const uint32_t pre22 = (d1 << 11) | d2;
      scan_row<NT>(s, 0, n, [&](int i, float v, bool in) {
        const uint32_t key = order_key(v);
        if (!in || (key >> 21) != d1) return;
        const uint32_t b = (key >> 10) & 0x7FF;
        if (b > d2) atomicOr(&sel[i >> 5], 1u << (i & 31));
        else if (b == d2) atomicAdd(&hist[key & 0x3FF], 1);
      });
      __syncthreads();
      find_threshold_bin_n<NT>(hist, need, scan_scratch, thr, 0, nullptr, this_thread());
      const uint32_t tkey = (pre22 << 10) | (uint32_t)thr[0];
      need = thr[1];  // how many elements equal to the threshold value are taken
      __syncthreads();
      scan_row<NT>(s, 0, n, [&](int i, float v, bool in) {
        const uint32_t key = order_key(v);
        if (!in || (key >> 10) != pre22) return;
        if (key > tkey) atomicOr(&sel[i >> 5], 1u << (i & 31));
        else if (key == tkey) atomicOr(&eq[i >> 5], 1u << (i & 31));
      });
      __syncthreads();
      mark_lowest<NT>(eq, sel, nwords, need, scan_scratch);
    }
  }
  write_marked<NT>(s, n, k, sel, scan_scratch, map, out_idx, out_val);
}

struct TopkArgs {
  Prob p;
  const float* S;
  int row_len, k;
  const int* map;
  int* idx;
  float* val;
  const int* pre;
  int cap, list_cap;
  bool all_slots;
};
struct TopkRow {   // a workgroup's row
  const float* s;
  int n;
  const int* map;
  int* idx;
  float* val;
};
__device__ __forceinline__ TopkRow topk_row_of(const TopkArgs& a) {
  // queries in descending order: under a causal mask the late ones have the longest rows, and
  // the workgroups with the most work should start first
  const int t = gridDim.x - 1 - blockIdx.x, seq = blockIdx.y;
  const size_t row = (size_t)seq * a.p.n_q + t;
  return {a.S + row * a.row_len, a.map || a.all_slots ? a.row_len : visible(a.p, seq, t),
          a.map ? a.map + row * a.row_len : nullptr, a.idx + row * a.k, a.val ? a.val + row * a.k : nullptr};
}

// The kernel's arguments once more, through an address that the compiler knows nothing of: kept in registers for
// hard_row, they cost the rows that do not need it, and between its stages they cost spills.
__device__ __forceinline__ const TopkArgs& kernel_args() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const TopkArgs*)p;
}

// A row that the linear bracket did not do (a stage of topk_kernel, whose arguments it reads).  passed: elements that
// reached the lower end of the first bracket, -1: it had none, -2: not worth another.
template <int NT>
__device__ __forceinline__ void hard_row(int passed, uint32_t* dyn, TopkLds<NT>& L) {
  uint32_t* sel = dyn;
  int* sample_hist = reinterpret_cast<int*>(sel);
  Found found = kNoBracket;
  Bracket br;
  auto write = [&](int listed) {
    const TopkArgs& a = kernel_args();
    const TopkRow r = topk_row_of(a);
    const uint2* list = reinterpret_cast<uint2*>(dyn + sel_words(a.row_len));
    uint16_t* before = reinterpret_cast<uint16_t*>(dyn + sel_words(a.row_len) + 2 * (a.cap + 64));
    write_listed<NT>(list, listed, r.n, a.k, sel, before, L.scan_scratch, r.map, r.idx, r.val, this_thread());
  };
  if (passed >= -1 && kernel_args().k < topk_row_of(kernel_args()).n) {
    // where a list was not usable: the rank that would have listed a number between k and the capacity
    auto aim = [&](int passed) {
      const TopkArgs& a = kernel_args();
      return 0.5f * (float)(a.k + a.cap) / (float)max(passed, 1);
    };
    float adjust = passed < 0 ? 0.f : aim(passed);
#pragma unroll 1
    for (int attempt = 0; attempt < kAttempts; ++attempt) {
      __syncthreads();
      {
        // adjust > 0: the lower end is the sample of adjust times the rank, the upper end is open
        const TopkArgs& a = kernel_args();
        const TopkRow r = topk_row_of(a);
        const int tid = this_thread();
        float held[held_hard(NT)];
        Sample sm = take_sample<NT, false>(r.s, r.n, a.row_len, a.k, tid, held, [] {});
        if (tid == 0) { L.few_len = 0; L.nan_seen = 0; L.list_fill = 0; }
        if (tid < kFew) L.frank[tid] = 0;
        if (adjust > 0.f) {
          sm.r_lo = (int)ceilf(fminf((float)sm.r_lo * adjust, 1e6f));
          sm.r_hi = 0;
          sm.rank_up = max(sm.r_lo / 16, 1);
        }
        found = key_bracket<NT>(a.cap, sm, held, sample_hist, L, br);
      }
      if (found != kBracket) break;
      const TopkArgs& a = kernel_args();
      const TopkRow r = topk_row_of(a);
      const int k = a.k, cap = a.cap;
      uint2* list = reinterpret_cast<uint2*>(dyn + sel_words(a.row_len));
      Stream<NT, 2> st;
      st.begin(r.s, r.n, this_thread());
      st.filter(br.lo, 0, list, cap, &L.list_fill);
      __syncthreads();
      const int listed = L.list_fill;
      if (select_listed<NT>(list, listed, cap, r.n, k, br, sel, L, this_thread())) {
        write(listed);
        return;
      }
      if (listed >= k && listed <= cap) {
        if (L.nan_seen || adjust > 0.f) break;           // (adjust: more than k infinite entries)
        adjust = 1.f;
        continue;
      }
      adjust = (adjust > 0.f ? adjust : 1.f) * aim(listed);
    }
  }
  // ---- the k-th largest is one of many equal values: marked from the ballots of one more pass, the counts prove it
  // (2048 rows of 65536, 99.5 % zeros: 1960 us when they were left to the two-pass path)
  if (found == kPlateau) {
    const TopkArgs& a = kernel_args();
    const TopkRow r = topk_row_of(a);
    const float* s = r.s;
    const int n = r.n, k = a.k, nwords = (n + 31) / 32, tid = this_thread();
    uint32_t* region = dyn + sel_words(a.row_len);
    uint32_t* eq = region + kBins;
    const uint32_t level = order_key(br.lo);
    int above = 0, equal = 0;
    __syncthreads();
    scan_row<NT, 4>(s, 0, n, [&](int i, float v, bool in) {
      const uint32_t key = order_key(v);
      const unsigned long long more = __builtin_amdgcn_ballot_w64(in && key > level), same = __builtin_amdgcn_ballot_w64(in && key == level);
      const int lane = tid & 63, w = ((i - lane) >> 5) + lane;
      if (lane < 2 && w < nwords) {
        sel[w] = (uint32_t)(lane ? more >> 32 : more);
        eq[w] = (uint32_t)(lane ? same >> 32 : same);
      }
      above += __popcll(more);
      equal += __popcll(same);
    });
    if ((tid & 63) == 0) { L.wave_sure[tid >> 6] = above; L.wave_more[tid >> 6] = equal; }
    __syncthreads();
    waves_before(L.wave_sure, NT / 64, &above);
    waves_before(L.wave_more, NT / 64, &equal);
    if (above < k && above + equal >= k) {
      mark_lowest<NT>(eq, sel, nwords, k - above, L.scan_scratch);
      write_marked<NT>(s, n, k, sel, L.scan_scratch, r.map, r.idx, r.val);
      return;
    }
    if (above >= k && above <= a.cap) {
      // the plateau ends above the k-th largest: what lies above it is the list
      uint2* list = reinterpret_cast<uint2*>(region);
      const int wpt = (nwords + NT - 1) / NT;
      const int w_lo = min(tid * wpt, nwords), w_hi = min(w_lo + wpt, nwords);
      int cnt = 0, total;
      for (int w = w_lo; w < w_hi; ++w) cnt += __popc(sel[w]);
      int pos = block_exclusive_scan(cnt, L.scan_scratch, &total);
      for (int w = w_lo; w < w_hi; ++w)
        for (uint32_t bits = sel[w]; bits; bits &= bits - 1) {
          const int i = w * 32 + __ffs(bits) - 1;
          list[pos++] = make_uint2(__float_as_uint(s[i]), (uint32_t)i);
        }
      __syncthreads();
      clear_hist<NT>(sample_hist);
      br.lo = key_value(level + 1);
      br.hi = INFINITY;
      br.edge = fmaxf(br.edge, key_value(level + 2));
      if (select_listed<NT>(list, above, a.cap, n, k, br, sel, L, this_thread())) {
        write(above);
        return;
      }
    }
  }
  __syncthreads();
  const TopkArgs& a = kernel_args();
  const TopkRow r = topk_row_of(a);
  two_pass_row<NT>(r.s, r.n, a.row_len, a.k, r.map, r.idx, r.val, a.list_cap, a.map || a.all_slots, dyn, L);
}

template <int NT, int KIND>
__device__ __forceinline__ void topk_row(const TopkArgs& a, uint32_t* dyn) {
  // dyn: sel bitmap (sampled path: and its histograms), then the list of the sampled path, or the two-pass
  // path's histogram and its eq bitmap OR list (keys, idx)
  __shared__ TopkLds<NT> L;

  const int tid = threadIdx.x;
  const TopkRow r = topk_row_of(a);
  const float* s = r.s;
  const int n = r.n, row_len = a.row_len, k = a.k, cap = a.cap;
  const bool all = !a.map && !a.all_slots;   // -inf may be selected
  uint32_t* sel = dyn;
  uint2* list = reinterpret_cast<uint2*>(dyn + sel_words(row_len));
  int passed = -1;

  if (k >= n && all) {   // every element
    for (int i = tid; i < k; i += NT) {
      r.idx[i] = i < n ? i : -1;
      if (r.val) r.val[i] = i < n ? s[i] : -INFINITY;
    }
    return;
  }
  if constexpr (KIND == kRowPlain) {
    two_pass_row<NT>(s, n, row_len, k, r.map, r.idx, r.val, a.list_cap, !all, dyn, L);
    return;
  } else if (k < n) {
    bool done = false;
    uint16_t* before = reinterpret_cast<uint16_t*>(list + cap + 64);
    int* sample_hist = reinterpret_cast<int*>(sel);
    Bracket br;
    if constexpr (KIND == kRowListed) {
      const int rlen = range_len(row_len), ranges_row = (row_len + rlen - 1) / rlen;
      for (int i = tid; i < kBins; i += NT) sample_hist[i] = 0;
      if (tid == 0) { L.few_len = 0; L.nan_seen = 0; }
      if (tid < kFew) L.frank[tid] = 0;
      bool whole;
      passed = gather_segments(a.pre + ((size_t)blockIdx.y * a.p.n_q + (gridDim.x - 1 - blockIdx.x)) * ranges_row * kSegInts, (n + rlen - 1) / rlen, list, cap, br, whole);
      __syncthreads();
      if (whole) done = select_listed<NT>(list, passed, cap, n, k, br, sel, L, tid);
      // (a segment overflowed that the list will hold, or sure > k: the same lower end once more, the upper end open)
      if (!done && passed >= k && passed <= cap) passed = whole && L.nan_seen ? -2 : (k + cap) / 2;
    } else if constexpr (KIND == kRowShort) {
      float held[held_short(NT)];
      if (sample_bracket<NT, true>(s, n, row_len, k, held, sample_hist, L, br, [] {})) {
#pragma unroll
        for (int u = 0; u < held_short(NT); u += 8) {
          float x[8];
#pragma unroll
          for (int c = 0; c < 8; ++c) x[c] = held[u + c];
          list_append(x, br.lo, list, cap, &L.list_fill, [&](int c) { return (u + c) * NT + tid; });
        }
        __syncthreads();
        passed = L.list_fill;
        done = select_listed<NT>(list, passed, cap, n, k, br, sel, L, tid);
        if (!done && passed >= k && passed <= cap) passed = L.nan_seen ? -2 : (k + cap) / 2;
      }
    } else {
      float held[kHeldLong];
      Stream<NT, NT == kTopkThreads ? 4 : 6> st;         // (64 registers: 32 wavefronts per CU; 80: 24)
      if (sample_bracket<NT, false>(s, n, row_len, k, held, sample_hist, L, br, [&] { st.begin(s, n, tid); })) {
        st.filter(br.lo, 0, list, cap, &L.list_fill);
        __syncthreads();
        passed = L.list_fill;
        done = select_listed<NT>(list, passed, cap, n, k, br, sel, L, tid);
        if (!done && passed >= k && passed <= cap) passed = L.nan_seen ? -2 : (k + cap) / 2;
      }
    }
    if (done) {
      const TopkArgs& b = kernel_args();
      const TopkRow w = topk_row_of(b);
      write_listed<NT>(list, passed, n, k, sel, before, L.scan_scratch, w.map, w.idx, w.val, tid);
      return;
    }
  }
  if constexpr (KIND != kRowPlain) hard_row<NT>(passed, dyn, L);
}

// Registers: 1024 threads leave room for two workgroups per CU, the smaller ones for 24 wavefronts.
template <int NT, int KIND>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == kTopkThreads ? 8 : 6, 8))) void topk_kernel(TopkArgs a) {
  extern __shared__ __align__(16) uint32_t dyn[];
  topk_row<NT, KIND>(a, dyn);
}

// Only the rows r with only[r] != 0 (rows another path could not finish).  Normally
// there is none, so a small grid strides over the rows.
__global__ __launch_bounds__(kTopkThreads) void topk_only_kernel(Prob p, const float* __restrict__ S,
                                                                 int k, int* __restrict__ idx,
                                                                 float* __restrict__ val, int list_cap,
                                                                 const int* __restrict__ only) {
  extern __shared__ __align__(16) uint32_t dyn[];
  __shared__ TopkLds<kTopkThreads> L;
  const int rows = p.n_seq * p.n_q;
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    if (!only[r]) continue;
    const size_t row = r;
    two_pass_row<kTopkThreads>(S + row * p.L, visible(p, r / p.n_q, r % p.n_q), p.L, k, nullptr, idx + row * k,
                               val ? val + row * k : nullptr, list_cap, false, dyn, L);
    __syncthreads();
  }
}

// Rows are cut into ranges where there are fewer rows than CUs and the rows are long, whatever k is (us, one launch /
// two: 65536 elements, k = 2048 17.0 / 15.8, k = 8192 21.1 / 22.0 and 128 rows of it 22.9 / 39.9; 100003, k = 2048
// 20.9 / 17.0; 131072, k = 8192 28.0 / 23.4).
static bool use_split(const Prob& p) {
  return (long long)p.n_seq * p.n_q < 256 && p.L > 65536;
}

size_t topk_ws_bytes(const Prob& p, int k) {
  if (!use_split(p) || k < 1) return 0;
  const int rlen = range_len(p.L);
  return (size_t)p.n_seq * p.n_q * ((p.L + rlen - 1) / rlen) * kSegInts * sizeof(int);
}

// List entries of a row.  With one line of every ls sampled, about r_lo ls elements of the row reach the
// lower end of sample_bracket (r_lo = k / ls + 6 sqrt(k / ls) + 8) and the number scatters by
// ls sqrt(r_lo): `sd` of those are added, also for a row that ends early, whose ls is no larger.  A short row
// lists little more than k.
static int pass_capacity(int row_len, int k, int nt, bool is_short, double sd) {
  const int lines = (row_len + 15) / 16, max_lines = is_short ? lines : sample_lines(row_len, row_len, k, nt);
  const double ls = (lines + max_lines - 1) / max_lines, kf = k / ls;
  const double r = kf + 6.0 * std::sqrt(kf) + 8.0;
  return std::min((int)(ls * (r + (ls > 1 ? sd * std::sqrt(r) : 56.0))), row_len);
}

hipError_t launch_topk(const Prob& p, const float* S, int row_len, int k, const int* map, int* idx,
                       float* val, void* ws, hipStream_t st, const int* only, bool all_slots) {
  // Short rows: as many threads as hold the row; few rows of up to 4096 take 512 threads (7.3 us for one
  // row against 9.3 us with 256).  Long rows: 1024 threads where there is at most one row per CU or the lists are
  // long; more rows with shorter lists take 512, of which a CU holds
  // three at different phases, so that memory is never idle (4096 x 65536: 212 us against 244 us).  Less than two rows
  // per CU: 512 threads, two rows per CU, up to 45056 elements (us, 1024 / 512: 333 x 10007 17.8 / 14.6, 400 x 20000
  // 19.2 / 17.1, 428 x 42624 24.7 / 23.0, 433 x 43590 23.7 / 23.9); beyond, a row that needs a second look takes too long
  // (490 x 118413 with scores alike in runs 63 / 74, 263 x 100783 on a plateau 101 / 114, 286 x 115232 Gaussian 40.5 / 41.8).
  constexpr size_t kLdsMost = 156 * 1024;
  const bool is_short = !only && row_len <= 8192;
  const bool split = !map && !all_slots && !only && use_split(p);
  size_t lds = 0;
  int cap = 0;
  auto fits = [&](int nt, size_t most, double sd = 6.0) {
    cap = pass_capacity(row_len, k, nt, is_short, sd);
    lds = (size_t)sel_words(row_len) * 4 + (size_t)(cap + 64) * 8 + (size_t)((row_len + 31) / 32) * 2;
    return lds <= most;
  };
  const long long rows = (long long)p.n_q * p.n_seq;
  const bool few_rows = rows < 256, one_set = rows < 512;
  int nt = row_len > 4096 ? kTopkThreads : few_rows ? 512 : 256;
  if (is_short) fits(nt, kLdsMost);
  else if (only) nt = kTopkThreads;
  else if (split || few_rows || (one_set && row_len > 45056) || !fits(nt = 512, one_set ? 76 * 1024 : 53 * 1024)) {
    nt = kTopkThreads;
    // the longest rows have room for half the reserve; k well above 8192: the two-pass path
    if (!fits(nt, kLdsMost) && !fits(nt, kLdsMost, 3.0)) cap = 0;
  }
  // the two-pass path shares the region: histogram and list, or a second bitmap
  const int list_cap = std::min(row_len, is_short || nt == 512 ? std::max((int)(lds / 8) - sel_words(row_len) / 2 - kBins / 2, 1) : kListTarget);
  const size_t words = (size_t)sel_words(row_len);
  lds = std::max(cap ? lds : 0, words * 4 + kBins * 4 + std::max((size_t)list_cap * 8, (size_t)((row_len + 31) / 32) * 4));
  const dim3 grid(p.n_q, p.n_seq);
  hipError_t e;
  int* pre = split && cap ? static_cast<int*>(ws) : nullptr;
#define GO(NT, KIND)                                                                               \
  do {                                                                                             \
    static LdsSeen seen;                                                                           \
    e = ensure_dynamic_lds(reinterpret_cast<const void*>(topk_kernel<NT, KIND>), lds, seen);       \
    if (e != hipSuccess) return e;   /* before the first launch: a failure leaves nothing enqueued */ \
    if (KIND == kRowListed) {                                                                      \
      const int rlen = range_len(p.L);                                                             \
      const dim3 ranges((p.L + rlen - 1) / rlen, p.n_q, p.n_seq);                                  \
      topk_prefilter_kernel<<<ranges, kTopkThreads, 0, st>>>(p, S, k, rlen, pre);                 \
    }                                                                                              \
    topk_kernel<NT, KIND><<<grid, NT, lds, st>>>(TopkArgs{p, S, row_len, k, map, idx, val, pre, cap, list_cap, all_slots}); \
  } while (0)
  if (only) {
    static LdsSeen seen;
    e = ensure_dynamic_lds(reinterpret_cast<const void*>(topk_only_kernel), lds, seen);
    if (e != hipSuccess) return e;
    topk_only_kernel<<<(unsigned)std::min<long long>(rows, 256), kTopkThreads, lds, st>>>(p, S, k, idx, val, list_cap, only);
  } else if (is_short && nt == 256) {
    GO(256, kRowShort);
  } else if (is_short && nt == 512) {
    GO(512, kRowShort);
  } else if (is_short) {
    GO(kTopkThreads, kRowShort);
  } else if (nt == 512) {
    GO(512, kRowLong);
  } else if (cap == 0) {
    GO(kTopkThreads, kRowPlain);
  } else if (pre) {
    GO(kTopkThreads, kRowListed);
  } else {
    GO(kTopkThreads, kRowLong);
  }
#undef GO
  return hipGetLastError();
}

}  // namespace misa
