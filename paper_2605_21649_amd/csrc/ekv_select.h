// Exact k-th-largest selection and order-preserving compaction over the pages of one
// (sequence, query head), shared by the top-k and the Gaussian-aware selectors.
//
// One 1024-thread workgroup.  Keys are order-preserving uint32 images of float scores.  Wavefront w owns
// the contiguous page range [w*64*items, (w+1)*64*items) and lane l holds pages w*64*items + i*64 + l,
// i < items: loads are coalesced, keys can live in registers for all passes, and (w, i, l) order is
// ascending page order, so ballots give an ordered compaction without sorting.
#pragma once
#include "ekv_device.h"

namespace ekv {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kRankMax = 256;             // elements ranked directly once the radix passes have narrowed to so few

struct SelectShared {
  uint32_t hist[kBins];
  uint32_t list[kRankMax];                // keys that are ranked against each other
  int scan_buf[kSelWaves + 1];
  int wave_total[2][kSelWaves];
  uint32_t red_lo[kSelWaves], red_hi[kSelWaves];
  uint32_t few_lo[kSelWaves], few_hi[kSelWaves];
  int wave_gt[kSelWaves], wave_eq[kSelWaves];
  uint32_t digit, above;
  int n_list;
};
static_assert(kSelWaves == 16, "one value per wavefront is one DPP row");
static_assert(4 * kRankMax <= kSelThreads, "four lanes per ranked key");

// Keys of one (b,h) row.  ITEMS > 0: held in registers (M <= 1024*ITEMS); ITEMS == 0: recomputed from
// memory on every access (any M).  `fn(p)` gives the key of page p.  Slots past M hold the value 0, in registers no other does.
// After rebase(kmin) every key is stored relative to kmin (so only one register array is live).
template <int ITEMS, typename KeyFn>
struct KeySet {
  KeyFn fn;
  int M, items, page0;                      // page0 = first page of this lane
  uint32_t base;                            // subtracted from every key
  uint32_t reg[ITEMS ? ITEMS : 1];
  __device__ __forceinline__ KeySet(KeyFn f, int M_) : fn(f), M(M_), base(0u) {
    items = ITEMS ? ITEMS : (M + kSelThreads - 1) / kSelThreads;
    page0 = (threadIdx.x >> 6) * 64 * items + (threadIdx.x & 63);
    if (ITEMS) {
      // unconditional loads from clamped pages (a load inside a divergent branch is waited for at
      // once, which would serialise all ITEMS loads), masked afterwards
#pragma unroll
      for (int i = 0; i < (ITEMS ? ITEMS : 1); ++i) reg[i] = fn(min(page(i), M - 1));
#pragma unroll
      for (int i = 0; i < (ITEMS ? ITEMS : 1); ++i) reg[i] = page(i) < M ? reg[i] : 0u;
    }
  }
  __device__ __forceinline__ int page(int i) const { return page0 + i * 64; }
  __device__ __forceinline__ bool valid(int i) const { return page(i) < M; }
  // key of slot i relative to `base`; slots past M (and keys below base) give 0
  __device__ __forceinline__ uint32_t key(int i) const {
    if (ITEMS) return reg[i];
    const uint32_t k0 = fn(min(page(i), M - 1));
    const uint32_t k = page(i) < M ? k0 : 0u;
    return max(k, base) - base;
  }
  // ITEMS == 0: the keys of slots i0 .. i0+7, all eight loads issued before any is used (a loop that calls
  // key(i) once per iteration waits for memory in every iteration).  Slots i >= items belong to the NEXT
  // wavefront's pages: the caller must skip them (i0 + j < items), not only pages >= M.
  __device__ __forceinline__ void key_batch(int i0, uint32_t (&k)[8]) const {
    uint32_t k0[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) k0[j] = fn(min(page(i0 + j), M - 1));
#pragma unroll
    for (int j = 0; j < 8; ++j) k[j] = max(page(i0 + j) < M ? k0[j] : 0u, base) - base;
  }
  __device__ __forceinline__ void rebase(uint32_t kmin) {
    base = kmin;
    if (ITEMS) {
#pragma unroll
      for (int i = 0; i < (ITEMS ? ITEMS : 1); ++i) reg[i] = max(reg[i], kmin) - kmin;
    }
  }
};

// The digit of the histogram that holds the k_rem-th largest element, and how many lie above it (sh.digit, sh.above).
__device__ __forceinline__ void find_digit(int k_rem, int pass, SelectShared& sh) {
  const int tid = threadIdx.x;
  // thread t owns digits (kBins-1-2t) and (kBins-2-2t): scan from the top digit downwards
  const int d_hi = kBins - 1 - 2 * tid, d_lo = d_hi - 1;
  const int c_hi = (int)sh.hist[d_hi], c_lo = (int)sh.hist[d_lo];
  const int inc = wave_incl_scan_i(c_hi + c_lo);
  int* totals = sh.wave_total[pass & 1];
  if ((tid & 63) == 63) totals[tid >> 6] = inc;
  __syncthreads();
  const int above = row16_sum_i((tid & 15) < (tid >> 6) ? totals[tid & 15] : 0) + inc - c_hi - c_lo;
  if (above < k_rem && k_rem <= above + c_hi) { sh.digit = d_hi; sh.above = above; }
  else if (above + c_hi < k_rem && k_rem <= above + c_hi + c_lo) { sh.digit = d_lo; sh.above = above + c_hi; }
  __syncthreads();
}
// The k_rem-th largest of the keys in sh.list, and how many lie above it (sh.digit, sh.above).
__device__ __forceinline__ void rank_list(int members, int k_rem, SelectShared& sh) {
  // four lanes per member
  const int tid = threadIdx.x, mem = tid >> 2;
  const uint32_t v = sh.list[min(mem, members - 1)];
  int g = 0, e = 0;
  for (int j = tid & 3; j < members; j += 4) { const uint32_t u = sh.list[j]; g += u > v; e += u == v; }
  g += dpp_move_i<0xB1>(g); g += dpp_move_i<0x4E>(g);
  e += dpp_move_i<0xB1>(e); e += dpp_move_i<0x4E>(e);
  if (mem < members && g < k_rem && k_rem <= g + e) { sh.digit = v; sh.above = (uint32_t)g; }    // equal keys write the same
  __syncthreads();
}

// Scores on both sides of zero (a last page of one or two tokens is enough): their keys span most of the 32 bits, so that a
// digit of the first pass is a quarter of an octave and holds hundreds of scores.  One histogram over equal steps of the
// scores lo..hi themselves finds the k-th among a few.  True: key_t is the k-th largest key, k_rem how many equal to it are taken.
// False: the step with the k-th holds more than kRankMax scores; lo, hi and k_rem are narrowed to that step, the histogram
// and the list's counter are cleared, and the radix passes go on inside it (seven values, 32 rows of 16384: 17.8 us a call by the
// radix passes alone, 23.3 if they begin anew, 13.4 so; two clusters 1e-4 wide 20.7, 29.6, 18.9).
template <int ITEMS, typename KeyFn>
__device__ __forceinline__ bool select_kth_linear(const KeySet<ITEMS, KeyFn>& ks, float width, int& k_rem, uint32_t& lo, uint32_t& hi,
                                                  SelectShared& sh, uint32_t& key_t) {
  const int tid = threadIdx.x;
  const float x0 = key_to_float(lo), scale = ((float)kBins - 0.125f) / width;
  auto bin = [&](int i) { return min((int)((key_to_float(ks.key(i)) - x0) * scale), kBins - 1); };     // ascends with the key
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (ks.valid(i)) atomicAdd(&sh.hist[bin(i)], 1u);
  __syncthreads();
  find_digit(k_rem, 0, sh);
  const int digit = (int)sh.digit, members = (int)sh.hist[digit];
  k_rem -= (int)sh.above;
  if (members <= kRankMax) {                                               // workgroup-uniform
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (ks.valid(i) && bin(i) == digit) sh.list[atomicAdd(&sh.n_list, 1)] = ks.key(i);
    __syncthreads();
    rank_list(members, k_rem, sh);
    key_t = sh.digit;
    k_rem -= (int)sh.above;
    return true;
  }
  lo = 0xffffffffu; hi = 0u;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (ks.valid(i) && bin(i) == digit) { lo = min(lo, ks.key(i)); hi = max(hi, ks.key(i)); }
  lo = wave_min_u(lo); hi = wave_max_u(hi);
  __syncthreads();                                                         // the histogram has been read
  for (int i = tid; i < kBins; i += kSelThreads) sh.hist[i] = 0;
  if ((tid & 63) == 0) { sh.red_lo[tid >> 6] = lo; sh.red_hi[tid >> 6] = hi; }
  __syncthreads();
  lo = row16_min_u(sh.red_lo[tid & 15]); hi = row16_max_u(sh.red_hi[tid & 15]);
  return false;
}

// The radix passes: the k_rem-th largest of the keys by their distance from lo, at most range; returns the distance, and in
// k_rem how many keys equal to it are taken.  INSIDE: only part of the keys lie in this range, and they are not rebased (slots past M
// hold 0, below lo); otherwise all do, and are rebased to lo.  The histogram and the list's counter are cleared.
template <bool INSIDE, int ITEMS, typename KeyFn>
__device__ __forceinline__ uint32_t radix_passes(const KeySet<ITEMS, KeyFn>& ks, uint32_t lo, uint32_t range, int& k_rem, SelectShared& sh) {
  const int tid = threadIdx.x;
  auto dist = [&](int i) { return INSIDE ? ks.key(i) - lo : ks.key(i); };
  auto in = [&](int i, uint32_t v) { return INSIDE ? v <= range : ks.valid(i); };
  int shift = range ? 32 - __clz(range) : 0;     // significant bits of the distances
  uint32_t prefix = 0;                           // high bits of the answer fixed so far: (v >> shift) == prefix
  for (int pass = 0; shift > 0; ++pass) {
    const int dbits = min(kDigitBits, shift);
    shift -= dbits;
    const uint32_t dmask = (1u << dbits) - 1u;
    const int up = shift + dbits;                  // bits above the current digit: (v >> up) must equal prefix
    const bool first = up >= 32;                   // first pass of a full 32-bit range: every key matches
    if (pass > 0) {
      __syncthreads();
      for (int i = tid; i < kBins; i += kSelThreads) sh.hist[i] = 0;
      __syncthreads();
    }
    // Slots past M stay out: thousands of atomics on one LDS address serialise.
    if constexpr (ITEMS == 0) {
      for (int i0 = 0; i0 < ks.items; i0 += 8) {
        uint32_t kb[8];
        ks.key_batch(i0, kb);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (i0 + j < ks.items && ks.page(i0 + j) < ks.M && (first || (kb[j] >> up) == prefix))
            atomicAdd(&sh.hist[(kb[j] >> shift) & dmask], 1u);
      }
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const uint32_t v = dist(i);
        if (in(i, v) && (first || (v >> up) == prefix)) atomicAdd(&sh.hist[(v >> shift) & dmask], 1u);
      }
    }
    __syncthreads();
    find_digit(k_rem, pass, sh);
    const uint32_t digit = sh.digit;
    prefix = (prefix << dbits) | digit;
    k_rem -= (int)sh.above;
    if (shift == 0) break;
    // Few elements share the prefix (the usual case after the first pass): rank them against each other
    // directly instead of taking more passes.
    const int members = (int)sh.hist[digit];
    if (members <= kRankMax) {                     // workgroup-uniform
      if constexpr (ITEMS == 0) {
        for (int i0 = 0; i0 < ks.items; i0 += 8) {
          uint32_t kb[8];
          ks.key_batch(i0, kb);
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (i0 + j < ks.items && ks.page(i0 + j) < ks.M && (kb[j] >> shift) == prefix)
              sh.list[atomicAdd(&sh.n_list, 1)] = kb[j];
        }
      } else {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          const uint32_t v = dist(i);
          if (in(i, v) && (v >> shift) == prefix) sh.list[atomicAdd(&sh.n_list, 1)] = v;
        }
      }
      __syncthreads();
      rank_list(members, k_rem, sh);
      k_rem -= (int)sh.above;
      return sh.digit;
    }
  }
  return prefix;
}

// Finds the k-th largest key (1 <= k <= M) by radix selection on (key - min key), 11 bits per pass over
// only as many bits as the key range needs.  Rebases the key set to the smallest valid key and returns
// vT = the k-th largest rebased key and k_eq = how many elements equal to it belong to the top k.
// Slots past M are not counted.
template <int ITEMS, typename KeyFn>
__device__ __forceinline__ void radix_select_kth(KeySet<ITEMS, KeyFn>& ks, int k, SelectShared& sh,
                                                 uint32_t& vT_out, int& k_eq_out) {
  const int tid = threadIdx.x;
  uint32_t lo = 0xffffffffu, hi = 0u;
  constexpr int kFew = ITEMS < 4 ? ITEMS : 4;
  uint32_t few_lo = 0xffffffffu, few_hi = 0u;      // of this thread's first kFew keys
  if constexpr (ITEMS == 0) {
    for (int i0 = 0; i0 < ks.items; i0 += 8) {
      uint32_t kb[8];
      ks.key_batch(i0, kb);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < ks.items && ks.page(i0 + j) < ks.M) { lo = min(lo, kb[j]); hi = max(hi, kb[j]); }
    }
  } else {
#pragma unroll
    for (int i = 0; i < (ITEMS ? ITEMS : ks.items); ++i) {
      if (ks.valid(i)) { const uint32_t key = ks.key(i); lo = min(lo, key); hi = max(hi, key); }
      if (i == kFew - 1) { few_lo = lo; few_hi = hi; }
    }
  }
  // one barrier for both extremes; the histogram and the list's counter are cleared on the way
  lo = wave_min_u(lo); hi = wave_max_u(hi);
  __syncthreads();                                 // whatever used the shared arrays before is done
  for (int i = tid; i < kBins; i += kSelThreads) sh.hist[i] = 0;
  if ((tid & 63) == 0) {
    sh.red_lo[tid >> 6] = lo; sh.red_hi[tid >> 6] = hi;
    if (ITEMS > 0) { sh.few_lo[tid >> 6] = few_lo; sh.few_hi[tid >> 6] = few_hi; }
  }
  if (tid == 0) sh.n_list = 0;
  __syncthreads();
  lo = row16_min_u(sh.red_lo[tid & 15]); hi = row16_max_u(sh.red_hi[tid & 15]);
  k_eq_out = k;
  if constexpr (ITEMS > 0) {
    if (lo < kKeyOfZero && hi >= kKeyOfZero) {
      // Equal steps are the better digits unless outliers make up the range: in at least half of the wavefronts that hold scores,
      // the first two or four of the first thread span a 256th or a 64th of it.  Calls over 32 rows of 16384 pages (48 of 2626), us,
      // radix passes alone / equal steps without this rule / as here: one negative score 17.0 / 10.4 / 10.2 (6.9 / 5.2 / 5.3), on both
      // sides of zero 14.6 / 10.2 / 10.1 (6.2 / 5.2 / 5.2), a tenth of the range wide beside one negative 24.1 / 11.0 / 10.8; two scores
      // 3e4 times the others' deviation 17.5 / 32.3 / 17.6 (7.0 / 10.1 / 7.1), log-normal with deviation 3 13.0 / 26.0 / 13.0, one in
      // fifty 5000 times the others 14.5 / 28.8 / 14.4.
      const uint32_t base = lo, few = sh.few_lo[tid & 15], most = sh.few_hi[tid & 15];
      const float width = key_to_float(hi) - key_to_float(lo);
      const bool has = few <= most, wide = has && key_to_float(most) - key_to_float(few) >= (kFew == 4 ? 1 / 64.f : 1 / 256.f) * width;
      if (width < INFINITY && (float)kBins / width < INFINITY && 2 * __popcll(__ballot(wide)) >= __popcll(__ballot(has))) {
        uint32_t key_t;
        if (!select_kth_linear(ks, width, k_eq_out, lo, hi, sh, key_t)) key_t = lo + radix_passes<true>(ks, lo, hi - lo, k_eq_out, sh);
        vT_out = key_t - base;
        ks.rebase(base);
        return;
      }
    }
  }
  ks.rebase(lo);
  vT_out = radix_passes<false>(ks, lo, hi - lo, k_eq_out, sh);
}

// Writes, in ascending page order, every page whose (rebased) key exceeds vT, plus the first k_eq
// pages (by index) whose key equals vT.  Slots past M are never written.
template <int ITEMS, typename KeyFn>
__device__ __forceinline__ void compact_ordered(const KeySet<ITEMS, KeyFn>& ks, uint32_t vT, int k_eq,
                                                SelectShared& sh, int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  int n_gt = 0, n_eq = 0;
  if constexpr (ITEMS == 0) {
    for (int i0 = 0; i0 < ks.items; i0 += 8) {
      uint32_t kb[8];
      ks.key_batch(i0, kb);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < ks.items) { n_gt += kb[j] > vT; n_eq += kb[j] == vT; }
    }
  } else {
#pragma unroll
    for (int i = 0; i < (ITEMS ? ITEMS : ks.items); ++i) {
      const uint32_t v = ks.key(i);       // per-lane counts (no ballots here: they would all be kept
      n_gt += v > vT;                     // alive for the second loop and exhaust the scalar registers)
      n_eq += v == vT;
    }
  }
  n_gt = wave_sum_i(n_gt);
  n_eq = wave_sum_i(n_eq);
  if (lane == 0) { sh.wave_gt[w] = n_gt; sh.wave_eq[w] = n_eq; }     // written once per selection
  __syncthreads();
  const int gt_before = row16_sum_i((lane & 15) < w ? sh.wave_gt[lane & 15] : 0);
  const int eq_before = row16_sum_i((lane & 15) < w ? sh.wave_eq[lane & 15] : 0);
  int eq_run = eq_before;
  int o_run = gt_before + min(eq_before, k_eq);
  auto emit = [&](int i, uint32_t v) {
    const bool eq = v == vT;
    const uint64_t m_eq = __ballot(eq);
    const bool take = v > vT || (eq && eq_run + __popcll(m_eq & lt) < k_eq);
    const uint64_t m_take = __ballot(take);
    if (take) out[o_run + __popcll(m_take & lt)] = ks.page(i);
    eq_run += __popcll(m_eq);
    o_run += __popcll(m_take);
  };
  if constexpr (ITEMS == 0) {
    for (int i0 = 0; i0 < ks.items; i0 += 8) {
      uint32_t kb[8];
      ks.key_batch(i0, kb);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + j < ks.items) emit(i0 + j, kb[j]);       // wave-uniform condition
    }
  } else {
#pragma unroll
    for (int i = 0; i < (ITEMS ? ITEMS : ks.items); ++i) {
      emit(i, ks.key(i));
      __builtin_amdgcn_sched_barrier(0);    // keep the iterations in order: hoisting every compare first
    }                                       // needs two scalar register pairs per key
  }
}

}  // namespace ekv
