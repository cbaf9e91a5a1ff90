// The decode's pass 1, what its kernels share: arguments, and how its items are dealt to the wavefronts.
#pragma once
#include "ekv_device.h"
#include "ekv_internal.h"

namespace ekv {

constexpr int kScoreThreads = 256;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// Candidate source of a launch: per query head its own page list (unit = (b, query head), G = 1);
// every page of the sequence; or one page list per KV head shared by its G query heads.  In the last
// two the unit is (b, KV head) and the G heads are scored from one read of K.
enum : int { kPerHead = 0, kAllPages = 1, kGroupList = 2 };

struct ScoreArgs {
  const void* q; const void* k_pool;
  const int32_t* block_table; const int32_t* seq_lens; const int32_t* page_idx; const int32_t* n_sel;
  float* zbuf; float* pmax;
  int Hq, Hkv, P, Mmax, cap, n_chunks_max, n_phys;
  size_t zstride;
  float zscale;
  int HkvPool;
  int U;                  // units of the launch: B*Hq page lists, or B*Hkv (all pages / one list per KV head)
  const int32_t* pre_g;   // exclusive prefix of the items per unit, [U + 1], when U is too large for LDS
  int parts;              // kXcds: each unit is split over the XCDs, 1: it is not
};

constexpr int kScoreWaves = kScoreThreads / 64;
constexpr int kUnitsLdsMax = 8192;      // units whose item prefix a workgroup keeps in LDS (32 KB)

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return min(max(x, lo), hi); }
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// LDS accesses of one wavefront on either side keep their order (the hardware executes them in order; the compiler is told).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// Work distribution of pass 1.  An item is one group of pmax_pages(P) page slots of one unit (64 tokens when P
// divides 64): the granularity of pmax.  The launch has a fixed number of wavefronts that does not depend on the
// capacity of the page lists: the items of all units, in (unit, group) order, form one sequence of T items, and
// wavefront i of W takes the contiguous range [i*T/W, (i+1)*T/W).  T and the unit boundaries come from the
// device-side lengths (n_sel, or seq_lens when every page is a candidate): every workgroup builds the exclusive
// prefix of the items per unit in LDS (launches with more units than LDS holds read it from `pre_g`, written by
// unit_prefix_kernel before).
template <int MODE>
__device__ __forceinline__ int unit_slots(const ScoreArgs& A, int u) {
  if (MODE == kAllPages) return clampi((A.seq_lens[u / A.Hkv] + A.P - 1) / A.P, 0, A.Mmax);
  return clampi(A.n_sel[u], 0, A.cap);
}

// Which part of every unit a workgroup works on.  Workgroups go to the eight XCDs in turn, each with an L2 of its own,
// and the query heads of a KV group often select the same pages: with per-head lists part x of EVERY list belongs to the
// workgroups of XCD x (rotated from group to group, so that short lists spread too), so that the heads of a group, whose
// lists cover about the same pages in the same eighth, meet in one L2 instead of fetching a page into several.  The parts
// are as even as the lists allow, whatever the shapes.  Whole calls, us: 32K-token Gaussian step (lists of about 40 % of
// the pages) 52.5 -> 46.6, decode over all pages of 3 x 21K float32 tokens within the refined step 147 -> 126.5; lists that
// hardly overlap (2 % of a million tokens) 113.4 -> 112.6.
constexpr int kXcds = 8;
struct Part { int index, count; };             // this workgroup's part, parts per unit (1: units are not split)
__device__ __forceinline__ Part unit_part(const ScoreArgs& A) {
  return {A.parts == kXcds ? (int)(blockIdx.x % kXcds) : 0, A.parts};
}
// The item range of this wavefront and the unit its first item lies in.
struct WaveItems { int begin, end, unit; };
template <typename P>
__device__ __forceinline__ WaveItems wave_item_range(const P pre, int U, int w, const Part& part) {
  const int total = uniform(pre[U]);
  const int W = gridDim.x / part.count * kScoreWaves, gw = blockIdx.x / part.count * kScoreWaves + w;
  // balanced contiguous partition: the first total % W wavefronts take one item more
  const int per = total / W, rem = total - per * W;
  WaveItems r;
  r.begin = gw * per + min(gw, rem);
  r.end = r.begin + per + (gw < rem ? 1 : 0);
  r.unit = wave_last_at_most(pre, U, r.begin);          // pre[unit] <= begin < pre[unit + 1] whenever begin < total
  return r;
}

static inline int device_compute_units() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}
// Score pass of a dense decode in common windows for the stores (decode_windows.hip); false, with nothing launched, where the
// kernels of decode.hip are the faster ones or the call has a form that it does not take.
template <int G> bool launch_scores_windows(const Dims& dm, const ScoreArgs& sa, long long items, size_t k_bytes, hipStream_t st);

}  // namespace ekv
