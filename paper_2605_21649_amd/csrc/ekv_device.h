// Device-side helpers shared by the gfx950 kernels: 16-byte row loads, wavefront (64-lane)
// reductions built on DPP row operations, order-preserving float<->uint keys.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ekv {

constexpr int kD = 128;            // head_dim the kernels are written for
constexpr int kLanesPerRow = 16;   // 16 lanes x 8 channels cover one 128-channel row
constexpr int kRowsPerWave = 4;    // a 64-lane wavefront covers 4 rows per step
constexpr int kWave = 64;

struct bf16_t { uint16_t bits; };

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// round-to-nearest-even float -> bf16 bits (finite inputs; NaN is kept quiet)
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Wave-uniform read of an int32 in device memory that nothing in the running launch writes (page lists, block
// table, lengths written by earlier launches): a load through the constant address space with a uniform address
// is a scalar load, which does not queue behind the vector loads in flight and costs no vector register.
typedef const int32_t __attribute__((address_space(4)))* const_i32_ptr;
__device__ __forceinline__ int32_t uniform_load(const int32_t* p) { return *(const_i32_ptr)(uintptr_t)p; }

// 16 bytes; STREAM: of a stream that this launch reads once (a non-temporal load: its line leaves the caches first).  Such
// streams run faster by themselves, with the same bytes from memory: page scoring of a million tokens 46.3 -> 41.9 us at 256.3
// MiB read and 8.0 written either way.  Beside a stream of stores, lines leave the caches before they are whole less often:
// the dense score pass over a million tokens, 64 bytes of scores at a time, wrote 155 MiB for its 130 and then 133
// (read 2052 and 2049), which is little of the 453 -> 409 us (362 since its stores go into windows: decode_windows.hip).
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
template <bool STREAM = false> __device__ __forceinline__ uint4 load16(const void* p) {
  if constexpr (STREAM) return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)));
  else return *reinterpret_cast<const uint4*>(p);
}
// Buffer resources of plain bytes, and the cache bits of the buffer instructions: non-temporal; through the caches to memory.
constexpr int kBufferFlags = 0x00020000, kBufferNt = 2, kBufferThrough = 17;
template <bool STREAM = false> __device__ __forceinline__ void store16(void* p, const uint4& v) {
  if constexpr (STREAM) __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t*>(p));
  else *reinterpret_cast<uint4*>(p) = v;
}

// Load 8 consecutive channels (one lane's share of a 128-channel row) as float.
template <typename T> __device__ __forceinline__ void load8(const T* p, float (&x)[8]);

template <> __device__ __forceinline__ void load8<float>(const float* p, float (&x)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
  x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

template <> __device__ __forceinline__ void load8<bf16_t>(const bf16_t* p, float (&x)[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);     // one 16-byte load: 8 bf16
  x[0] = __uint_as_float(a.x << 16); x[1] = __uint_as_float(a.x & 0xffff0000u);
  x[2] = __uint_as_float(a.y << 16); x[3] = __uint_as_float(a.y & 0xffff0000u);
  x[4] = __uint_as_float(a.z << 16); x[5] = __uint_as_float(a.z & 0xffff0000u);
  x[6] = __uint_as_float(a.w << 16); x[7] = __uint_as_float(a.w & 0xffff0000u);
}

// The same 8 channels kept as loaded (16 or 32 bytes), to be widened only where they are consumed:
// a batch of rows in flight then costs 4 (bf16) or 8 (f32) registers per row, not 8 floats.
template <typename T> struct Raw8;
template <> struct Raw8<float> { float4 a, b; };
template <> struct Raw8<bf16_t> { uint4 a; };
__device__ __forceinline__ void load_raw8(const float* p, Raw8<float>& r) {
  r.a = *reinterpret_cast<const float4*>(p);
  r.b = *reinterpret_cast<const float4*>(p + 4);
}
__device__ __forceinline__ void load_raw8(const bf16_t* p, Raw8<bf16_t>& r) { r.a = *reinterpret_cast<const uint4*>(p); }
// A row in the sixteen lanes of a DPP row, for streams (STREAM as in load16): bf16 channels 8c..8c+7 in lane c, float32
// channels 4c..4c+3 and 64+4c..64+4c+3, so that either type takes whole lines with each load; eight channels in a row take a
// float32 line in halves, and one that is not kept is fetched twice.  p: the row's first channel of the lane.
template <typename T> __device__ __forceinline__ constexpr int lane_channel(int c) { return sizeof(T) == 4 ? 4 * c : 8 * c; }
template <bool STREAM = false> __device__ __forceinline__ void load_row8(const float* p, Raw8<float>& r) {
  r.a = __builtin_bit_cast(float4, load16<STREAM>(p));
  r.b = __builtin_bit_cast(float4, load16<STREAM>(p + kD / 2));
}
template <bool STREAM = false> __device__ __forceinline__ void load_row8(const bf16_t* p, Raw8<bf16_t>& r) { r.a = load16<STREAM>(p); }
// The same for two groups of float32 rows, one per half of the wavefront, where a row's sum has to run over lane c's channels
// 8c..8c+7: r.a is fetched from the lower half's group and r.b from the upper's, each whole, and the halves then hand each
// other what is theirs.  p0, p1: the lane's row of the group at channel 8c + 4 * (its half).
template <bool STREAM = false> __device__ __forceinline__ void load_halves(const float* p0, const float* p1, Raw8<float>& r) {
  r.a = __builtin_bit_cast(float4, load16<STREAM>(p0));
  r.b = __builtin_bit_cast(float4, load16<STREAM>(p1));
}
__device__ __forceinline__ void swap_halves(float& a, float& b) {      // lanes 32..63 of a with lanes 0..31 of b
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(Raw8<float>& r) {
  swap_halves(r.a.x, r.b.x); swap_halves(r.a.y, r.b.y); swap_halves(r.a.z, r.b.z); swap_halves(r.a.w, r.b.w);
}
__device__ __forceinline__ void widen8(const Raw8<float>& r, float (&x)[8]) {
  x[0] = r.a.x; x[1] = r.a.y; x[2] = r.a.z; x[3] = r.a.w;
  x[4] = r.b.x; x[5] = r.b.y; x[6] = r.b.z; x[7] = r.b.w;
}
__device__ __forceinline__ void widen8(const Raw8<bf16_t>& r, float (&x)[8]) {
  x[0] = __uint_as_float(r.a.x << 16); x[1] = __uint_as_float(r.a.x & 0xffff0000u);
  x[2] = __uint_as_float(r.a.y << 16); x[3] = __uint_as_float(r.a.y & 0xffff0000u);
  x[4] = __uint_as_float(r.a.z << 16); x[5] = __uint_as_float(r.a.z & 0xffff0000u);
  x[6] = __uint_as_float(r.a.w << 16); x[7] = __uint_as_float(r.a.w & 0xffff0000u);
}

__device__ __forceinline__ uint4 pack8(const float (&x)[8]) {
  uint4 a;
  a.x = float_to_bf16_bits(x[0]) | ((uint32_t)float_to_bf16_bits(x[1]) << 16);
  a.y = float_to_bf16_bits(x[2]) | ((uint32_t)float_to_bf16_bits(x[3]) << 16);
  a.z = float_to_bf16_bits(x[4]) | ((uint32_t)float_to_bf16_bits(x[5]) << 16);
  a.w = float_to_bf16_bits(x[6]) | ((uint32_t)float_to_bf16_bits(x[7]) << 16);
  return a;
}
__device__ __forceinline__ void store8(float* p, const float (&x)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(x[0], x[1], x[2], x[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(x[4], x[5], x[6], x[7]);
}
__device__ __forceinline__ void store8(bf16_t* p, const float (&x)[8]) { store16(p, pack8(x)); }
// the lane's channels of load_row8, past the caches
__device__ __forceinline__ void stream_row8(float* p, const float (&x)[8]) {
  store16<true>(p, __builtin_bit_cast(uint4, make_float4(x[0], x[1], x[2], x[3])));
  store16<true>(p + kD / 2, __builtin_bit_cast(uint4, make_float4(x[4], x[5], x[6], x[7])));
}
__device__ __forceinline__ void stream_row8(bf16_t* p, const float (&x)[8]) { store16<true>(p, pack8(x)); }

// ---- 8-bit bounds: OCP E4M3 (bias 7, 3 mantissa bits, subnormals, max 448, 0x7f = NaN) -----------
// Directed rounding of a float: UP gives the code of the smallest format value >= x, otherwise of the
// largest <= x; the NaN code when no finite format value qualifies (or x is NaN).
template <bool UP> __device__ __forceinline__ uint32_t f32_to_e4m3_directed(float x) {
  const uint32_t bits = __float_as_uint(x);
  const uint32_t sign = bits >> 31, abits = bits & 0x7fffffffu;
  const float a = __uint_as_float(abits);
  const bool away = UP ? sign == 0u : sign != 0u;        // the magnitude is rounded up
  if (!(a <= 448.0f)) return (a != a || away) ? 0x7fu : ((sign << 7) | 0x7eu);
  uint32_t mag;
  if (a < 0.015625f) {                                   // below 2^-6: multiples of 2^-9 (codes 0..8)
    const float s = a * 512.0f, f = floorf(s);
    mag = (uint32_t)f + ((away && s != f) ? 1u : 0u);
  } else {
    uint32_t t = abits & ~0xfffffu;                      // three mantissa bits kept
    if (away && t != abits) t += 0x100000u;              // next format value; a carry moves to the next binade
    mag = (t >> 20) - (120u << 3);                       // exponent field = float exponent - 127 + 7
  }
  return (sign << 7) | mag;
}

// One 16-byte unit of the 8-bit bounds: k_min of 8 channels (rounded down), then k_max (rounded up).
__device__ __forceinline__ void store_box8_unit(uint8_t* p, const float (&mn)[8], const float (&mx)[8]) {
  uint4 u;
  u.x = f32_to_e4m3_directed<false>(mn[0]) | (f32_to_e4m3_directed<false>(mn[1]) << 8) |
        (f32_to_e4m3_directed<false>(mn[2]) << 16) | (f32_to_e4m3_directed<false>(mn[3]) << 24);
  u.y = f32_to_e4m3_directed<false>(mn[4]) | (f32_to_e4m3_directed<false>(mn[5]) << 8) |
        (f32_to_e4m3_directed<false>(mn[6]) << 16) | (f32_to_e4m3_directed<false>(mn[7]) << 24);
  u.z = f32_to_e4m3_directed<true>(mx[0]) | (f32_to_e4m3_directed<true>(mx[1]) << 8) |
        (f32_to_e4m3_directed<true>(mx[2]) << 16) | (f32_to_e4m3_directed<true>(mx[3]) << 24);
  u.w = f32_to_e4m3_directed<true>(mx[4]) | (f32_to_e4m3_directed<true>(mx[5]) << 8) |
        (f32_to_e4m3_directed<true>(mx[6]) << 16) | (f32_to_e4m3_directed<true>(mx[7]) << 24);
  *reinterpret_cast<uint4*>(p) = u;
}

// ---- DPP cross-lane moves (no LDS traffic) -------------------------------------------------
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ int dpp_move_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}

// Sum over each aligned group of 16 lanes (a DPP "row"); every lane of the row gets the total.
// Fixed butterfly order: xor 1, xor 2, half-row mirror, row mirror.
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return v;
}

// Wavefront reductions: DPP butterflies inside each 16-lane row, then the two cross-row DPP broadcasts
// (lane 15 of a row into the next row, lane 31 into the upper half), which leave the result in lane 63;
// it is returned to every lane through a scalar register.  No LDS traffic, fixed order.  All 64 lanes of
// the wavefront must be active at the call (every call site is wavefront-uniform).
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_rows(float old, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
template <int CTRL, int ROW_MASK> __device__ __forceinline__ int dpp_rows_i(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ float wave_sum(float v) {
  v = row16_sum(v);
  v += dpp_rows<0x142, 0xa>(0.f, v);     // row_bcast15 into rows 1 and 3
  v += dpp_rows<0x143, 0xc>(0.f, v);     // row_bcast31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));
  v = fmaxf(v, dpp_move<0x4E>(v));
  v = fmaxf(v, dpp_move<0x141>(v));
  v = fmaxf(v, dpp_move<0x140>(v));
  v = fmaxf(v, dpp_rows<0x142, 0xa>(v, v));
  v = fmaxf(v, dpp_rows<0x143, 0xc>(v, v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ int wave_sum_i(int v) {
  v += dpp_move_i<0xB1>(v);
  v += dpp_move_i<0x4E>(v);
  v += dpp_move_i<0x141>(v);
  v += dpp_move_i<0x140>(v);
  v += dpp_rows_i<0x142, 0xa>(0, v);
  v += dpp_rows_i<0x143, 0xc>(0, v);
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ uint32_t row16_min_u(uint32_t v) {
  v = min(v, (uint32_t)dpp_move_i<0xB1>((int)v));
  v = min(v, (uint32_t)dpp_move_i<0x4E>((int)v));
  v = min(v, (uint32_t)dpp_move_i<0x141>((int)v));
  return min(v, (uint32_t)dpp_move_i<0x140>((int)v));
}
__device__ __forceinline__ uint32_t row16_max_u(uint32_t v) {
  v = max(v, (uint32_t)dpp_move_i<0xB1>((int)v));
  v = max(v, (uint32_t)dpp_move_i<0x4E>((int)v));
  v = max(v, (uint32_t)dpp_move_i<0x141>((int)v));
  return max(v, (uint32_t)dpp_move_i<0x140>((int)v));
}
__device__ __forceinline__ uint32_t wave_min_u(uint32_t v) {
  v = row16_min_u(v);
  v = min(v, (uint32_t)dpp_rows_i<0x142, 0xa>((int)v, (int)v));
  v = min(v, (uint32_t)dpp_rows_i<0x143, 0xc>((int)v, (int)v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
  v = row16_max_u(v);
  v = max(v, (uint32_t)dpp_rows_i<0x142, 0xa>((int)v, (int)v));
  v = max(v, (uint32_t)dpp_rows_i<0x143, 0xc>((int)v, (int)v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ int row16_sum_i(int v) {
  v += dpp_move_i<0xB1>(v);
  v += dpp_move_i<0x4E>(v);
  v += dpp_move_i<0x141>(v);
  return v + dpp_move_i<0x140>(v);
}
// Inclusive prefix sum over the wavefront (row shifts, then the two cross-row broadcasts).
__device__ __forceinline__ int wave_incl_scan_i(int v) {
  v += dpp_rows_i<0x111, 0xf>(0, v);     // row_shr 1, 2, 4, 8: lanes shifted in from outside the row count as 0
  v += dpp_rows_i<0x112, 0xf>(0, v);
  v += dpp_rows_i<0x114, 0xf>(0, v);
  v += dpp_rows_i<0x118, 0xf>(0, v);
  v += dpp_rows_i<0x142, 0xa>(0, v);     // row_bcast15 into rows 1 and 3
  v += dpp_rows_i<0x143, 0xc>(0, v);     // row_bcast31 into rows 2 and 3
  return v;
}

// Block-wide reductions through a small LDS array (one slot per wavefront); all threads get the
// result.  The combination order is fixed (wavefront 0,1,2,...), so results are reproducible.
// `buf` must hold blockDim.x/64 floats and must not be in use by a pending reduction.
__device__ __forceinline__ float block_sum(float v, float* buf) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) buf[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += buf[i];
  return t;
}
__device__ __forceinline__ float block_max(float v, float* buf) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) buf[w] = v;
  __syncthreads();
  float t = buf[0];
  for (int i = 1; i < nw; ++i) t = fmaxf(t, buf[i]);
  return t;
}
__device__ __forceinline__ int block_sum_i(int v, int* buf) {
  v = wave_sum_i(v);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) buf[w] = v;
  __syncthreads();
  int t = 0;
  for (int i = 0; i < nw; ++i) t += buf[i];
  return t;
}

// Exclusive prefix over `U` counts produced by `count_of(u)`, written to pre[0..U] (pre[U] = total); `wsum` holds
// one int per wavefront.  Called by every thread of the workgroup.
template <int THREADS, typename F>
__device__ __forceinline__ void block_exclusive_prefix(int U, F&& count_of, int* pre, int* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (U <= THREADS) {
    // one unit per thread (the usual launch): a wavefront scan, the wavefront totals, two barriers; every workgroup
    // of the launch runs this before its first load, so it is kept to a few dozen instructions
    const int c = tid < U ? count_of(tid) : 0;
    const int inc = wave_incl_scan_i(c);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int base = inc - c;
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) base += i < w ? wsum[i] : 0;
    if (tid < U) pre[tid] = base;
    if (tid == U - 1) pre[U] = base + c;
    __syncthreads();
    return;
  }
  for (int u = tid; u < U; u += THREADS) pre[u] = count_of(u);
  __syncthreads();
  const int upt = (U + THREADS - 1) / THREADS;          // a contiguous segment per thread
  const int s0 = min(tid * upt, U), s1 = min(s0 + upt, U);
  int s = 0;
  for (int u = s0; u < s1; ++u) s += pre[u];
  const int inc = wave_incl_scan_i(s);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int base = inc - s;
  for (int i = 0; i < w; ++i) base += wsum[i];
  for (int u = s0; u < s1; ++u) { const int c = pre[u]; pre[u] = base; base += c; }
  if (tid == THREADS - 1) pre[U] = base;                // the last segment ends at U
  __syncthreads();
}

// The last of entries [0, n) of the ascending pre that is not above v (pre[0] <= v), the same for the whole wavefront: 64 entries
// compared at a time, so one LDS latency up to 64 entries and two up to 4096, where halving the range takes six and twelve.
// Every launch over lists begins with the prefix of their lengths and this search.  By LDS permutes and halving, and with the
// solve's segment ends so too, decode calls took 0.4 to 0.6 us more: over shared lists of 328 pages of 262144 tokens 12.9 -> 12.5 us,
// of 16 pages for 64 sequences 17.8 -> 17.3, lists per head of 328 17.6 -> 17.0.
template <typename P> __device__ __forceinline__ int wave_last_at_most(const P pre, int n, int v) {
  const int lane = threadIdx.x & 63;
  int lo = 0;
  while (n > 1) {
    const int step = (n + 63) >> 6, at = lane * step;
    const int k = __popcll(__ballot(at < n && pre[lo + min(at, n - 1)] <= v)) - 1;
    lo += k * step;
    n = min(step, n - k * step);
  }
  return lo;
}
// The same for ascending values of the lanes, v <= last in every lane; first: any entry not above all of them.
template <typename P> __device__ __forceinline__ int lane_last_at_most(const P pre, int n, int first, int v, int last) {
  int lo = first, hi = first + 1;
  if (__builtin_amdgcn_readfirstlane(pre[hi]) <= last) {               // more than one entry: halved between the first and the last
    hi = first + wave_last_at_most(pre + first, n - first, last) + 1;
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (pre[mid] <= v) lo = mid; else hi = mid; }
  }
  return lo;
}

// Order-preserving map float -> uint32 (larger float <=> larger key); -inf maps near 0.
__device__ __forceinline__ uint32_t float_to_key(float f) {
  const uint32_t u0 = __float_as_uint(f);
  const uint32_t u = u0 == 0x80000000u ? 0u : u0;        // -0.0 and +0.0 are one value (a tie), not two
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr uint32_t kKeyOfZero = 0x80000000u;
__device__ __forceinline__ float key_to_float(uint32_t k) { return __uint_as_float(k & 0x80000000u ? k ^ 0x80000000u : ~k); }

// x^beta for x > 0 with the small integer exponents special-cased (exact products).
__device__ __forceinline__ float pow_beta(float x, float beta, int ibeta) {
  switch (ibeta) {
    case 1: return x;
    case 2: return x * x;
    case 3: return x * x * x;
    case 4: { const float y = x * x; return y * y; }
    default: return __builtin_exp2f(beta * __builtin_log2f(x));
  }
}
// x^(beta-1)
__device__ __forceinline__ float pow_beta_m1(float x, float beta, int ibeta) {
  switch (ibeta) {
    case 1: return 1.f;
    case 2: return x;
    case 3: return x * x;
    case 4: return x * x * x;
    default: return __builtin_exp2f((beta - 1.f) * __builtin_log2f(x));
  }
}

// Calls fn with beta as a compile-time exponent (1..4, or 0 for any other), so that a loop over registers carries one
// product per entry instead of a branch on the exponent.
template <int N> struct IntC { static constexpr int value = N; };
template <typename F> __device__ __forceinline__ auto with_beta(int ibeta, F&& fn) {
  switch (ibeta) {
    case 1: return fn(IntC<1>{});
    case 2: return fn(IntC<2>{});
    case 3: return fn(IntC<3>{});
    case 4: return fn(IntC<4>{});
    default: return fn(IntC<0>{});
  }
}

}  // namespace ekv
