// Score pass of the dense decode for large calls: the stores of the scores are put off and made by all of the GPU at once.
#include "ekv_scores.h"

namespace ekv {

constexpr int kHoldScores = 8192;       // scores a wavefront of decode_scores_windows_kernel holds back
constexpr int kHoldUnitsMax = 4096;     // and the most units of such a launch (16 KB of LDS beside 132, with one head 138)

// bf16 pages with P in {16, 32, 64}, every page a candidate, calls whose scores the L2s do not hold.  What bounds such a call is
// not the bytes: a stream of reads at 6.9 TB/s falls to 5.5 as soon as a few stores are mixed in, hardly further with more of
// them (1 GiB read: 156 us alone, 197 with 64 MiB written meanwhile, 217 with 256, which take 39 by themselves), because the
// memory turns round for each handful.  So a wavefront holds its scores in LDS and all of them write in the same few
// microseconds: when the clock that all compute units share (100 MHz) passes a multiple of `window` ticks, when 32 KiB
// are held, and at the end.  The stores go through the caches, which would spread them over the next window.  One workgroup
// of four wavefronts per compute unit, with two items (32 KiB) each in flight, reads as fast as eight workgroups do and reaches
// the end of an item every 2.4 us, so that they write together; eight wavefronts with half the LDS each: 726 us for 706 below.
// Score pass, us, one chunk at a time by decode_scores_mfma_kernel / here: 8 x 262144 tokens in pages of 32, four heads to a KV
// head 826 / 706 (650 without the stores), without the clock 765; 1 x 1048576 in pages of 16 413 / 365, 1 x 262144 100 / 93.5,
// 64 x 8192 204 / 180; eight heads, 1 x 524288 221 / 201; one head, 1 x 1048576 369 / 340.
template <int G, int PT>
__global__ __launch_bounds__(kScoreThreads) void decode_scores_windows_kernel(const ScoreArgs A, uint32_t window) {
  constexpr int NSET = (G + 3) / 4, GP = 64 / PT, KEEP = PT / 16;
  constexpr int kBatchItems = 64 / GP;
  constexpr int NB = kHoldScores / (64 * G);       // items a wavefront holds
  extern __shared__ int pre_lds[];
  __shared__ __attribute__((aligned(16))) float hold_z[kScoreWaves][kHoldScores];
  __shared__ float hold_max[kScoreWaves][NB * G];
  __shared__ int4 hold_at[kScoreWaves][NB];        // first row, group, scores stored per row
  __shared__ int wsum[kScoreWaves];
  static_assert(sizeof(hold_z) + sizeof(hold_max) + sizeof(hold_at) + sizeof(wsum) + (kHoldUnitsMax + 1) * sizeof(int) <= 160 * 1024,
                "the LDS of a compute unit");
  const bf16_t* q = (const bf16_t*)A.q;
  const bf16_t* k_pool = (const bf16_t*)A.k_pool;
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
  const int m = lane & 15, j = lane >> 4, kq = m & 3, gl = m >> 2;      // as in decode_scores_mfma_kernel
  const int lane_off = (gl * kD + (kq * 4 + j) * 8) * 2;
  block_exclusive_prefix<kScoreThreads>(A.U, [&](int u) { return (unit_slots<kAllPages>(A, u) + GP - 1) / GP; }, pre_lds, wsum);
  const WaveItems wi = wave_item_range((const int*)pre_lds, A.U, w, Part{0, 1});
  if (wi.begin >= wi.end) return;

  // lane l: page slot l % GP of item it0 + l / GP (clamped to the last item): unit, group, physical page
  struct Slots { int unit, grp, phys; };
  int unit0 = wi.unit;                             // the batch's first unit, or one before
  auto look_up = [&](int it0) {
    const int my_it = min(it0 + lane / GP, wi.end - 1);
    const int lo = lane_last_at_most((const int*)pre_lds, A.U, unit0, my_it, min(it0 + kBatchItems, wi.end) - 1);
    unit0 = __builtin_amdgcn_readlane(lo, 63);
    Slots s{lo, my_it - pre_lds[lo], 0};
    const int slot = min(s.grp * GP + lane % GP, A.Mmax - 1);
    s.phys = clampi(A.block_table[(size_t)(lo / A.Hkv) * A.Mmax + slot], 0, A.n_phys - 1);
    return s;
  };
  int batch0 = wi.begin;
  Slots now = look_up(batch0), next = look_up(batch0 + kBatchItems);

  // chunk c (16 tokens) of an item; past the wavefront's range the buffer has no bytes and nothing is read
  auto request = [&](int it, int c, u32x4_t (&a)[4]) {
    const int o = it - batch0, in = o < kBatchItems ? o : o - kBatchItems;
    const int pg = in * GP + c / KEEP;
    const int unit = __builtin_amdgcn_readlane(o < kBatchItems ? now.unit : next.unit, pg & 63);
    const int phys = __builtin_amdgcn_readlane(o < kBatchItems ? now.phys : next.phys, pg & 63);
    const bf16_t* kc = k_pool + (((size_t)phys * A.HkvPool + unit % A.Hkv) * PT + 16 * (c % KEEP)) * kD;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)kc, 0, it < wi.end ? 16 * kD * 2 : 0, kBufferFlags);
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + s * 4 * kD * 2, 0, kBufferNt);
  };

  int held = 0;
  auto flush = [&]() {
    wave_order();
    for (int i0 = 0; i0 < held; i0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(i0 + u, held - 1);
        const int4 at = hold_at[w][i];
        const int row0 = uniform(at.x), grp = uniform(at.y), lim = uniform(at.z);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(A.zbuf + (size_t)row0 * A.zstride + (size_t)grp * 64, 0, -1, kBufferFlags);
#pragma unroll
        for (int s = 0; s < NSET; ++s) {
          const int g = 4 * s + (lane >> 4), tok = 4 * (lane & 15);
          const u32x4_t v = *reinterpret_cast<const u32x4_t*>(&hold_z[w][i * 64 * G + min(g, G - 1) * 64 + ((tok + 16 * g) & 63)]);
          if (i0 + u < held && g < G && tok < lim)
            __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)((g * A.zstride + tok) * 4), 0, kBufferThrough);
        }
      }
    }
    for (int i = lane; i < held; i += 64) {
      const int4 at = hold_at[w][i];
#pragma unroll
      for (int g = 0; g < G; ++g) A.pmax[(size_t)(at.x + g) * A.n_chunks_max + at.y] = hold_max[w][i * G + g];
    }
    held = 0;
    wave_order();
  };

  uint32_t due = (uint32_t)__builtin_amdgcn_s_memrealtime();
  due += window - due % window;
  int unit_now = -1, n = 0, n_slots = 0, row0 = 0;
  u32x4_t bq[NSET];
#pragma unroll
  for (int s = 0; s < NSET; ++s) bq[s] = u32x4_t{0u, 0u, 0u, 0u};
  auto process = [&](int it, u32x4_t (&a)[4][4]) {
    const int at = (it - batch0) * GP;
    const int unit = __builtin_amdgcn_readlane(now.unit, at), grp = __builtin_amdgcn_readlane(now.grp, at);
    if (unit != unit_now) {
      const int b = unit / A.Hkv, hq0 = unit % A.Hkv * G;
      unit_now = unit;
      row0 = b * A.Hq + hq0;
      n = uniform_load(A.seq_lens + b);
      n_slots = clampi((n + PT - 1) / PT, 0, A.Mmax);
#pragma unroll
      for (int s = 0; s < NSET; ++s) {
        bq[s] = *reinterpret_cast<const u32x4_t*>(q + ((size_t)row0 + min(4 * s + gl, G - 1)) * kD + kq * 32 + j * 8);
        asm volatile("" : "+v"(bq[s]));            // waited for here: behind the branch the wait would drain the loads of K
      }
    }
    float wmax[NSET];
#pragma unroll
    for (int s = 0; s < NSET; ++s) wmax[s] = -INFINITY;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float zkeep[NSET];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool valid = grp * 64 + 16 * c + 4 * s + j < n;
#pragma unroll
        for (int cs = 0; cs < NSET; ++cs) {
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          const f32x4_t d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[c][s]),
                                                                    __builtin_bit_cast(bf16x8_t, bq[cs]), zero, 0, 0, 0);
          const float v01 = (kq & 1) ? d[1] : d[0], v23 = (kq & 1) ? d[3] : d[2];
          float v = (kq & 2) ? v23 : v01;
          v += dpp_move<0xB1>(v);
          v += dpp_move<0x4E>(v);
          const float z = valid ? A.zscale * v : -INFINITY;
          if (s == kq) zkeep[cs] = z;
          wmax[cs] = fmaxf(wmax[cs], z);
        }
      }
#pragma unroll
      for (int cs = 0; cs < NSET; ++cs) {
        const int g = 4 * cs + gl;
        if (g < G) hold_z[w][held * 64 * G + g * 64 + ((16 * c + 16 * g + 4 * kq + j) & 63)] = zkeep[cs];
      }
      __builtin_amdgcn_sched_barrier(0);
      request(it + 2, c, a[c]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int cs = 0; cs < NSET; ++cs) {
      float mx = wmax[cs];
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const int g = 4 * cs + gl;
      if (j == 0 && kq == 0 && g < G) hold_max[w][held * G + g] = mx;
    }
    if (lane == 0) hold_at[w][held] = make_int4(row0, grp, n_slots * PT - grp * 64, 0);
    if (it < wi.end) ++held;
    const uint32_t t = (uint32_t)__builtin_amdgcn_s_memrealtime();
    const bool tick = (int)(t - due) >= 0;
    if (held == NB || tick) flush();
    if (tick) due = t + window - t % window;
  };

  // The first requests are held in the order of their use: the compiler issued a0[0] last, and as the loop's waits have to hold
  // for that way in too, they then drained both items on every turn (1 x 262144 in pages of 16, a whole step: 151.0 / 149.8 us).
  u32x4_t a0[4][4], a1[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    request(wi.begin, c, a0[c]);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    request(wi.begin + 1, c, a1[c]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int it = wi.begin; it < wi.end; it += 2) {
    if (it == batch0 + kBatchItems) {
      batch0 = it;
      now = next;
      next = look_up(batch0 + kBatchItems);
    }
    process(it, a0);
    process(it + 1, a1);
  }
  flush();
}

// Below these lines the scores stay in the L2s until the launch ends anyway, and a range of few items shows the ramp of its one
// wavefront per SIMD.  Score pass, us, by chunks / in windows, K and scores in MB: 134 + 8 (four heads to a KV head) 26.4 / 26.9,
// 201 + 13 39.9 / 39.7, 268 + 17 51.7 / 50.2, 537 + 34 101.8 / 94.0; 268 + 34 (eight heads) 55.7 / 54.5; 268 + 8 (two) 48.6 /
// 48.1; 268 + 4 (one) 46.2 / 49.3, 537 + 8 90.6 / 89.9.  A window is what fills most of a wavefront's LDS at full rate: 60 us at
// four heads to a KV head.  The grid does not follow the capacity: decode of 4096 tokens in a capacity of a million 30.5 -> 15.4
// us, of 32768 37.1 -> 22.8.
// A change of unit waits for the new query behind the K in flight, and a workgroup starts only where a compute unit's LDS is free, on
// a fixed share of the call: neither shows against the launch by chunks, which pays more for its many workgroups.  Calls, us,
// by chunks / here, heads four to a KV head: 512 sequences of 512 tokens (4096 units of 8 items) 316 / 267, of 64 tokens in a
// capacity of 4096 225 / 146, 64 of 512 in 8192 54.7 / 40.5; one head, caches of 537 MB filled to half 58.2 / 56.8, of 1 GB 111 /
// 103; two calls at once on two streams, 1 x 262144 212 / 193 the pair, 64 x 8192 456 / 403, beside four calls of 32768 tokens each
// 313 / 288.
template <int G>
bool launch_scores_windows(const Dims& dm, const ScoreArgs& sa, long long items, size_t k_bytes, hipStream_t st) {
  const unsigned long long z_bytes = (unsigned long long)sa.U * G * sa.zstride * 4;
  if (dm.dtype != EKV_BF16 || (dm.P != 16 && dm.P != 32 && dm.P != 64) || sa.U > kHoldUnitsMax || k_bytes < (256u << 20) ||
      z_bytes < (8u << 20) || (unsigned long long)sa.zstride * G * 4 > 0xffffffffull) return false;
  const long long wgs = (items + kScoreWaves - 1) / kScoreWaves;
  const int cus = device_compute_units();
  const dim3 grid((unsigned)(wgs < cus ? wgs : cus)), block(kScoreThreads);
  const size_t lds = (size_t)(sa.U + 1) * sizeof(int);
  const uint32_t window = 24000 / G;
  if (dm.P == 16) hipLaunchKernelGGL((decode_scores_windows_kernel<G, 16>), grid, block, lds, st, sa, window);
  else if (dm.P == 32) hipLaunchKernelGGL((decode_scores_windows_kernel<G, 32>), grid, block, lds, st, sa, window);
  else hipLaunchKernelGGL((decode_scores_windows_kernel<G, 64>), grid, block, lds, st, sa, window);
  return true;
}
template bool launch_scores_windows<1>(const Dims&, const ScoreArgs&, long long, size_t, hipStream_t);
template bool launch_scores_windows<2>(const Dims&, const ScoreArgs&, long long, size_t, hipStream_t);
template bool launch_scores_windows<4>(const Dims&, const ScoreArgs&, long long, size_t, hipStream_t);
template bool launch_scores_windows<8>(const Dims&, const ScoreArgs&, long long, size_t, hipStream_t);

}  // namespace ekv
