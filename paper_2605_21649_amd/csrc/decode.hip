// Sparse and dense alpha-entmax decode (paper Sec. 4.1, Sec. 4.4; Eq. 1-3).
//
// Entmax has no online rescaling: the threshold tau needs every candidate score.  The work is split:
//   pass 1 (many workgroups, HBM-bound): gather the K pages, z_j = a*scale*q.k_j, write z (4 B/token)
//           and one maximum per group of pages (64 tokens) to scratch.  bf16 pages go through the matrix cores:
//           an MFMA tile's 16 rows are 4 tokens x 4 channel quarters, so each lane's A operand is the
//           16 bytes of a fully coalesced load, its 16 columns are (query head, channel quarter); the
//           blocks with matching quarters are summed with two DPP quad steps.
//   pass 2 (one workgroup per (b,h)): the group maxima alone give the row maximum and a certified lower
//           bound of tau; only groups whose maximum exceeds it are read, their survivors compacted IN
//           ORDER into LDS; tau is solved there; p_j = (z_j - tau)^beta; V rows are gathered only where
//           p_j > 0.
// Short per-head lists take both passes in one launch with the scores in LDS (decode_row_kernel).
// All reductions have a fixed order, so results are bit-reproducible.
#include "ekv_scores.h"

namespace ekv {

constexpr int kSolveThreads = 1024;
constexpr int kSolveWaves = kSolveThreads / 64;
constexpr int kListCap = 4096;          // candidate entries the general path holds in LDS
constexpr int kSegs = 16;               // candidate lists are cut into this many segments, whatever the workgroup's size
constexpr int kSpillCap = 65536;        // entries of a row's overflow list in the workspace (longer lists: the row is streamed)
constexpr int kWaveGroups = 1024;       // up to this many group maxima are bounded by one wavefront, more by all of them
constexpr int kRoundLoads = 16;         // loads per lane and compaction round
constexpr int kWaveList = 256;          // candidates of a row that one wavefront finishes in registers

// ------------------------------------------------------------------------------------------
// pass 1: scores
// ------------------------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(1024) void unit_prefix_kernel(const ScoreArgs A, int32_t* pre_out) {
  __shared__ int wsum[16];
  const int gp = pmax_pages(A.P);
  block_exclusive_prefix<1024>(A.U, [&](int u) { return (unit_slots<MODE>(A, u) + gp - 1) / gp; }, pre_out, wsum);
}

// first item of a unit of n items that belongs to the part
__device__ __forceinline__ int part_first(const Part& p, int group, int n) {
  return p.count == 1 ? 0 : (int)(((unsigned)n * (unsigned)((p.index + group) % kXcds)) / kXcds);
}
__device__ __forceinline__ int part_length(const Part& p, int group, int n) {
  if (p.count == 1) return n;
  const unsigned i = (unsigned)((p.index + group) % kXcds);
  return (int)((unsigned)n * (i + 1) / kXcds - (unsigned)n * i / kXcds);
}

// Sums of G values over the 16 lanes of a DPP row, one head's sum in 16 / G lanes: two heads share a step by passing each
// other's half on, so eight heads take 8 exchanges instead of 32, and what follows is done once instead of per head.
// The pairs added are those of row16_sum, so the sums are its to the last bit.  The mirrors of the third and fourth step turn
// a quad round, which is why odd quads hold their heads in reverse.
template <int G> struct RowHeads {
  bool s1, s2, s3;                                 // which of two heads this lane keeps in steps 1, 2 and 3
  int head, keep;                                  // its head, and its number among the lanes with that head
  __device__ __forceinline__ explicit RowHeads(int c) {
    const int quad = c >> 2;
    s1 = ((c ^ quad) & 1) != 0; s2 = (((c >> 1) ^ quad) & 1) != 0; s3 = quad == 1 || quad == 2;
    head = G == 1 ? 0 : G == 2 ? s1 : G == 4 ? s1 + 2 * s2 : s1 + 2 * s2 + 4 * s3;
    keep = G == 1 ? c : G == 2 ? s2 + 2 * quad : G == 4 ? quad : quad >> 1;
  }
  template <int CTRL> static __device__ __forceinline__ float merge(bool second, float a, float b) {
    return (second ? b : a) + dpp_move<CTRL>(second ? a : b);
  }
  __device__ __forceinline__ float sum(const float (&v)[G]) const {
    float x[G];
#pragma unroll
    for (int g = 0; g < G; ++g) x[g] = v[g];
    if constexpr (G == 1) x[0] += dpp_move<0xB1>(x[0]);
    else {
#pragma unroll
      for (int g = 0; g < G / 2; ++g) x[g] = merge<0xB1>(s1, x[2 * g], x[2 * g + 1]);
    }
    if constexpr (G <= 2) x[0] += dpp_move<0x4E>(x[0]);
    else {
#pragma unroll
      for (int g = 0; g < G / 4; ++g) x[g] = merge<0x4E>(s2, x[2 * g], x[2 * g + 1]);
    }
    if constexpr (G <= 4) x[0] += dpp_move<0x141>(x[0]);
    else x[0] = merge<0x141>(s3, x[0], x[1]);
    return x[0] + dpp_move<0x140>(x[0]);
  }
};

// Any page size and either type, by steps of four tokens (the pages of an item hold 9 to 16 of them).  float32 caches, whose
// products stay float32, take FMAs and DPP row sums; bf16 pages other than 16, 32 and 64 the matrix cores, as below.
// The rows of 64 steps (four items) are resolved at once, one step per lane (page list -> block table), and handed out with
// v_readlane; K is read in chunks of 4 KiB with two register sets, the next chunk requested before the current one is
// consumed.  Page by page, with the lookups in front of every page and FMAs for either type, a wavefront had one step in
// flight.  Whole calls, us, before / now, four heads to a KV head: all pages of 2 x 262144 bf16 tokens in pages of 12
// 270.6 / 246.7 (1.07 GB, 4.6 TB/s in the pass; eight heads 377.7 / 283.7), per-head lists of 5000 tokens, 128 rows, pages of 8
// 37.8 / 29.0; float32, 2 x 131072 tokens in pages of 8 242.6 / 231.0, 128 lists of 5000 tokens in pages of 16 52.7 / 44.5.
// float32 rows by loads of whole lines and past the caches, as load_halves: 2 x 131072 tokens in pages of 16 229.6 -> 208.5,
// 262144 in pages of 48 237.3 -> 217.5 (227.5 page by page), refined step of 3 x 21003 tokens in pages of 8 109.0 -> 104.9.
// The sum runs over channels 8c..8c+7 in lane c and then over the lanes, as in decode_row_kernel and in the page scores:
// a threshold on page bounds compares them with what is solved from these scores.
template <typename T, int G, int MODE, bool STREAM, bool PRE_GLOBAL>
__global__ __launch_bounds__(kScoreThreads)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? (G <= 4 ? 8 : 6) : G == 1 ? 8 : G == 2 ? 6 : G == 4 ? 5 : 4)))
void decode_scores_steps_kernel(const ScoreArgs A) {
  constexpr bool DENSE = MODE == kAllPages, GROUPED = MODE != kPerHead, MFMA = sizeof(T) == 2;
  constexpr int CS = MFMA ? 4 : 2;                 // steps per chunk of 4 KiB
  constexpr int KS = 16 / G;                       // FMAs: steps whose scores the lanes of a row hold between them
  constexpr int NR = MFMA ? CS : 2 * CS;           // 16-byte loads per lane and chunk
  constexpr int NSET = (G + 3) / 4;
  constexpr int kStepLanes = 16, kBatchItems = 64 / kStepLanes;
  extern __shared__ int pre_lds[];
  __shared__ int wsum[kScoreWaves];
  const T* q = (const T*)A.q;
  const int P = A.P, Hq = A.Hq, Hkv = A.Hkv;
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
  const int gp = pmax_pages(P), spp = P / 4, spi = gp * spp;      // steps per page and per item
  const int item_steps = (spi + CS - 1) / CS * CS;                // in whole chunks; the last step again past the item's end
  const int my_st = min(lane % kStepLanes, spi - 1), my_pg = my_st / spp, my_t0 = 4 * (my_st - my_pg * spp);
  const int r = lane >> 4, c = lane & 15;          // FMAs: token of the step, the lane's channels
  const int m = lane & 15, j = lane >> 4, kq = m & 3, gl = m >> 2;      // matrix cores: as in decode_scores_mfma_kernel
  const T* k_pool = (const T*)A.k_pool + (MFMA ? gl * kD + (kq * 4 + j) * 8 : (r & 1) * kD + 8 * c + 4 * (r >> 1));
  const int ratio = Hq / Hkv;
  const Part part = PRE_GLOBAL || GROUPED ? Part{0, 1} : unit_part(A);
  if (!PRE_GLOBAL)
    block_exclusive_prefix<kScoreThreads>(A.U, [&](int u) {
      return part_length(part, u / ratio, (unit_slots<MODE>(A, u) + gp - 1) / gp); }, pre_lds, wsum);
  const int* pre = PRE_GLOBAL ? A.pre_g : pre_lds;
  const WaveItems wi = wave_item_range(pre, A.U, w, part);
  const int last = (DENSE ? A.Mmax : A.cap) - 1;

  int unit0 = wi.unit;                             // the batch's first unit, or one before
  for (int it0 = wi.begin; it0 < wi.end; it0 += kBatchItems) {
    // lane l: step l % 16 of item it0 + l / 16 (clamped to the last item and step): its row of K and how many of its
    // tokens are valid (-1: the step is not stored)
    int l_unit, l_grp, l_row, l_left;
    {
      const int my_it = min(it0 + lane / kStepLanes, wi.end - 1);
      const int lo = lane_last_at_most(pre, A.U, unit0, my_it, min(it0 + kBatchItems, wi.end) - 1);
      l_unit = lo;
      unit0 = __builtin_amdgcn_readlane(lo, 63);
      const int b = GROUPED ? lo / Hkv : lo / Hq, hkv = GROUPED ? lo - b * Hkv : (lo - b * Hq) / ratio;
      const int n = A.seq_lens[b], n_slots = DENSE ? clampi((n + P - 1) / P, 0, A.Mmax) : unit_slots<MODE>(A, lo);
      l_grp = my_it - pre[lo];
      if (!GROUPED && part.count != 1) l_grp += part_first(part, lo / ratio, (n_slots + gp - 1) / gp);
      const int slot = l_grp * gp + my_pg, slot_c = min(slot, last);
      const int lp = clampi(DENSE ? slot_c : A.page_idx[(size_t)lo * A.cap + slot_c], 0, A.Mmax - 1);
      const int phys = clampi(A.block_table[(size_t)b * A.Mmax + lp], 0, A.n_phys - 1);
      l_row = (phys * A.HkvPool + hkv) * P + my_t0;
      l_left = lane % kStepLanes < spi && slot < n_slots ? clampi(n - (lp * P + my_t0), 0, 4) : -1;
    }
    const uint64_t stored = __ballot(l_left >= 0);
    const int total = (min(it0 + kBatchItems, wi.end) - it0) * (item_steps / CS);

    // cursors: the chunk requested next and the one consumed next, as (first lane of the item, first step in it)
    int rq = 0, rq_s = 0, at = 0, at_s = 0;
    auto request = [&](uint4 (&a)[NR]) {
#pragma unroll
      for (int s = 0; s < CS; ++s) {
        const int row = __builtin_amdgcn_readlane(l_row, rq + rq_s + s);
        const T* p = k_pool + (size_t)(uint32_t)row * kD;
        if constexpr (MFMA) a[s] = load16<STREAM>(p);
        else {                                     // as load_halves: tokens 0 and 1, tokens 2 and 3
          a[2 * s] = load16<STREAM>(p);
          a[2 * s + 1] = load16<STREAM>(p + 2 * kD);
        }
      }
      rq_s += CS;
      if (rq_s == item_steps) { rq_s = 0; rq += kStepLanes; }
    };
    // state of the item being consumed, refreshed at its first chunk
    size_t row0 = 0;                               // first row of z / pmax written
    int grp = 0, lim = 0;                          // its stored steps
    uint4 bq[MFMA ? NSET : 1];
    float coef[MFMA ? 1 : G][8], zkeep[MFMA ? NSET : 1], wmax[MFMA ? NSET : 1];
    const RowHeads<G> rh(c);
    auto open_item = [&]() {
      const int unit = __builtin_amdgcn_readlane(l_unit, at);
      const int b = GROUPED ? unit / Hkv : unit / Hq, hq0 = GROUPED ? (unit - b * Hkv) * G : unit - b * Hq;
      grp = __builtin_amdgcn_readlane(l_grp, at);
      lim = __popc((uint32_t)(stored >> at) & 0xffffu);
      row0 = GROUPED ? (size_t)b * Hq + hq0 : (size_t)unit;
      const T* qr = q + ((size_t)b * Hq + hq0) * kD;
      if constexpr (MFMA) {
#pragma unroll
        for (int s = 0; s < NSET; ++s) {
          bq[s] = *reinterpret_cast<const uint4*>(qr + min(4 * s + gl, G - 1) * kD + kq * 32 + j * 8);
          wmax[s] = -INFINITY;
        }
      } else {
#pragma unroll
        for (int g = 0; g < G; ++g) load8<T>(qr + g * kD + 8 * c, coef[g]);
        wmax[0] = -INFINITY;
      }
    };
    auto consume = [&](const uint4 (&a)[NR]) {
      const int z0 = grp * spi * 4;                // first token of the item in its row of z
      int left[CS];
#pragma unroll
      for (int s = 0; s < CS; ++s) left[s] = __builtin_amdgcn_readlane(l_left, at + at_s + s);
      if constexpr (MFMA) {
#pragma unroll
        for (int s = 0; s < CS; ++s) {
          const bool valid = j < left[s];
#pragma unroll
          for (int cs = 0; cs < NSET; ++cs) {
            const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4_t d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[s]),
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
      } else {
#pragma unroll
        for (int s = 0; s < CS; ++s) {
          Raw8<float> raw = {__builtin_bit_cast(float4, a[2 * s]), __builtin_bit_cast(float4, a[2 * s + 1])};
          swap_halves(raw);
          float x[8], acc[G];
          widen8(raw, x);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            acc[g] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[g] = fmaf(coef[g][i], x[i], acc[g]);
          }
          const float v = rh.sum(acc), z = r < left[s] ? A.zscale * v : -INFINITY;
          if ((at_s + s) % KS == rh.keep) zkeep[0] = z;          // lane (r, c) keeps token r of that step
          wmax[0] = fmaxf(wmax[0], z);
        }
      }
      if constexpr (MFMA) {
        if (at_s + kq < lim) {                     // lane (j, head, kq) holds token j of the chunk's step kq
#pragma unroll
          for (int cs = 0; cs < NSET; ++cs) {
            const int g = 4 * cs + gl;
            if (g < G) A.zbuf[(row0 + g) * A.zstride + z0 + 4 * (at_s + kq) + j] = zkeep[cs];
          }
        }
      } else if ((at_s + CS) % KS == 0 || at_s + CS == item_steps) {
        const int st = at_s / KS * KS + rh.keep;
        if (st < lim) A.zbuf[(row0 + rh.head) * A.zstride + z0 + 4 * st + r] = zkeep[0];
      }
      at_s += CS;
      if (at_s == item_steps) {                     // last chunk of the item: its maximum (and its scores)
        at_s = 0; at += kStepLanes;
        if constexpr (MFMA) {
#pragma unroll
          for (int cs = 0; cs < NSET; ++cs) {
            float mx = wmax[cs];                   // equal over the four kq lanes of a head
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const int g = 4 * cs + gl;
            if (j == 0 && kq == 0 && g < G) A.pmax[(row0 + g) * A.n_chunks_max + grp] = mx;
          }
        } else {
          float mx = wmax[0];
          mx = fmaxf(mx, __shfl_xor(mx, 16));
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          if (r == 0 && rh.keep == 0) A.pmax[(row0 + rh.head) * A.n_chunks_max + grp] = mx;
        }
      }
    };

    // two chunks in flight; the query of a new item is requested before the next chunk (see decode_scores_mfma_kernel)
    uint4 a0[NR], a1[NR];
    request(a0);
    int ck = 0;
    for (; ck + 2 < total; ck += 2) {
      if (at_s == 0) open_item();
      __builtin_amdgcn_sched_barrier(0);
      request(a1);
      __builtin_amdgcn_sched_barrier(0);
      consume(a0);
      if (at_s == 0) open_item();
      __builtin_amdgcn_sched_barrier(0);
      request(a0);
      __builtin_amdgcn_sched_barrier(0);
      consume(a1);
    }
    if (at_s == 0) open_item();
    __builtin_amdgcn_sched_barrier(0);
    if (ck + 1 < total) {
      request(a1);
      __builtin_amdgcn_sched_barrier(0);
      consume(a0);
      consume(a1);                                 // of the same item: an item has at least two chunks
    } else {
      consume(a0);
    }
  }
}

// bf16 pages with P in {16, 32, 64}: matrix-core path.  Many resident wavefronts with little in flight each stream
// better than few with much: the kernel is compiled for eight wavefronts per SIMD and a wavefront holds two chunks
// of 16 tokens at a time (the next chunk is requested before the current one is consumed).  The page-list and block-table entries
// of up to 64 page slots are resolved at once, one slot per lane (two dependent vector loads per batch of 64 / GP
// items instead of two per page), and handed out with v_readlane.
template <int G, int MODE, int PT, bool STREAM, bool PRE_GLOBAL>
__global__ __launch_bounds__(kScoreThreads) __attribute__((amdgpu_waves_per_eu(G <= 4 ? 8 : 6)))
void decode_scores_mfma_kernel(const ScoreArgs A) {
  constexpr bool DENSE = MODE == kAllPages, GROUPED = MODE != kPerHead;
  constexpr int NSET = (G + 3) / 4;
  constexpr int KEEP = PT / 16;                   // 16-token chunks per page
  constexpr int GP = 64 / PT;                     // page slots per item
  constexpr int kBatchItems = 64 / GP;
  extern __shared__ int pre_lds[];
  __shared__ int wsum[kScoreWaves];
  const bf16_t* q = (const bf16_t*)A.q;
  const bf16_t* k_pool = (const bf16_t*)A.k_pool;
  const int Hq = A.Hq, Hkv = A.Hkv;
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
  const int m = lane & 15, j = lane >> 4;          // MFMA row/column index, K group
  const int kq = m & 3, gl = m >> 2;               // channel quarter; as a row: token of the step,
                                                   // as a column: head within the set
  // row (token gl of the step, quarter kq), K group j -> bytes [gl*256 + (kq*4+j)*16, +16) of the step
  const int lane_off = gl * kD + (kq * 4 + j) * 8;
  const int ratio = Hq / Hkv;
  const Part part = PRE_GLOBAL || GROUPED ? Part{0, 1} : unit_part(A);
  if (!PRE_GLOBAL)
    block_exclusive_prefix<kScoreThreads>(A.U, [&](int u) {
      return part_length(part, u / ratio, (unit_slots<MODE>(A, u) + GP - 1) / GP); }, pre_lds, wsum);
  const int* pre = PRE_GLOBAL ? A.pre_g : pre_lds;
  const WaveItems wi = wave_item_range(pre, A.U, w, part);
  const int last = (DENSE ? A.Mmax : A.cap) - 1;

  int unit0 = wi.unit;                             // the batch's first unit, or one before
  for (int it0 = wi.begin; it0 < wi.end; it0 += kBatchItems) {
    // lane l: page slot l % GP of item it0 + l / GP (clamped to the last item): its unit, logical and physical page
    int l_unit, l_lp, l_phys, l_grp;
    {
      const int my_it = min(it0 + lane / GP, wi.end - 1);
      const int lo = lane_last_at_most(pre, A.U, unit0, my_it, min(it0 + kBatchItems, wi.end) - 1);
      l_unit = lo;
      unit0 = __builtin_amdgcn_readlane(lo, 63);
      l_grp = my_it - pre[lo];
      if (!GROUPED && part.count != 1) l_grp += part_first(part, lo / ratio, (unit_slots<MODE>(A, lo) + GP - 1) / GP);
      const int slot = min(l_grp * GP + lane % GP, last);
      const int b = GROUPED ? lo / Hkv : lo / Hq;
      l_lp = clampi(DENSE ? slot : A.page_idx[(size_t)lo * A.cap + slot], 0, A.Mmax - 1);
      l_phys = clampi(A.block_table[(size_t)b * A.Mmax + l_lp], 0, A.n_phys - 1);
    }
    const int n_ck = (min(it0 + kBatchItems, wi.end) - it0) * 4;       // 16-token chunks of this batch

    // state of the item being consumed (wave-uniform), refreshed at its first chunk
    int n = 0, n_slots = 0, slot0 = 0, grp = 0;
    size_t row0 = 0;
    uint4 bq[NSET];
    float wmax[NSET];
    auto open_item = [&](int pg) {
      const int unit = __builtin_amdgcn_readlane(l_unit, pg);
      const int b = GROUPED ? unit / Hkv : unit / Hq;
      const int hq0 = GROUPED ? (unit % Hkv) * G : unit % Hq;
      grp = __builtin_amdgcn_readlane(l_grp, pg);
      slot0 = grp * GP;
      row0 = GROUPED ? (size_t)b * Hq + hq0 : (size_t)unit;      // first row of z / pmax written
      n = uniform_load(A.seq_lens + b);
      n_slots = DENSE ? clampi((n + PT - 1) / PT, 0, A.Mmax) : clampi(uniform_load(A.n_sel + unit), 0, A.cap);
#pragma unroll
      for (int s = 0; s < NSET; ++s) {
        const int g = min(4 * s + gl, G - 1);          // columns past the group repeat its last head (not stored)
        bq[s] = *reinterpret_cast<const uint4*>(q + ((size_t)b * Hq + hq0 + g) * kD + kq * 32 + j * 8);
        wmax[s] = -INFINITY;
      }
    };
    // chunk ck of the batch = tokens [16 t, 16 t + 16) of page slot pg = ck / KEEP, t = ck % KEEP
    auto request = [&](int ck, uint4 (&a)[4]) {
      const int pg = ck / KEEP, t = ck % KEEP;
      const int unit = __builtin_amdgcn_readlane(l_unit, pg);
      const int hkv = GROUPED ? unit % Hkv : (unit % Hq) / (Hq / Hkv);
      const int phys = __builtin_amdgcn_readlane(l_phys, pg);
      const bf16_t* kc = k_pool + (((size_t)phys * A.HkvPool + hkv) * PT + 16 * t) * kD + lane_off;
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = load16<STREAM>(kc + s * 4 * kD);
    };
    auto consume = [&](int ck, const uint4 (&a)[4]) {
      const int pg = ck / KEEP, t = ck % KEEP;
      const int slot = slot0 + pg % GP;
      const bool slot_ok = slot < n_slots;             // wave-uniform
      const int tok0 = __builtin_amdgcn_readlane(l_lp, pg) * PT + 16 * t + j;
      float zkeep[NSET];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        // result rows 4j..4j+3 belong to token j of the step
        const bool valid = slot_ok && tok0 + 4 * s < n;
#pragma unroll
        for (int cs = 0; cs < NSET; ++cs) {
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          const f32x4_t c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[s]),
                                                                    __builtin_bit_cast(bf16x8_t, bq[cs]), zero, 0, 0, 0);
          const float v01 = (kq & 1) ? c[1] : c[0], v23 = (kq & 1) ? c[3] : c[2];   // c[kq] in two selects
          float v = (kq & 2) ? v23 : v01;
          v += dpp_move<0xB1>(v);
          v += dpp_move<0x4E>(v);
          const float z = valid ? A.zscale * v : -INFINITY;
          if (s == kq) zkeep[cs] = z;                  // lane (j, head, kq) keeps token 4 kq + j of the chunk
          wmax[cs] = fmaxf(wmax[cs], z);
        }
      }
      if (slot_ok) {
#pragma unroll
        for (int cs = 0; cs < NSET; ++cs) {
          const int g = 4 * cs + gl;
          if (g < G) A.zbuf[(row0 + g) * A.zstride + (size_t)slot * PT + 16 * t + 4 * kq + j] = zkeep[cs];
        }
      }
      if (ck % 4 == 3) {                               // last chunk of the item: its maximum
#pragma unroll
        for (int cs = 0; cs < NSET; ++cs) {
          float mx = wmax[cs];                         // equal over the four kq lanes of a head
          mx = fmaxf(mx, __shfl_xor(mx, 16));
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          const int g = 4 * cs + gl;
          if (j == 0 && kq == 0 && g < G) A.pmax[(row0 + g) * A.n_chunks_max + grp] = mx;
        }
      }
    };

    // two chunks in flight, alternating register sets (n_ck is a multiple of 4).  Loads return in issue order, so the
    // query of a new item (every fourth chunk) is requested BEFORE the next chunk's K loads: waiting for it then
    // leaves those in flight.
    // Every request in the loop is unconditional (a load behind a branch makes the wait at the join drain the queue);
    // the last pair of chunks is taken after the loop.
    uint4 a0[4], a1[4];
    request(0, a0);
    int ck = 0;
    for (; ck + 2 < n_ck; ck += 2) {
      if (ck % 4 == 0) open_item(ck / KEEP);
      __builtin_amdgcn_sched_barrier(0);
      request(ck + 1, a1);
      __builtin_amdgcn_sched_barrier(0);
      consume(ck, a0);
      request(ck + 2, a0);
      __builtin_amdgcn_sched_barrier(0);
      consume(ck + 1, a1);
    }
    if (ck % 4 == 0) open_item(ck / KEEP);
    __builtin_amdgcn_sched_barrier(0);
    request(ck + 1, a1);
    __builtin_amdgcn_sched_barrier(0);
    consume(ck, a0);
    consume(ck + 1, a1);
  }
}

// ------------------------------------------------------------------------------------------
// pass 1b (long rows only): multi-workgroup candidate filter
// ------------------------------------------------------------------------------------------
// One workgroup of the solve cannot stream a row of a million scores, and it does not have to: the
// maxima of the 64-token groups written by pass 1 already bound tau from below.
//   level   (one workgroup per row): row maximum from the group maxima, then a 64-bin count histogram of
//           the group maxima above zmax-1.  Every counted group holds at least one score (its maximum)
//           in that bin, and an entry of bin g lies at least (g-i) bins above grid point i, so the counts
//           give a lower bound of the mass at every grid point; the highest grid point whose bound is >= 1
//           is a certified lower bound of tau.  Reads 4 bytes per 64 tokens.
//   compact (slices of kFilterSliceChunks groups x rows): only groups whose maximum exceeds that bound are
//           read (a few hundred per row); their scores above the bound are written out in order.
// The solve then gathers the survivors of all slices into LDS.

// Counts per bin above a base point give a lower bound of the mass at every grid point i.  Returns the
// highest i in [0, 64) whose bound sum_{g > i} cnt[g] * ((g - i - 0.02) * step)^beta reaches 1 (with a
// margin), or 0.  Called by all 1024 threads of a workgroup: 16 lanes per grid point, a DPP row sum, one
// barrier; `flags` is LDS [64].
template <int NB>
__device__ __forceinline__ int certified_level(const int* cnt, float step, float beta, int ibeta, int* flags) {
  const int i = threadIdx.x >> 4, l = threadIdx.x & 15;
  float lb = 0.f;
#pragma unroll
  for (int g = l; g < NB; g += 16)
    if (g > i) lb += (float)cnt[g] * pow_beta(((float)(g - i) - 0.02f) * step, beta, ibeta);
  lb = row16_sum(lb);
  if (l == 0) flags[i] = lb >= 1.0001f ? 1 : 0;
  __syncthreads();
  const uint64_t okm = __ballot(flags[threadIdx.x & 63] != 0);
  return okm ? 63 - __clzll(okm) : 0;
}

constexpr int kFilterThreads = 1024;
constexpr int kFilterWaves = kFilterThreads / 64;
constexpr int kFilterWaveChunks = kFilterSliceChunks / kFilterWaves;   // groups per wavefront: 32
static_assert(kFilterWaveChunks <= 64, "one ballot covers a wavefront's groups");

struct FilterArgs {
  const int32_t* seq_lens; const int32_t* n_sel; const float* zbuf; const float* pmax;
  int32_t* fcount; float* frow; float* flist_u; int32_t* flist_pos;
  int Hq, Hkv, grouped, P, n_slices_max, max_slots, n_chunks_max;
  size_t zstride;
  float beta; int ibeta;
};

template <bool DENSE>
__device__ __forceinline__ int filter_n_slots(const FilterArgs& A, int row) {
  const int lrow = A.grouped ? (row / A.Hq) * A.Hkv + (row % A.Hq) / (A.Hq / A.Hkv) : row;
  const int slots = DENSE ? (A.seq_lens[row / A.Hq] + A.P - 1) / A.P : A.n_sel[lrow];
  return clampi(slots, 0, A.max_slots);
}

template <bool DENSE>
__global__ __launch_bounds__(kFilterThreads) void filter_level_kernel(const FilterArgs A) {
  __shared__ float red[kFilterWaves];
  __shared__ int hist[64];
  __shared__ int flags[64];
  const int row = blockIdx.x, tid = threadIdx.x;
  const int gp = pmax_pages(A.P);
  const int n_chunks = (filter_n_slots<DENSE>(A, row) + gp - 1) / gp;
  if (n_chunks <= kPreGroups) return;                         // short row: the solve reads its group maxima itself
  const float* pm = A.pmax + (size_t)row * A.n_chunks_max;
  float mx = -INFINITY;
  for (int i0 = 0; i0 < n_chunks; i0 += kFilterThreads * 16) {
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = pm[min(i0 + k * kFilterThreads + tid, n_chunks - 1)];
#pragma unroll
    for (int k = 0; k < 16; ++k) mx = fmaxf(mx, v[k]);        // clamped repeats do not change a maximum
  }
  if (tid < 64) hist[tid] = 0;
  const float zmax = block_max(mx, red);
  if (!(zmax > -INFINITY)) {                                  // empty row, or nothing but masked tokens
    if (tid == 0) { A.frow[2 * row] = -INFINITY; A.frow[2 * row + 1] = 0.f; }
    return;
  }
  const float thr0 = zmax - 1.0f - 4e-6f * fmaxf(1.f, fabsf(zmax));
  const float width = zmax - thr0, step = width * (1.0f / 64.0f), inv_step = 64.0f / width;
  for (int i0 = 0; i0 < n_chunks; i0 += kFilterThreads * 16) {
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = pm[min(i0 + k * kFilterThreads + tid, n_chunks - 1)];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (i0 + k * kFilterThreads + tid < n_chunks && v[k] > thr0)
        atomicAdd(&hist[min(63, (int)((v[k] - thr0) * inv_step))], 1);
  }
  __syncthreads();
  int level = certified_level<64>(hist, step, A.beta, A.ibeta, flags);
  float thr = thr0 + (float)level * step;
  // A flat row crowds its group maxima into the last few steps below the maximum, and most groups still pass: the
  // same certificate on a histogram of [bound, maximum] resolves them (twice at most).
  for (int refine = 0; refine < 2; ++refine) {
    int above = 0;
    for (int g = level; g < 64; ++g) above += hist[g];
    if (above <= 1024) break;
    __syncthreads();                                          // every thread has read the counts
    const float w2 = zmax - thr, step2 = w2 * (1.0f / 64.0f), inv_step2 = 64.0f / w2;
    if (tid < 64) hist[tid] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n_chunks; i0 += kFilterThreads * 16) {
      float v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = pm[min(i0 + k * kFilterThreads + tid, n_chunks - 1)];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (i0 + k * kFilterThreads + tid < n_chunks && v[k] > thr)
          atomicAdd(&hist[min(63, (int)((v[k] - thr) * inv_step2))], 1);
    }
    __syncthreads();
    level = certified_level<64>(hist, step2, A.beta, A.ibeta, flags);
    if (level == 0) break;
    thr += (float)level * step2;
  }
  if (tid == 0) { A.frow[2 * row] = zmax; A.frow[2 * row + 1] = thr; }
}

// Scores of up to four groups of a wavefront at once (lane = token of the group), -inf where masked.
__device__ __forceinline__ void filter_group_scores(const float* zr, const int (&chunk)[4], int n_valid, int ct,
                                                    int n_cand, float (&z)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 4; ++k) z[k] = zr[min(chunk[min(k, n_valid - 1)] * ct + min(lane, ct - 1), n_cand - 1)];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (k >= n_valid || lane >= ct || chunk[k] * ct + lane >= n_cand) z[k] = -INFINITY;
}

template <bool DENSE>
__global__ __launch_bounds__(kFilterThreads) void filter_compact_kernel(const FilterArgs A) {
  __shared__ int wtot[kFilterWaves];
  const int row = blockIdx.y, slice = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  const int gp = pmax_pages(A.P), ct = gp * A.P;              // tokens per group (<= 64)
  const int n_slots = filter_n_slots<DENSE>(A, row);
  const int n_cand = n_slots * A.P, n_chunks = (n_slots + gp - 1) / gp;
  const int c0 = slice * kFilterSliceChunks;
  if (c0 >= n_chunks || n_chunks <= kPreGroups) return;      // past the row's end, or a short row (see the level pass)
  const float zmax = A.frow[2 * row], thr = A.frow[2 * row + 1];
  const float* zr = A.zbuf + (size_t)row * A.zstride;
  const float* pm = A.pmax + (size_t)row * A.n_chunks_max;
  // groups of this wavefront whose maximum can hold a survivor
  const int cw = c0 + w * kFilterWaveChunks;
  const float pmv = pm[min(cw + min(lane, kFilterWaveChunks - 1), n_chunks - 1)];
  const uint64_t pass = __ballot(lane < kFilterWaveChunks && cw + lane < n_chunks && pmv > thr);
  int c = 0;
  for (uint64_t m = pass; m != 0;) {
    int chunk[4], nv = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (m != 0) { chunk[k] = cw + __builtin_ctzll(m); m &= m - 1; ++nv; } else chunk[k] = cw;
    float z[4];
    filter_group_scores(zr, chunk, nv, ct, n_cand, z);
#pragma unroll
    for (int k = 0; k < 4; ++k) c += __popcll(__ballot(z[k] > thr));
  }
  if (lane == 0) wtot[w] = c;
  __syncthreads();
  int off = 0, tot = 0;
  for (int i = 0; i < kFilterWaves; ++i) { const int ci = wtot[i]; if (i < w) off += ci; tot += ci; }
  if (tid == 0) A.fcount[(size_t)row * A.n_slices_max + slice] = tot;
  if (c == 0) return;
  float* lu = A.flist_u + ((size_t)row * A.n_slices_max + slice) * kFilterSliceCap;
  int32_t* lp = A.flist_pos + ((size_t)row * A.n_slices_max + slice) * kFilterSliceCap;
  for (uint64_t m = pass; m != 0;) {                          // second sweep (from cache): ordered write
    int chunk[4], nv = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (m != 0) { chunk[k] = cw + __builtin_ctzll(m); m &= m - 1; ++nv; } else chunk[k] = cw;
    float z[4];
    filter_group_scores(zr, chunk, nv, ct, n_cand, z);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = z[k] > thr;
      const uint64_t mk = __ballot(in);
      const int o = off + __popcll(mk & lt);
      if (in && o < kFilterSliceCap) { lu[o] = z[k] - zmax; lp[o] = chunk[k] * ct + lane; }
      off += __popcll(mk);
    }
  }
}

// ------------------------------------------------------------------------------------------
// pass 2: threshold, probabilities, weighted value sum
// ------------------------------------------------------------------------------------------
// NW wavefronts, SEG candidates per segment, LIST entries of the general path's list, up to GROUPS groups per row.
template <int NW, int SEG, int LIST, int GROUPS>
struct SolveSharedT {
  static constexpr int kWaves = NW, kSegCap = SEG, kListCap = LIST, kMaxGroups = GROUPS;
  static constexpr bool kOverflows = true;   // a segment may have more candidates than it holds
  union {
    // Candidates, z - zmax (float bits) and position in the candidate order; segment i is [i * kSegCap, (i + 1) * kSegCap).
    uint2 seg[kSegs * SEG];
    struct {                      // the general path's one list, and the support of a row that one wavefront finishes
      float list_u[LIST];
      int32_t list_pos[LIST];
      uint32_t list_row[LIST];    // their V row: (phys*Hkv + hkv)*P + tok
    };
  };
  uint16_t glist[GROUPS];         // the groups that can hold a candidate, ascending
  float obuf[kSegs][kD];
  float red[2][kSegs][3];
  int wcount[2][kSegs];
  int pre[kSegs + 1];             // exclusive prefix of the segments' lengths
  float red1[NW];
  int hist[64];                   // candidates per 1/64 slice of [thr, zmax] (threshold tightening)
  int flags[64];
  float zmax, bound;              // row maximum, certified lower bound of tau relative to it
  int n_pass;
};
static_assert(kPreGroups <= 65536, "group numbers are 16 bits wide");
// One row per compute unit: sixteen wavefronts and most of the LDS, rows of any length.  Sixteen maxima per thread take a row
// of a million tokens from its group maxima in one launch.
using SolveShared = SolveSharedT<kSolveWaves, 768, kListCap, kPreGroups>;
// Four rows per compute unit (registers allow 16 wavefronts, LDS four times 34 KB): many short rows, whose usual solve is
// one wavefront's work.  192 entries per segment take all of a row of up to 2048 tokens whatever the page size (180 in
// groups of 60), so that such a row's result is that of its one-launch decode to the last bit however flat it is.
using SolveSharedMany = SolveSharedT<4, 192, 2048, kWaveGroups / 4>;
constexpr int kOneGroups = kSegs;           // a row of at most this many groups has one in each segment

// Many rows of at most kOneGroups groups (lists shared per KV head; per-head lists of that length are decoded in one launch,
// below): one wavefront each.  A segment holds all tokens of its one group, so nothing overflows, and 9 KB of LDS let a
// compute unit keep as many rows as its registers do.
struct SolveSharedOne {
  static constexpr int kWaves = 1, kSegCap = 64, kMaxGroups = kOneGroups;
  static constexpr bool kOverflows = false;
  union {
    uint2 seg[kSegs * kSegCap];
    float obuf[kSegs][kD];        // a segment's partial output replaces its candidates
    struct { float list_u[kWaveList]; int32_t list_pos[kWaveList]; uint32_t list_row[kWaveList]; };
  };
  float red[2][kSegs][3];
  int wcount[2][kSegs];
  int pre[kSegs + 1];
  float red1[1];
  uint16_t glist[kOneGroups];
  float zmax, bound;
  int n_pass;
};
static_assert(sizeof(float[kD]) == sizeof(uint2[SolveSharedOne::kSegCap]), "partial output i covers segment i and no other");

// Sum of one value per segment (or wavefront) kept in LDS at a stride: one read per lane and a DPP row sum, the same in
// every wavefront (a loop reads LDS sixteen times in a row).
static_assert(kSegs == 16 && kSolveWaves == 16, "one DPP row");
template <int N = kSegs>
__device__ __forceinline__ float sum_waves(const float* v, int stride) {
  const int l = threadIdx.x & 15;
  return row16_sum(l < N ? v[l * stride] : 0.f);
}
template <int N = kSegs>
__device__ __forceinline__ int sum_waves_i(const int* v, int stride) {
  const int l = threadIdx.x & 15;
  int x = l < N ? v[l * stride] : 0;
  x += dpp_move_i<0xB1>(x); x += dpp_move_i<0x4E>(x); x += dpp_move_i<0x141>(x); x += dpp_move_i<0x140>(x);
  return __builtin_amdgcn_readfirstlane(x);
}

// Candidate source: the compacted list (in LDS, or the row's overflow list in the workspace), or the score row itself.
struct ListSrc {
  const float* u; const int32_t* pos; int n;
  __device__ __forceinline__ float get_u(int i) const { return u[i]; }
  __device__ __forceinline__ int get_pos(int i) const { return pos[i]; }
};
struct RowSrc {
  const float* z; int n; float zmax;
  __device__ __forceinline__ float get_u(int i) const { return z[i] - zmax; }
  __device__ __forceinline__ int get_pos(int i) const { return i; }
};

// F = sum (u-tau)_+^beta, D = beta * sum (u-tau)_+^(beta-1), cnt = #{u > tau}; one barrier per call
// (double-buffered by `parity`).
template <typename Src, typename SH>
__device__ __forceinline__ void eval_mass(const Src& src, float tau, float beta, int ibeta, SH& sh,
                                          int parity, float& F, float& D, int& cnt) {
  constexpr int NT = 64 * SH::kWaves;
  float f = 0.f, d = 0.f; int c = 0;
  for (int i0 = threadIdx.x; i0 < src.n; i0 += 8 * NT) {     // eight loads in flight per thread
    float u[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) u[j] = src.get_u(min(i0 + j * NT, src.n - 1));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float x = i0 + j * NT < src.n ? u[j] - tau : -1.f;
      if (x > 0.f) { f += pow_beta(x, beta, ibeta); d += pow_beta_m1(x, beta, ibeta); ++c; }
    }
  }
  f = wave_sum(f); d = wave_sum(d); c = wave_sum_i(c);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sh.red[parity][w][0] = f; sh.red[parity][w][1] = d; sh.red[parity][w][2] = __int_as_float(c); }
  __syncthreads();
  F = sum_waves<SH::kWaves>(&sh.red[parity][0][0], 3);
  D = beta * sum_waves<SH::kWaves>(&sh.red[parity][0][1], 3);
  cnt = sum_waves_i<SH::kWaves>(reinterpret_cast<const int*>(&sh.red[parity][0][2]), 3);
}

// f += x^beta, d += x^(beta - 1) (0 for x = 0), x >= 0.  The products are spelled out, and what follows of the solve is
// compiled without contraction, so that every kernel that solves a row takes the same steps to the last bit.
template <int IB>
__device__ __forceinline__ void add_mass(float x, float beta, float& f, float& d) {
  if constexpr (IB == 0) {
    if (x > 0.f) { f += pow_beta(x, beta, 0); d += pow_beta_m1(x, beta, 0); }
  } else {
    const float y = IB == 1 ? (x > 0.f ? 1.f : 0.f) : pow_beta_m1(x, beta, IB);
    f = fmaf(x, y, f);
    d += y;
  }
}

// Root of sum (u - tau)_+^beta = 1 for u <= 0 with max u = 0: tau in [lo_init, 0), where lo_init >= -1
// is any point with mass >= 1.
// Safeguarded iteration inside a bracket [lo,hi], F(lo) >= 1 > F(hi).  From a left point the step is
// the exact root for the current support when beta is 1 or 2 (closed forms), Newton otherwise; from a
// right point a Newton step (F is convex, so it lands left of the root).  For beta in {1,2} the root is
// accepted as exact once a closed-form step leaves the support count unchanged.
// `eval(tau, F, D, cnt)` evaluates the mass, its negated derivative and the support count at tau.
// `seed`: where to take the first evaluation if it lies inside the bracket (NaN: none); `evals` counts
// the evaluations.
template <typename Eval>
__device__ __forceinline__ float solve_tau_core(Eval&& eval, float lo_init, float seed, int ibeta, int& supp,
                                                int& evals) {
#pragma clang fp contract(off)
  float lo = lo_init, hi = 0.f;
  float tau = (seed > lo && seed < hi) ? seed : lo;
  int pending_cnt = -1;
  int cnt = 0;
  bool last = false;                                         // tau is settled; evaluated once more for its support
  evals = 0;
  for (int it = 0;; ++it) {                                  // one call of `eval`: it is most of the code of every solve
    float F, D;
    eval(tau, F, D, cnt);
    ++evals;
    if (last) break;
    if (pending_cnt >= 0 && cnt == pending_cnt) break;       // exact step kept the support: done
    if (fabsf(F - 1.0f) <= 4e-7f) break;                     // float32 resolution of F: tau is the root
    pending_cnt = -1;
    float step;
    if (F >= 1.0f) {
      lo = tau;
      const float e = F - 1.0f;
      if (ibeta == 1) { step = e / (float)cnt; pending_cnt = cnt; }
      else if (ibeta == 2) {
        const float A = 0.5f * D;                            // sum (u - tau)
        const float disc = fmaf(A, A, -(float)cnt * e);
        if (disc > 0.f) { step = e / (A + sqrtf(disc)); pending_cnt = cnt; }
        else step = e / D;
      } else step = e / D;
    } else {
      hi = tau;
      step = D > 0.f ? (F - 1.0f) / D : -INFINITY;
    }
    float next = tau + step;
    if (next == tau) break;                                  // no representable progress
    if (!(next > lo && next < hi)) { next = 0.5f * (lo + hi); pending_cnt = -1; }
    last = hi - lo <= 1.2e-7f || (pending_cnt < 0 && fabsf(next - tau) <= 6e-8f);
    tau = next;
    if (it == 63 && !last) break;
  }
  supp = cnt;
  return tau;
}

// The whole workgroup iterates (one barrier per evaluation).
template <typename Src, typename SH>
__device__ __forceinline__ float solve_tau(const Src& src, float lo_init, float seed, float beta, int ibeta,
                                           SH& sh, int& supp, int& evals) {
  int parity = 0;
  return solve_tau_core([&](float tau, float& F, float& D, int& cnt) {
    eval_mass(src, tau, beta, ibeta, sh, parity, F, D, cnt);
    parity ^= 1;
  }, lo_init, seed, ibeta, supp, evals);
}

// Short candidate lists (at most kWaveList entries, the usual case once the certified bound has been
// applied): one wavefront holds them in registers and iterates without any barrier; the result is handed
// to the other wavefronts through LDS.  Called by the whole workgroup.
// entries of one wavefront in registers (u[k] of lane l is list entry l + 64 k, -inf past the end)
template <int KW>
__device__ __forceinline__ float solve_tau_regs(const float (&u)[KW], float lo_init, float seed, float beta, int ibeta,
                                                int& supp, int& evals) {
  return with_beta(ibeta, [&](auto ib) {
    constexpr int IB = decltype(ib)::value;
    return solve_tau_core([&](float t, float& F, float& D, int& cnt) {
      float f = 0.f, d = 0.f;
      cnt = 0;
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const float x = fmaxf(u[k] - t, 0.f);
        add_mass<IB>(x, beta, f, d);
        cnt += __popcll(__ballot(x > 0.f));
      }
      F = wave_sum(f); D = beta * wave_sum(d);
    }, lo_init, seed, IB, supp, evals);
  });
}
template <typename SH>
__device__ __forceinline__ float solve_tau_wave(const float* list_u, int n, float lo_init, float seed, float beta,
                                                int ibeta, SH& sh, int& supp, int& evals) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    float u[kWaveList / 64];
#pragma unroll
    for (int k = 0; k < kWaveList / 64; ++k) u[k] = lane + 64 * k < n ? list_u[lane + 64 * k] : -INFINITY;
    int sp = 0, ev = 0;
    const float tau = solve_tau_regs(u, lo_init, seed, beta, ibeta, sp, ev);
    if (lane == 0) { sh.red1[0] = tau; sh.wcount[0][0] = sp; sh.wcount[0][1] = ev; }
  }
  __syncthreads();
  supp = sh.wcount[0][0];
  evals = sh.wcount[0][1];
  return sh.red1[0];
}

struct SolveArgs {
  const void* v_pool;
  const int32_t* block_table; const int32_t* seq_lens; const int32_t* page_idx; const int32_t* n_sel;
  const float* zbuf; const float* pmax;
  float* out; float* tau_out; int32_t* supp_out;
  ekv_decode_extras ex;
  int Hq, Hkv, P, Mmax, cap, n_chunks_max, n_phys;
  size_t zstride;
  float a, beta; int ibeta;
  // results of the filter passes (null for short rows)
  const int32_t* fcount; const float* frow; const float* flist_u; const int32_t* flist_pos; int n_slices_max;
  int grouped;
  int HkvPool;
  // per-row overflow list in the workspace for candidate lists beyond the LDS list (null / 0 when rows cannot have one)
  float* spill_u; int32_t* spill_pos; int spill_cap;
};

// V row index (phys*Hkv + hkv)*P + tok of candidate position `pos`.
template <bool DENSE>
__device__ __forceinline__ uint32_t v_row_of(const SolveArgs& A, int b, int bh, int hkv, int pos) {
  const int slot = pos / A.P, tok = pos - slot * A.P;
  const int lp = DENSE ? slot : clampi(A.page_idx[(size_t)bh * A.cap + slot], 0, A.Mmax - 1);
  const int phys = clampi(A.block_table[(size_t)b * A.Mmax + lp], 0, A.n_phys - 1);
  return (uint32_t)((phys * A.HkvPool + hkv) * A.P + tok);
}
template <bool DENSE>
__device__ __forceinline__ int token_of(const SolveArgs& A, int bh, int pos) {
  const int slot = pos / A.P, tok = pos - slot * A.P;
  const int lp = DENSE ? slot : A.page_idx[(size_t)bh * A.cap + slot];
  return lp * A.P + tok;
}

// Partial output of one segment: the per-lane sums acc[8] (channels 8c..8c+7 of a row slot) of one wavefront.
template <typename SH>
__device__ __forceinline__ void store_partial(float (&acc)[8], SH& sh, int seg) {
  const int lane = threadIdx.x & 63, c = lane & 15;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    acc[i] += __shfl_xor(acc[i], 16);
    acc[i] += __shfl_xor(acc[i], 32);
  }
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) sh.obuf[seg][8 * c + i] = acc[i];
  }
}
// The segments' partial outputs, added in their order.  Starts with a barrier.
template <int N = kSegs, typename SH>
__device__ __forceinline__ void sum_partials(const SH& sh, float* __restrict__ out) {
  __syncthreads();
  for (int c = threadIdx.x; c < kD; c += 64 * SH::kWaves) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) s += sh.obuf[i][c];
    out[c] = s;
  }
}

// Weighted sum of the V rows of the `tot` support entries in LDS (weight list_u[e], row list_row[e]): 64 row
// slots x 16 lanes, eight independent 16-byte loads in flight per lane (clamped entries carry weight 0).  A row
// slot adds its entries in ascending order.
template <typename T, typename SH>
__device__ __forceinline__ void gather_support(const T* __restrict__ v_pool, const SH& sh, int tot, float (&acc)[8]) {
  const int rs = threadIdx.x >> 4, c = threadIdx.x & 15;
  constexpr int kSlots = 4 * SH::kWaves;
  for (int e0 = 0; e0 < tot; e0 += 8 * kSlots) {
    Raw8<T> vr[8]; float pw[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = e0 + kSlots * j + rs;
      const int ec = min(e, tot - 1);
      pw[j] = e < tot ? sh.list_u[ec] : 0.f;
      load_raw8(v_pool + (size_t)sh.list_row[ec] * kD + 8 * c, vr[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float vv[8];
      widen8(vr[j], vv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fmaf(pw[j], vv[i], acc[i]);
    }
  }
}

// Ranges of a row's candidates, as a wavefront that finishes the row needs them.
struct RowRef { int b, bh, lrow, hkv, n_cand, chunk_tokens, n_chunks; };

// A certified lower bound of tau (relative to the row maximum) from group maxima relative to it: every group holds at
// least its maximum, so the mass of the maxima alone is a lower bound of the mass, and any point where it is >= 1 lies
// left of tau.  F^(1/beta) is a norm of (u - t)_+, hence convex in t: Newton's steps on it from a point where F >= 1
// stay left of the root.  They aim at a mass of 1.0001, which covers the rounding of the sums.  Below beta = 1 (alpha
// above 2) that fails, but sum x^beta >= (sum x)^beta there, so the point where the plain sum reaches 1 is a bound.
// `sums(f, d)` adds f and d up over all threads that hold maxima.
template <int R, typename Sums>
__device__ __forceinline__ float group_bound(const float (&u)[R], float t0, float beta, int ibeta, Sums&& sums) {
#pragma clang fp contract(off)
  if (beta < 1.f) { beta = 1.f; ibeta = 1; }
  return with_beta(ibeta, [&](auto ib) {
#pragma clang fp contract(off)
    constexpr int IB = decltype(ib)::value;
    const float target = 1.0f + 1e-4f / beta;
    float t = t0;
    for (int it = 0; it < 8; ++it) {
      float f = 0.f, d = 0.f;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        add_mass<IB>(fmaxf(u[k] - t, 0.f), beta, f, d);
      }
      sums(f, d);
      const float r = IB == 1 ? f : IB == 2 ? __builtin_amdgcn_sqrtf(f) : __builtin_exp2f(__builtin_log2f(f) / beta);
      if (!(r > target)) break;
      t += (r - target) * f * __builtin_amdgcn_rcpf(r * d);
      if (r < 1.02f) break;                                   // within two per cent of the norm: close enough
    }
    return t;
  });
}

// The end of a row whose candidates are few: threshold, support and weighted value sum by ONE wavefront, KW entries per
// lane, taken from the segments (ends: where segment `lane` ends among the candidates).  V rows are looked up while the
// threshold is solved.
template <typename T, bool DENSE, int KW, typename SH>
__device__ __forceinline__ void finish_row_wave(const SolveArgs& A, const RowRef& R, int n_list, int ends, float lo_u, float zmax,
                                                float seed_u, SH& sh) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1ull;
  const T* v_pool = (const T*)A.v_pool;
  float* lu = sh.list_u; int32_t* lp = sh.list_pos; uint32_t* lr = sh.list_row;
  float u[KW]; int pos[KW]; uint32_t row[KW];
  int at[KW];
  if constexpr (KW == 1) {                                            // segment ends from lane to lane: no LDS latency
    int seg = 0, start = 0;
#pragma unroll
    for (int d = 0; d < kSegs - 1; ++d) {
      const int end = __builtin_amdgcn_readlane(ends, d);
      if (end <= lane) { seg = d + 1; start = end; }
    }
    at[0] = seg * SH::kSegCap + min(lane - start, SH::kSegCap - 1);
  } else {
    if (lane < kSegs) sh.pre[lane + 1] = ends;
    if (lane == 0) sh.pre[0] = 0;
    wave_order();
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int e = lane + 64 * k;
      int seg = 0;                                                    // last segment that starts at or before e
#pragma unroll
      for (int d = kSegs / 2; d >= 1; d >>= 1) seg += sh.pre[seg + d] <= e ? d : 0;
      at[k] = seg * SH::kSegCap + min(e - sh.pre[seg], SH::kSegCap - 1);
    }
  }
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const int e = lane + 64 * k;
    const uint2 c = sh.seg[at[k]];
    u[k] = e < n_list ? __uint_as_float(c.x) : -INFINITY;
    pos[k] = e < n_list ? (int)c.y : 0;
  }
  wave_order();                                                       // the support is written over the segments below
#pragma unroll
  for (int k = 0; k < KW; ++k) row[k] = v_row_of<DENSE>(A, R.b, R.lrow, R.hkv, pos[k]);     // clamped, unconditional
  int supp = 0, evals = 0;
  const float tau_u = solve_tau_regs<KW>(u, lo_u, seed_u, A.beta, A.ibeta, supp, evals);
  // ordered compaction of the support: (p, row, position) of entry e = lane + 64 k, k-major = candidate order
  int n_sup = 0;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    const float x = u[k] - tau_u;
    const bool in = x > 0.f;
    const uint64_t mk = __ballot(in);
    if (in) {
      const int o = n_sup + __popcll(mk & lt);
      lu[o] = pow_beta(x, A.beta, A.ibeta);
      lr[o] = row[k];
      lp[o] = pos[k];
    }
    n_sup += __popcll(mk);
  }
  __builtin_amdgcn_wave_barrier();
  // weighted value sum: 4 row slots x 16 lanes, batches of 8 independent 16-byte loads per lane
  const int rs = lane >> 4, c = lane & 15;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int e0 = 0; e0 < n_sup; e0 += 32) {
    Raw8<T> vr[8]; float pw[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = e0 + 4 * j + rs;
      const int ec = min(e, n_sup - 1);                              // clamped: loads stay unconditional
      pw[j] = e < n_sup ? lu[ec] : 0.f;
      load_raw8(v_pool + (size_t)lr[ec] * kD + 8 * c, vr[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float vv[8];
      widen8(vr[j], vv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fmaf(pw[j], vv[i], acc[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    acc[i] += __shfl_xor(acc[i], 16);
    acc[i] += __shfl_xor(acc[i], 32);
  }
  float* out = A.out + (size_t)R.bh * kD;
  if (lane < 16) {
    *reinterpret_cast<float4*>(out + 8 * c) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    *reinterpret_cast<float4*>(out + 8 * c + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
  if (A.ex.support_tokens != nullptr) {
    int32_t* dst = A.ex.support_tokens + (size_t)R.bh * A.ex.support_cap;
    for (int e = lane; e < n_sup && e < A.ex.support_cap; e += 64) dst[e] = token_of<DENSE>(A, R.lrow, lp[e]);
  }
  if (lane == 0) {
    A.tau_out[R.bh] = tau_u + zmax; A.supp_out[R.bh] = supp;
    if (A.ex.solve_evals != nullptr) A.ex.solve_evals[R.bh] = evals;
  }
}

// Outputs of a row without any valid candidate, written by one wavefront.
template <bool DENSE>
__device__ __forceinline__ void empty_row_wave(const SolveArgs& A, int bh) {
  const int lane = threadIdx.x & 63;
  if (lane < kD / 4) *reinterpret_cast<float4*>(A.out + (size_t)bh * kD + 4 * lane) = make_float4(0.f, 0.f, 0.f, 0.f);
  if (lane == 0) {
    A.tau_out[bh] = INFINITY; A.supp_out[bh] = 0;
    if (A.ex.solve_evals != nullptr) A.ex.solve_evals[bh] = 0;
    if (A.ex.tau_ref != nullptr && A.ex.kept_mass_ref != nullptr) A.ex.kept_mass_ref[bh] = 0.f;
    if (A.ex.tau_ref != nullptr && A.ex.kept_supp_ref != nullptr) A.ex.kept_supp_ref[bh] = 0;
    if (DENSE && A.ex.lse != nullptr) A.ex.lse[bh] = -INFINITY;
  }
}

// Maxima of a row's groups -> row maximum, bound of tau and the ordered list of the groups above it (sh.zmax, sh.bound,
// sh.n_pass, sh.glist), by the wavefronts whose turn it is: group (w * 64 * R + 64 k + lane) sits in register k.  With one
// wavefront (rows of up to kWaveGroups groups: up to 65 536 candidates) nothing in here waits at a barrier.
template <int R, bool ONE_WAVE, typename Max, typename SH>
__device__ __forceinline__ void bound_groups(Max&& group_max, int n_chunks, float beta, int ibeta, SH& sh) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, w = ONE_WAVE ? 0 : uniform(threadIdx.x >> 6);
  const uint64_t lt = (1ull << lane) - 1ull;
  const int g0 = w * 64 * R + lane, last = max(n_chunks - 1, 0);
  float m[R];
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < R; ++k) m[k] = group_max(min(g0 + 64 * k, last));
#pragma unroll
  for (int k = 0; k < R; ++k) { m[k] = g0 + 64 * k < n_chunks ? m[k] : -INFINITY; mx = fmaxf(mx, m[k]); }
  const float zmax = ONE_WAVE ? wave_max(mx) : block_max(mx, sh.red1);
  const float eps = 4e-6f * fmaxf(1.f, fabsf(zmax));
  float t = -1.0f - eps;
  int n_pass = 0;
  if (zmax > -INFINITY) {                                             // the same for all threads
#pragma unroll
    for (int k = 0; k < R; ++k) m[k] -= zmax;
    int parity = 0;
    t = group_bound(m, t, beta, ibeta, [&](float& f, float& d) {
      f = wave_sum(f); d = wave_sum(d);
      if (!ONE_WAVE) {
        if (lane == 0) { sh.red[parity][w][0] = f; sh.red[parity][w][1] = d; }
        __syncthreads();
        f = sum_waves<SH::kWaves>(&sh.red[parity][0][0], 3); d = sum_waves<SH::kWaves>(&sh.red[parity][0][1], 3);
        parity ^= 1;
      }
    });
    t = fmaxf(t - eps, -1.0f - eps);
    int off = 0;
    if (!ONE_WAVE) {
#pragma unroll
      for (int k = 0; k < R; ++k) off += __popcll(__ballot(m[k] > t));
      if (lane == 0) sh.wcount[0][w] = off;
      __syncthreads();
      off = 0;
      for (int i = 0; i < SH::kWaves; ++i) { const int ci = sh.wcount[0][i]; if (i < w) off += ci; n_pass += ci; }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const bool in = m[k] > t;
      const uint64_t mk = __ballot(in);
      if (in) sh.glist[off + __popcll(mk & lt)] = (uint16_t)(g0 + 64 * k);
      off += __popcll(mk);
    }
    if (ONE_WAVE) n_pass = off;
  }
  if (threadIdx.x == 0) { sh.zmax = zmax; sh.bound = t; sh.n_pass = n_pass; }
}

// Scores of the listed groups above thr of segment s, in candidate order: put(i, z, position) for its i-th one.  Segment s
// takes n_pass / kSegs consecutive groups.  Sixteen lanes read the (at most 64) scores of a group with one 16-byte load
// each, so a load takes four groups and the usual row needs one; the lanes' order, and within a lane the four scores',
// is candidate order.  Returns how many there are.
template <typename SH, typename Put>
__device__ __forceinline__ int fetch_candidates(const RowRef& R, const float* zr, int s, int n_pass, float thr, const SH& sh,
                                                Put&& put) {
  const int lane = threadIdx.x & 63;
  const int per = (n_pass + kSegs - 1) / kSegs;
  const int j0 = s * per, j1 = min(j0 + per, n_pass);
  if (j0 >= j1) return 0;                                             // wave-uniform
  const int sub = lane >> 4, in_group = 4 * (lane & 15);
  int cnt = 0;
  // tokens per group and per row are multiples of 4: a lane's four scores are valid together
  const int in_c = min(in_group, R.chunk_tokens - 4), p_end = in_group < R.chunk_tokens ? R.n_cand : 0;
  auto request = [&](int j, int& p, float4& v) {
    const int g = sh.glist[min(j + sub, j1 - 1)];
    p = g * R.chunk_tokens + in_c;
    v = *reinterpret_cast<const float4*>(zr + min(p, R.n_cand - 4));
    if (j + sub >= j1 || p >= p_end) p = -1;
  };
  auto all_four = [&](int p, const float4& v, float t) {
    const bool i0 = v.x > t, i1 = v.y > t, i2 = v.z > t, i3 = v.w > t;
    const uint64_t m0 = __ballot(i0), m1 = __ballot(i1), m2 = __ballot(i2), m3 = __ballot(i3);
    int o = cnt;
    o = __builtin_amdgcn_mbcnt_hi((uint32_t)(m0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m0, o));
    o = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m1, o));
    o = __builtin_amdgcn_mbcnt_hi((uint32_t)(m2 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m2, o));
    o = __builtin_amdgcn_mbcnt_hi((uint32_t)(m3 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m3, o));
    cnt += __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
    if (i0) put(o, v.x, p);
    o += i0;
    if (i1) put(o, v.y, p + 1);
    o += i1;
    if (i2) put(o, v.z, p + 2);
    o += i2;
    if (i3) put(o, v.w, p + 3);
  };
  // The same, with a shorter way where no lane has two: nearly all loads of a peaked row, most of a long flat one.  Its branches wait
  // for the comparisons, so a row of one or two whole batches, where a flat one has many such lanes and nothing to hide the
  // wait behind, goes without.  Solve, us, without / with: supports of 3000 and 5300 of 32768 tokens 28.3 / 29.5 and 39.7 / 41.4, of
  // 262144 tokens with scores as flat 53.8 / 50.2 and 122.1 / 118.7; four wavefronts a row, 64 x 8192 dense calls 246 / 239.
  auto few = [&](int p, const float4& v, float t) {
    const bool i0 = v.x > t, i1 = v.y > t, i2 = v.z > t, i3 = v.w > t;
    const uint64_t m0 = __ballot(i0), m1 = __ballot(i1), m2 = __ballot(i2), m3 = __ballot(i3);
    const uint64_t m01 = m0 | m1, m23 = m2 | m3, m = m01 | m23;
    if (m == 0) return;                                               // wave-uniform, as the next
    if (((m0 & m1) | (m2 & m3) | (m01 & m23)) == 0) {
      if (i0 || i1 || i2 || i3) {
        const int o = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, cnt));
        put(o, i0 ? v.x : i1 ? v.y : i2 ? v.z : v.w, p + (i0 ? 0 : i1 ? 1 : i2 ? 2 : 3));
      }
      cnt += __popcll(m);
      return;
    }
    all_four(p, v, t);
  };
  if (j1 - j0 <= 4) {
    int p; float4 v;
    request(j0, p, v);
    few(p, v, p >= 0 ? thr : INFINITY);
  } else {
    const bool branches = SH::kWaves < 16 || j1 - j0 <= 16 || j1 - j0 > 64;
    for (int j = j0; j < j1; j += 32) {                               // eight loads, 32 groups in flight
      int p[8]; float4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) request(j + 4 * i, p[i], v[i]);     // past j1: its last group again, masked
      if (__builtin_expect(branches, 1)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) few(p[i], v[i], p[i] >= 0 ? thr : INFINITY);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) all_four(p[i], v[i], p[i] >= 0 ? thr : INFINITY);
      }
    }
  }
  return cnt;
}

// The same for a row with at most one group per segment, by one wavefront: four loads take all groups.
template <typename SH>
__device__ __forceinline__ void fetch_single_groups(const RowRef& R, const float* zr, int n_pass, float zmax, float thr, SH& sh) {
  const int lane = threadIdx.x & 63, sub = lane >> 4, in_group = 4 * (lane & 15);
  const uint64_t row = 0xffffull << (lane & 48), before = row & ((1ull << lane) - 1ull);
  int p[kSegs / 4]; float4 v[kSegs / 4];
#pragma unroll
  for (int i = 0; i < kSegs / 4; ++i) {
    const int g = sh.glist[min(4 * i + sub, max(n_pass - 1, 0))];
    p[i] = min(g * R.chunk_tokens + min(in_group, R.chunk_tokens - 4), R.n_cand - 4);
    v[i] = *reinterpret_cast<const float4*>(zr + p[i]);
    if (4 * i + sub >= n_pass || in_group >= R.chunk_tokens || g * R.chunk_tokens + in_group >= R.n_cand) p[i] = -1;
  }
#pragma unroll
  for (int i = 0; i < kSegs / 4; ++i) {
    const float t = p[i] >= 0 ? thr : INFINITY;
    const float z[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
    uint2* seg = sh.seg + (4 * i + sub) * SH::kSegCap;
    int o = 0, n = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t m = __ballot(z[k] > t);
      o += __popcll(m & before);
      n += __popcll(m & row);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (z[k] > t) seg[o++] = make_uint2(__float_as_uint(z[k] - zmax), (uint32_t)(p[i] + k));
    if ((lane & 15) == 0) sh.wcount[1][4 * i + sub] = n;
  }
}

// Threshold, support and weighted value sum of a row whose candidates lie in the segments (sh.wcount[1]: their lengths).
// A wavefront keeps the entries of its kSegs / kWaves segments in registers, an evaluation of the mass costs one barrier,
// and each then gathers the value rows of its own part of the support.  Every sum is taken per segment first, so the
// result does not depend on the number of wavefronts.
template <typename T, bool DENSE, typename SH>
__device__ __forceinline__ void finish_row_block(const SolveArgs& A, const RowRef& R, float lo_u, float zmax, float seed_u, SH& sh) {
#pragma clang fp contract(off)
  constexpr int KR = SH::kSegCap / 64, SPW = kSegs / SH::kWaves;
  const int tid = threadIdx.x, lane = tid & 63, s0 = uniform(tid >> 6) * SPW;
  const uint64_t lt = (1ull << lane) - 1ull;
  const T* v_pool = (const T*)A.v_pool;
  uint2* seg0 = sh.seg + s0 * SH::kSegCap;
  int n[SPW], n_sup[SPW];
  float u[SPW][KR];
#pragma unroll
  for (int i = 0; i < SPW; ++i) {
    n[i] = uniform(sh.wcount[1][s0 + i]);
#pragma unroll
    for (int k = 0; k < KR; ++k)
      u[i][k] = lane + 64 * k < n[i] ? __uint_as_float(seg0[i * SH::kSegCap + lane + 64 * k].x) : -INFINITY;
  }
  const int n_groups = uniform(sh.n_pass);
  int supp = 0, evals = 0, parity = 0;
  const float tau_u = with_beta(A.ibeta, [&](auto ib) {
    constexpr int IB = decltype(ib)::value;
    return solve_tau_core([&](float t, float& F, float& D, int& cnt) {
      auto segment_mass = [&](int i, float& f, float& d, int& c) {
        f = d = 0.f;
        c = 0;
#pragma unroll
        for (int k = 0; k < KR; ++k) {
          if (KR == 1 || 64 * k < n[i]) {                             // wave-uniform
            const float x = fmaxf(u[i][k] - t, 0.f);
            add_mass<IB>(x, A.beta, f, d);
            c += __popcll(__ballot(x > 0.f));
          }
        }
        f = wave_sum(f); d = wave_sum(d);
      };
      float f, d;
      int c;
      if constexpr (SH::kWaves == 1) {
        float fs = 0.f, ds = 0.f;                                     // lane i keeps segment i's sums
        cnt = 0;
#pragma unroll
        for (int b = 0; b < SPW; b += 4) {                            // four segments at a time, as far as there are groups
          if (b < n_groups) {
#pragma unroll
            for (int i = b; i < b + 4; ++i) {
              segment_mass(i, f, d, c);
              fs = (lane & 15) == i ? f : fs; ds = (lane & 15) == i ? d : ds;
              cnt += c;
            }
          }
        }
        F = row16_sum(fs); D = A.beta * row16_sum(ds);
      } else {
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
          segment_mass(i, f, d, c);
          if (lane == 0) { sh.red[parity][s0 + i][0] = f; sh.red[parity][s0 + i][1] = d; sh.red[parity][s0 + i][2] = __int_as_float(c); }
        }
        __syncthreads();
        F = sum_waves(&sh.red[parity][0][0], 3);
        D = A.beta * sum_waves(&sh.red[parity][0][1], 3);
        cnt = sum_waves_i(reinterpret_cast<const int*>(&sh.red[parity][0][2]), 3);
        parity ^= 1;
      }
    }, lo_u, seed_u, IB, supp, evals);
  });
  // the support in place: (weight, position), ascending
#pragma unroll
  for (int i = 0; i < SPW; ++i) {
    uint2* seg = seg0 + i * SH::kSegCap;
    n_sup[i] = 0;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      if (64 * k < n[i]) {
        const float x = u[i][k] - tau_u;
        const bool in = x > 0.f;
        const uint64_t mk = __ballot(in);
        const uint32_t pos = seg[lane + 64 * k].y;
        wave_order();
        if (in) seg[n_sup[i] + __popcll(mk & lt)] = make_uint2(__float_as_uint(pow_beta(x, A.beta, A.ibeta)), pos);
        n_sup[i] += __popcll(mk);
        wave_order();
      }
    }
  }
  if (A.ex.support_tokens != nullptr) {
#pragma unroll
    for (int i = 0; i < SPW; ++i)
      if (lane == 0) sh.wcount[0][s0 + i] = n_sup[i];
    __syncthreads();
    int off = 0;
    for (int i = 0; i < s0; ++i) off += sh.wcount[0][i];
    int32_t* dst = A.ex.support_tokens + (size_t)R.bh * A.ex.support_cap;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      for (int e = lane; e < n_sup[i] && off + e < A.ex.support_cap; e += 64)
        dst[off + e] = token_of<DENSE>(A, R.lrow, (int)seg0[i * SH::kSegCap + e].y);
      off += n_sup[i];
    }
  }
  const int rs = lane >> 4, c = lane & 15;
  if constexpr (SH::kWaves == 1) {
    // value rows of all segments are looked up together (page list -> block table) and take the positions' place; then 4
    // row slots x 16 lanes, four rows of a segment per step and the steps of all segments in one sequence, sixteen loads in
    // flight per lane (float32: eight).  A wait per segment was most of a flat row's time: 2048 rows of 512 tokens with a
    // support of 80, whole call: 62 us, in sequence 54.
    uint32_t row[SPW];
    int ns_of = 0;                                                      // lane i: support entries of segment i
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      row[i] = v_row_of<DENSE>(A, R.b, R.lrow, R.hkv, n_sup[i] > 0 ? (int)seg0[i * SH::kSegCap + min(lane, n_sup[i] - 1)].y : 0);
      ns_of = lane == i ? n_sup[i] : ns_of;
    }
    wave_order();
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      seg0[i * SH::kSegCap + lane].y = row[i];
      if (lane >= n_sup[i]) seg0[i * SH::kSegCap + lane].x = 0u;        // past the end: its last row with weight 0
    }
    wave_order();
    const uint32_t full = (uint32_t)__ballot(ns_of > 0);                // segments with an entry; the others' output is 0
    for (uint32_t none = ~full & 0xffffu; none != 0; none &= none - 1) {
      const int i = __builtin_ctz(none);
      sh.obuf[i][lane] = 0.f; sh.obuf[i][lane + 64] = 0.f;
    }
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.f;
    uint32_t left = full;
    int at = 0;
    constexpr int U = sizeof(T) == 2 ? 16 : 8;
    while (left != 0) {                                                 // wave-uniform, as everything about the steps
      Raw8<T> vr[U]; float pw[U];
      int ends[U];                                                      // the segment that ends with the step, or -1
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int i = left != 0 ? __builtin_ctz(left) : 0;
        const bool real = left != 0;
        const uint2 e = seg0[i * SH::kSegCap + min(at + rs, SH::kSegCap - 1)];
        pw[j] = real ? __uint_as_float(e.x) : 0.f;
        load_raw8(v_pool + (size_t)(real ? e.y : row[0]) * kD + 8 * c, vr[j]);
        at += 4;
        ends[j] = -1;
        if (real && at >= __builtin_amdgcn_readlane(ns_of, i)) { ends[j] = i; left &= left - 1; at = 0; }
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        float vv[8];
        widen8(vr[j], vv);
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = fmaf(pw[j], vv[q], acc[q]);
        if (ends[j] >= 0) {
          wave_order();                                                 // the partial output takes the segment's place
          store_partial(acc, sh, ends[j]);
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[q] = 0.f;
        }
      }
    }
  } else {
    // value rows: 64 looked up at a time (page list -> block table), then 4 row slots x 16 lanes, eight 16-byte loads in
    // flight per lane; the next 64 are looked up before these are consumed
#pragma unroll 1
    for (int i = 0; i < SPW; ++i) {
      const uint2* seg = seg0 + i * SH::kSegCap;
      int ns = n_sup[0];
#pragma unroll
      for (int j = 1; j < SPW; ++j) ns = i == j ? n_sup[j] : ns;
      float acc[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] = 0.f;
      uint32_t row = ns > 0 ? v_row_of<DENSE>(A, R.b, R.lrow, R.hkv, (int)seg[min(lane, ns - 1)].y) : 0u;
      for (int e0 = 0; e0 < ns; e0 += 64) {
        const uint32_t row_now = row;
        row = v_row_of<DENSE>(A, R.b, R.lrow, R.hkv, (int)seg[min(e0 + 64 + lane, ns - 1)].y);
        const float p_now = e0 + lane < ns ? __uint_as_float(seg[e0 + lane].x) : 0.f;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          Raw8<T> vr[8]; float pw[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int src = 32 * half + 4 * j + rs;
            pw[j] = __shfl(p_now, src);
            load_raw8(v_pool + (size_t)(uint32_t)__shfl((int)row_now, src) * kD + 8 * c, vr[j]);
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            float vv[8];
            widen8(vr[j], vv);
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(pw[j], vv[q], acc[q]);
          }
          if (e0 + 32 >= ns) break;                                     // wave-uniform
        }
      }
      store_partial(acc, sh, s0 + i);
    }
  }
  sum_partials(sh, A.out + (size_t)R.bh * kD);
  if (tid == 0) {
    A.tau_out[R.bh] = tau_u + zmax; A.supp_out[R.bh] = supp;
    if (A.ex.solve_evals != nullptr) A.ex.solve_evals[R.bh] = evals;
  }
}

// Side outputs over ALL candidates of a row (mass and count above a given threshold, log-sum-exp of the whole cache).
template <bool DENSE, typename SH>
__device__ __forceinline__ void side_outputs(const SolveArgs& A, int bh, int n_cand, const float* zr, float zmax, SH& sh) {
  const int tid = threadIdx.x;
  if (A.ex.tau_ref != nullptr && (A.ex.kept_mass_ref != nullptr || A.ex.kept_supp_ref != nullptr)) {
    const float tr = A.ex.tau_ref[bh];
    constexpr int V = SH::kWaves == 1 ? 4 : 1;         // one wavefront adds up in the order of four
    float f = 0.f; int c = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      float part = 0.f;
      for (int i = tid + 64 * v; i < n_cand; i += 64 * SH::kWaves * V) {
        const float x = zr[i] - tr;
        if (x > 0.f) { part += pow_beta(x, A.beta, A.ibeta); ++c; }
      }
      f += V == 1 ? block_sum(part, sh.red1) : wave_sum(part);
    }
    c = block_sum_i(c, sh.wcount[0]);
    if (tid == 0) {
      if (A.ex.kept_mass_ref != nullptr) A.ex.kept_mass_ref[bh] = f;
      if (A.ex.kept_supp_ref != nullptr) A.ex.kept_supp_ref[bh] = c;
    }
  }
  if (DENSE && A.ex.lse != nullptr) {
    // log sum_j exp(s_j) with s_j = z_j / a, shifted by the maximum
    const float inv_a = 1.0f / A.a;
    float f = 0.f;
    for (int i = tid; i < n_cand; i += 64 * SH::kWaves) f += __expf((zr[i] - zmax) * inv_a);
    f = block_sum(f, sh.red1);
    if (tid == 0) A.ex.lse[bh] = zmax * inv_a + __logf(f);
  }
}

// A row from the bound of its groups (sh.zmax, sh.bound, sh.n_pass, sh.glist, visible to all) to the outputs.  Returns
// false, with nothing written, when a segment is too small for its candidates.
template <typename T, bool DENSE, typename SH>
__device__ __forceinline__ bool solve_bounded_row(const SolveArgs& A, const RowRef& R, const float* zr, float seed_z,
                                                  bool block_extras, SH& sh) {
#pragma clang fp contract(off)
  constexpr int SPW = kSegs / SH::kWaves;
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
  const float zmax = sh.zmax;
  float bound = sh.bound;
  if (!(zmax > -INFINITY)) {                                          // no valid candidate at all
    if (w == 0) empty_row_wave<DENSE>(A, R.bh);
    return true;
  }
  const int n_pass = uniform(sh.n_pass);
  int cw;
  for (int attempt = 0;; ++attempt) {
    if constexpr (SH::kMaxGroups <= kSegs) {
      fetch_single_groups(R, zr, n_pass, zmax, zmax + bound, sh);
    } else {
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
        uint2* seg = sh.seg + (w * SPW + i) * SH::kSegCap;
        const int n = fetch_candidates(R, zr, w * SPW + i, n_pass, zmax + bound, sh, [&](int o, float z, int p) {
          if (!SH::kOverflows || o < SH::kSegCap) seg[o] = make_uint2(__float_as_uint(z - zmax), (uint32_t)p);
        });
        if (lane == 0) sh.wcount[1][w * SPW + i] = n;
      }
    }
    __syncthreads();
    cw = lane < kSegs ? sh.wcount[1][lane] : 0;
    if constexpr (!SH::kOverflows) break;
    if (__builtin_expect(__ballot(cw > SH::kSegCap) == 0, 1)) break;
    // a row that a tighter bound leaves far too many candidates will not fit after the next one either
    if (attempt == 3 || (attempt > 0 && __ballot(cw > SH::kSegCap + SH::kSegCap / 2) != 0)) return false;
    // A segment is too small.  What the segments do hold is a subset of the candidates, so its mass bounds tau from below
    // like the maxima's, and far tighter on a row this flat: the groups are read again against that bound, which a
    // support that fits the segments reaches after one or two rounds.
    if constexpr (SH::kOverflows) {
      constexpr int KR = SH::kSegCap / 64;
      float u[SPW * KR];
#pragma unroll
      for (int i = 0; i < SPW; ++i) {
        const int kept = min(uniform(sh.wcount[1][w * SPW + i]), SH::kSegCap);
#pragma unroll
        for (int k = 0; k < KR; ++k)
          u[i * KR + k] = lane + 64 * k < kept ? __uint_as_float(sh.seg[(w * SPW + i) * SH::kSegCap + lane + 64 * k].x) : -INFINITY;
      }
      int parity = 0;
      const float t = group_bound(u, bound, A.beta, A.ibeta, [&](float& f, float& d) {
        f = wave_sum(f); d = wave_sum(d);
        if (lane == 0) { sh.red[parity][w][0] = f; sh.red[parity][w][1] = d; }
        __syncthreads();
        f = sum_waves<SH::kWaves>(&sh.red[parity][0][0], 3); d = sum_waves<SH::kWaves>(&sh.red[parity][0][1], 3);
        parity ^= 1;
      });
      const float tighter = t - 4e-6f * fmaxf(1.f, fabsf(zmax));
      if (!(tighter > bound)) return false;                           // the same for all threads
      bound = tighter;
      if (threadIdx.x == 0) sh.bound = bound;
      __syncthreads();                                                // the segments are read
    }
  }
  const int total = sum_waves_i(sh.wcount[1], 1);
  const float lo_u = fminf(bound, -1e-7f), seed_u = seed_z - zmax;
  if (__builtin_expect(block_extras, 0)) side_outputs<DENSE>(A, R.bh, R.n_cand, zr, zmax, sh);
  if (__builtin_expect(total <= kWaveList, 1)) {
    if (w == 0) {
      const int ends = wave_incl_scan_i(cw);                          // where the segments end
      if (total <= 64) finish_row_wave<T, DENSE, 1>(A, R, total, ends, lo_u, zmax, seed_u, sh);
      else finish_row_wave<T, DENSE, kWaveList / 64>(A, R, total, ends, lo_u, zmax, seed_u, sh);
    }
  } else {
    finish_row_block<T, DENSE>(A, R, lo_u, zmax, seed_u, sh);
  }
  return true;
}

// A row of at most SH::kMaxGroups groups, from the group maxima to the outputs.  False: its candidates outgrow the
// segments (attention so flat that one of the sixteen gets more than 192 or 768).
template <typename T, bool DENSE, typename SH>
__device__ __forceinline__ bool solve_row(const SolveArgs& A, const RowRef& R, const float* zr, const float* pm, float seed_z,
                                          bool block_extras, SH& sh) {
  const int w = uniform(threadIdx.x >> 6);
  auto group_max = [pm](int g) { return pm[g]; };
  if (R.n_chunks <= kWaveGroups) {
    if (w == 0) {
      if (SH::kMaxGroups <= 128 || R.n_chunks <= 128) bound_groups<2, true>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
      else if (R.n_chunks <= kWaveGroups / 2) bound_groups<kWaveGroups / 128, true>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
      else bound_groups<kWaveGroups / 64, true>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
    }
  } else if constexpr (SH::kMaxGroups > kWaveGroups) {
    constexpr int kThreads = 64 * SH::kWaves;
    if (R.n_chunks <= 4 * kThreads)
      bound_groups<4, false>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
    else
      bound_groups<SH::kMaxGroups / kThreads, false>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
  }
  __syncthreads();
  return solve_bounded_row<T, DENSE>(A, R, zr, seed_z, block_extras, sh);
}

__device__ __forceinline__ RowRef whole_row(const SolveArgs& A, int bh) {
  const int b = bh / A.Hq, hq = bh % A.Hq, hkv = hq / (A.Hq / A.Hkv), gp = pmax_pages(A.P);
  const int n_slots = clampi((A.seq_lens[b] + A.P - 1) / A.P, 0, A.Mmax);
  return {b, bh, bh, hkv, n_slots * A.P, gp * A.P, (n_slots + gp - 1) / gp};
}
// Side outputs that need a pass over all candidates.
template <bool DENSE>
__device__ __forceinline__ bool wants_side_outputs(const SolveArgs& A) {
  return (A.ex.tau_ref != nullptr && (A.ex.kept_mass_ref != nullptr || A.ex.kept_supp_ref != nullptr)) ||
         (DENSE && A.ex.lse != nullptr);
}

// Row of workgroup i: the heads of a group, which read many of the same pages and value rows, go to one XCD (workgroups go to
// the XCDs in turn) as far as whole rounds of groups last.  A permutation of [0, rows).  2048 rows of 256 tokens, support 246,
// groups of four: 37.5 -> 30.2 us; 4096 rows of 1024, support 720, groups of eight: 172 -> 136.
__device__ __forceinline__ int group_on_one_xcd(int i, int rows, int heads) {
  if (heads == 1) return i;
  const int round = kXcds * heads, t = i / kXcds;
  return i >= rows / round * round ? i : (t / heads * kXcds + i % kXcds) * heads + t % heads;
}

template <typename T>
__global__ __launch_bounds__(64) void decode_solve_one_kernel(const SolveArgs A) {
  __shared__ SolveSharedOne sh;
  const int heads = A.Hq / A.Hkv, gp = pmax_pages(A.P);
  const int bh = group_on_one_xcd(blockIdx.x, gridDim.x, heads), b = bh / A.Hq, hkv = (bh - b * A.Hq) / heads;
  const int lrow = A.grouped ? b * A.Hkv + hkv : bh;
  const int n_slots = clampi(A.n_sel[lrow], 0, A.cap);
  const float seed_z = A.ex.tau_seed != nullptr ? A.ex.tau_seed[bh] : NAN;
  const RowRef R{b, bh, lrow, hkv, n_slots * A.P, gp * A.P, (n_slots + gp - 1) / gp};
  solve_row<T, false>(A, R, A.zbuf + (size_t)bh * A.zstride, A.pmax + (size_t)bh * A.n_chunks_max, seed_z,
                      wants_side_outputs<false>(A), sh);
}

// Its 160 KB of code are fetched anew by few compute units in every call, behind a stream that has emptied the caches, so that
// where they lie shows: the same instructions at other addresses took 1 x 32K tokens from 22.4 to 22.7 us (across a boundary
// of 2 MB) and its Gaussian step from 42.9 to 43.5.  From the start of a page on: 22.4 and 42.6.
template <typename T, bool DENSE, typename SH>
__global__ __launch_bounds__(64 * SH::kWaves) __attribute__((aligned(4096))) void decode_solve_kernel(const SolveArgs A) {
  __shared__ SH sh;
  constexpr int NT = 64 * SH::kWaves, NW = SH::kWaves, LIST = SH::kListCap;
  constexpr int kRoundTokens = NT * kRoundLoads;
  constexpr bool kLong = SH::kMaxGroups >= kPreGroups;   // false: the launch has only rows of at most kMaxGroups groups
  const int bh = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6);
  const uint64_t lt = (1ull << lane) - 1ull;
  const T* v_pool = (const T*)A.v_pool;
  // The compiler's order of the scalar loads in here is a few tenths of a microsecond of every solve: written out they overlap
  // for a list (refined float32 step 125.5 us, 126.3 behind a function), behind a function for a whole sequence (dense 32K
  // 22.0 us, 22.6 written out).
  RowRef R;
  if constexpr (DENSE) {
    R = whole_row(A, bh);
  } else {
    const int Hq = A.Hq, Hkv = A.Hkv, P = A.P;
    const int hq = bh % Hq;
    R.b = bh / Hq; R.bh = bh; R.hkv = hq / (Hq / Hkv);
    R.lrow = A.grouped ? R.b * Hkv + R.hkv : bh;            // row of the page list this head reads
    const int n_slots = clampi(A.n_sel[R.lrow], 0, A.cap);
    R.n_cand = n_slots * P;
    R.n_chunks = (n_slots + pmax_pages(P) - 1) / pmax_pages(P);
    R.chunk_tokens = pmax_pages(P) * P;
  }
  const int b = R.b, lrow = R.lrow, hkv = R.hkv, n_cand = R.n_cand, n_chunks = R.n_chunks, chunk_tokens = R.chunk_tokens;
  const float* zr = A.zbuf + (size_t)bh * A.zstride;
  const float* pm = A.pmax + (size_t)bh * A.n_chunks_max;
  const float beta = A.beta; const int ibeta = A.ibeta;
  float* out = A.out + (size_t)bh * kD;

  // warm start (optional): requested with the first loads, used once zmax is known
  const float seed_z = A.ex.tau_seed != nullptr ? A.ex.tau_seed[bh] : NAN;
  const bool block_extras = wants_side_outputs<DENSE>(A);
  float zmax, thr_f = 0.f;
  const bool pre = !kLong || n_chunks <= kPreGroups;
  if (__builtin_expect(pre, 1)) {
    if (__builtin_expect(solve_row<T, DENSE>(A, R, zr, pm, seed_z, block_extras, sh), 1)) return;
  }
  // Longer rows, and those whose candidates outgrow LDS.
  // The filter passes are launched when the list CAPACITY allows longer rows than kPreGroups; whether this row took
  // them is decided here, from its actual length (they leave shorter rows alone).
  const bool filt = kLong && A.fcount != nullptr && !pre;
  if (filt) {
    zmax = n_cand > 0 ? A.frow[2 * bh] : -INFINITY;
    thr_f = n_cand > 0 ? A.frow[2 * bh + 1] : 0.f;
  } else if (pre) {
    zmax = sh.zmax; thr_f = sh.zmax + sh.bound;
  } else {
    float mx = -INFINITY;
    for (int i = tid; i < n_chunks; i += NT) mx = fmaxf(mx, pm[i]);
    zmax = block_max(mx, sh.red1);
  }
  if (!(zmax > -INFINITY)) {                // no valid candidate at all
    if (tid < kD) out[tid] = 0.f;
    if (tid == 0) {
      A.tau_out[bh] = INFINITY; A.supp_out[bh] = 0;
      if (A.ex.solve_evals != nullptr) A.ex.solve_evals[bh] = 0;
      if (A.ex.tau_ref != nullptr && A.ex.kept_mass_ref != nullptr) A.ex.kept_mass_ref[bh] = 0.f;
      if (A.ex.tau_ref != nullptr && A.ex.kept_supp_ref != nullptr) A.ex.kept_supp_ref[bh] = 0;
      if (DENSE && A.ex.lse != nullptr) A.ex.lse[bh] = -INFINITY;
    }
    return;
  }
  // The candidates above the bound (only z > zmax - 1 can be in the support; `pre` and filtered rows have a tighter
  // one) are compacted IN ORDER.  Rows that have neither list of groups nor filter results sweep their scores in rounds
  // (wavefront w of a round owns consecutive positions, so (round, w, load, lane) order is candidate order), skipping
  // chunks whose maximum is <= thr, and histogram the candidates over 64 slices of [thr, zmax]: counts alone give a lower
  // bound of the mass at every slice boundary (an entry of slice j lies at least j-i slices above boundary i), hence a
  // tighter threshold for the solve or, if the candidates did not fit in LDS, for one more compaction pass.
  float thr = filt || pre ? thr_f : zmax - 1.0f - 4e-6f * fmaxf(1.f, fabsf(zmax));
  const float seed_u = seed_z - zmax;
  int evals = 0;
  float lo_u = thr - zmax;
  // chunk skipping pays only when there is a lot to skip (dense rows); short candidate lists are read whole,
  // which saves the dependent load of the chunk maxima in every round
  const bool can_skip = (chunk_tokens & 63) == 0 && n_cand > 4 * kRoundTokens;
  int n_list = 0, parity = 0;
  bool in_lds = true;
  bool in_spill = false;          // the candidate list outgrew LDS and lives in this row's overflow list
  bool prefilled = false;
  float* const su = A.spill_u != nullptr ? A.spill_u + (size_t)bh * A.spill_cap : nullptr;
  int32_t* const sp = A.spill_pos != nullptr ? A.spill_pos + (size_t)bh * A.spill_cap : nullptr;
  if constexpr (kLong) if (filt) {
    // survivors of the filter passes: gather the per-slice lists, in slice order, if they fit
    const int n_slices = (n_chunks + kFilterSliceChunks - 1) / kFilterSliceChunks;
    const int cs = tid < n_slices ? A.fcount[(size_t)bh * A.n_slices_max + tid] : 0;
    int inc = cs;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int t = __shfl_up(inc, d); if (lane >= d) inc += t; }
    if (lane == 63) sh.wcount[0][w] = inc;
    const int bad = __syncthreads_or(cs > kFilterSliceCap);
    int base = 0, tot = 0;
    for (int i = 0; i < NW; ++i) { const int ci = sh.wcount[0][i]; if (i < w) base += ci; tot += ci; }
    if (!bad && tot <= LIST) {
      int* start = reinterpret_cast<int*>(sh.list_row);      // free until the solve is done
      if (tid < n_slices) { start[2 * tid] = base + inc - cs; start[2 * tid + 1] = cs; }
      __syncthreads();
      for (int sl = w; sl < n_slices; sl += NW) {
        const int o0 = start[2 * sl], cnt = start[2 * sl + 1];
        const float* lu = A.flist_u + ((size_t)bh * A.n_slices_max + sl) * kFilterSliceCap;
        const int32_t* lp = A.flist_pos + ((size_t)bh * A.n_slices_max + sl) * kFilterSliceCap;
        for (int e = lane; e < cnt; e += 64) { sh.list_u[o0 + e] = lu[e]; sh.list_pos[o0 + e] = lp[e]; }
      }
      n_list = tot;
      prefilled = true;
      lo_u = fminf(thr - zmax, -1e-7f);
    } else if (!bad && su != nullptr && tot <= A.spill_cap) {
      // too many survivors for LDS: concatenate the per-slice lists, in slice order, into the row's overflow list
      int* start = reinterpret_cast<int*>(sh.list_row);
      if (tid < n_slices) { start[2 * tid] = base + inc - cs; start[2 * tid + 1] = cs; }
      __syncthreads();
      for (int sl = w; sl < n_slices; sl += NW) {
        const int o0 = start[2 * sl], cnt = start[2 * sl + 1];
        const float* lu = A.flist_u + ((size_t)bh * A.n_slices_max + sl) * kFilterSliceCap;
        const int32_t* lp = A.flist_pos + ((size_t)bh * A.n_slices_max + sl) * kFilterSliceCap;
        for (int e = lane; e < cnt; e += 64) { su[o0 + e] = lu[e]; sp[o0 + e] = lp[e]; }
      }
      n_list = tot;
      prefilled = true;
      in_lds = false; in_spill = true;
      lo_u = fminf(thr - zmax, -1e-7f);
    }
    __syncthreads();
  }
  if (pre) {
    // The row outgrew its segments.  Their lengths are known (sh.wcount[1], from the last fetch against this bound), so every
    // wavefront fetches its segments once more to their places in one list: in LDS if it fits, else in the row's overflow
    // list.  (In rounds of 16 groups per wavefront with an exchange of the counts each, a million-token row with a support of
    // 35 000 took 1220 us a call.)
    constexpr int SPW = kSegs / NW;
    const int n_pass = uniform(sh.n_pass);
    int inc = lane < kSegs ? sh.wcount[1][lane] : 0;
#pragma unroll
    for (int d = 1; d < kSegs; d <<= 1) { const int t = __shfl_up(inc, d); if (lane >= d) inc += t; }
    n_list = __builtin_amdgcn_readlane(inc, kSegs - 1);
    in_lds = n_list <= LIST;
    in_spill = !in_lds && su != nullptr && n_list <= A.spill_cap;
    auto fill = [&](float* du, int32_t* dp) {
#pragma unroll 1
      for (int i = 0; i < SPW; ++i) {
        const int s = w * SPW + i, off = s > 0 ? __shfl(inc, s - 1) : 0;
        fetch_candidates(R, zr, s, n_pass, thr, sh, [&](int o, float z, int p) { du[off + o] = z - zmax; dp[off + o] = p; });
      }
    };
    if (in_lds) fill(sh.list_u, sh.list_pos);
    else if (in_spill) fill(su, sp);
    if (in_lds || in_spill) lo_u = fminf(thr - zmax, -1e-7f);
  }
  if constexpr (kLong) for (int pass = 0; pass < 3 && !prefilled && !pre; ++pass) {
    const float width = zmax - thr, slice = width * (1.0f / 64.0f), inv_slice = 64.0f / width;
    if (tid < 64) sh.hist[tid] = 0;
    n_list = 0; in_lds = true;
    __syncthreads();
    for (int round0 = 0; round0 < n_cand; round0 += kRoundTokens) {
      const int seg = round0 + w * 64 * kRoundLoads;
      // The chunk maxima of the round are fetched first as one batch (clamped, unconditional), then the
      // score loads of the chunks that can hold a candidate are issued back to back; nothing is consumed
      // before all of them are in flight.
      float pmv[kRoundLoads];
#pragma unroll
      for (int i = 0; i < kRoundLoads; ++i) pmv[i] = can_skip ? pm[min(seg + i * 64, n_cand - 1) / chunk_tokens] : INFINITY;
      float v[kRoundLoads];
#pragma unroll
      for (int i = 0; i < kRoundLoads; ++i) {
        const int pos0 = seg + i * 64;
        const float pmu = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(pmv[i])));
        v[i] = -INFINITY;
        if (pos0 < n_cand && (!can_skip || pmu > thr)) v[i] = zr[min(pos0 + lane, n_cand - 1)];
      }
#pragma unroll
      for (int i = 0; i < kRoundLoads; ++i) v[i] = seg + i * 64 + lane < n_cand ? v[i] : -INFINITY;
      int c = 0;
#pragma unroll
      for (int i = 0; i < kRoundLoads; ++i) {
        const bool in = v[i] > thr;
        c += __popcll(__ballot(in));
        if (in) atomicAdd(&sh.hist[min(63, (int)((v[i] - thr) * inv_slice))], 1);
      }
      if (lane == 0) sh.wcount[parity][w] = c;
      __syncthreads();
      int off = n_list, tot = 0;
      for (int i = 0; i < NW; ++i) { const int ci = sh.wcount[parity][i]; if (i < w) off += ci; tot += ci; }
      n_list += tot;
      parity ^= 1;
      if (n_list > LIST) in_lds = false;
      if (in_lds) {
#pragma unroll
        for (int i = 0; i < kRoundLoads; ++i) {
          const bool in = v[i] > thr;
          const uint64_t mk = __ballot(in);
          if (in) {
            const int o = off + __popcll(mk & lt);
            sh.list_u[o] = v[i] - zmax;
            sh.list_pos[o] = seg + i * 64 + lane;
          }
          off += __popcll(mk);
        }
      }
    }
    __syncthreads();
    // highest slice boundary whose counted lower bound of the mass is still >= 1
    const int level = certified_level<64>(sh.hist, slice, beta, ibeta, sh.flags);
    const float thr2 = thr + (float)level * slice;
    if (in_lds) { lo_u = fminf(thr2 - zmax, -1e-7f); break; }
    if (level == 0) break;                       // no tighter threshold from counts: stream the row
    thr = thr2;
    lo_u = thr - zmax;
  }
  __syncthreads();

  float tau_u; int supp;
  if (in_lds) {
    // V row of every candidate, fetched now (two dependent loads) and consumed after the solve
    uint32_t rowreg[LIST / NT];
#pragma unroll
    for (int k = 0; k < LIST / NT; ++k) {
      const int e = min(tid + k * NT, n_list - 1);      // clamped: loads stay unconditional
      rowreg[k] = v_row_of<DENSE>(A, b, lrow, hkv, sh.list_pos[e]);
    }
    const ListSrc ls{sh.list_u, sh.list_pos, n_list};
    if (n_list <= kWaveList) tau_u = solve_tau_wave(sh.list_u, n_list, lo_u, seed_u, beta, ibeta, sh, supp, evals);
    else tau_u = solve_tau(ls, lo_u, seed_u, beta, ibeta, sh, supp, evals);
#pragma unroll
    for (int k = 0; k < LIST / NT; ++k) {
      const int e = tid + k * NT;
      if (e < n_list) sh.list_row[e] = rowreg[k];
    }
    __syncthreads();
    // in-place ordered compaction of the support: entry e keeps (p_e, pos_e, row_e)
    int n_sup = 0;
    for (int e0 = 0; e0 < n_list; e0 += NT) {
      const int e = e0 + tid;
      const float x = e < n_list ? sh.list_u[e] - tau_u : -1.f;
      const int pe = e < n_list ? sh.list_pos[e] : 0;
      const uint32_t re = e < n_list ? sh.list_row[e] : 0u;
      const bool in = x > 0.f;
      const uint64_t mk = __ballot(in);
      if (lane == 0) sh.wcount[parity][w] = __popcll(mk);
      __syncthreads();                                     // all reads of this block are done
      int off = n_sup, tot = 0;
      for (int i = 0; i < NW; ++i) { const int ci = sh.wcount[parity][i]; if (i < w) off += ci; tot += ci; }
      parity ^= 1;
      if (in) {
        const int o = off + __popcll(mk & lt);
        sh.list_u[o] = pow_beta(x, beta, ibeta);
        sh.list_pos[o] = pe;
        sh.list_row[o] = re;
      }
      n_sup += tot;
    }
    __syncthreads();
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    gather_support<T>(v_pool, sh, n_sup, acc);
    __syncthreads();
    store_partial(acc, sh, w);
    sum_partials<NW>(sh, out);
    if (A.ex.support_tokens != nullptr) {
      int32_t* dst = A.ex.support_tokens + (size_t)bh * A.ex.support_cap;
      for (int e = tid; e < n_sup && e < A.ex.support_cap; e += NT)
        dst[e] = token_of<DENSE>(A, lrow, sh.list_pos[e]);
    }
  } else {
    // The candidates do not fit in LDS.  They are iterated where they are: in the row's overflow list (every
    // evaluation of the mass reads that list), or -- a row so flat that even that list is too small -- in the score
    // row itself.  The support is then gathered in rounds of 4096 candidates (wavefront w owns 256 consecutive ones):
    // the support tokens of a round are compacted into LDS (weight, V row, position) -- at most 4096, so they always
    // fit -- and their V rows summed by the 64 row slots with batched independent loads.
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    int n_out = 0;
    auto finish = [&](const auto& src) {
      tau_u = solve_tau(src, lo_u, seed_u, beta, ibeta, sh, supp, evals);
      for (int base = 0; base < src.n; base += 4 * NT) {
        float xs[4]; int ps[4]; uint32_t rw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int idx = min(base + w * 256 + i * 64 + lane, src.n - 1);
          xs[i] = src.get_u(idx); ps[i] = src.get_pos(idx);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) rw[i] = v_row_of<DENSE>(A, b, lrow, hkv, min(ps[i], n_cand - 1));   // unconditional
        int cw = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          xs[i] = base + w * 256 + i * 64 + lane < src.n ? xs[i] - tau_u : -1.f;
          cw += __popcll(__ballot(xs[i] > 0.f));
        }
        if (lane == 0) sh.wcount[parity][w] = cw;
        __syncthreads();                                   // also: the previous round's gather is done
        int off = 0, tot = 0;
        for (int i = 0; i < NW; ++i) { const int ci = sh.wcount[parity][i]; if (i < w) off += ci; tot += ci; }
        parity ^= 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool in = xs[i] > 0.f;
          const uint64_t mk = __ballot(in);
          if (in) {
            const int o = off + __popcll(mk & lt);
            sh.list_u[o] = pow_beta(xs[i], beta, ibeta);
            sh.list_row[o] = rw[i];
            sh.list_pos[o] = ps[i];
          }
          off += __popcll(mk);
        }
        __syncthreads();
        gather_support<T>(v_pool, sh, tot, acc);
        if (A.ex.support_tokens != nullptr) {
          int32_t* dst = A.ex.support_tokens + (size_t)bh * A.ex.support_cap;
          for (int e = tid; e < tot && n_out + e < A.ex.support_cap; e += NT)
            dst[n_out + e] = token_of<DENSE>(A, lrow, sh.list_pos[e]);
        }
        n_out += tot;
      }
    };
    if (in_spill) {
      __syncthreads();                                     // the overflow list is complete and visible to the workgroup
      finish(ListSrc{su, sp, n_list});
    } else {
      finish(RowSrc{zr, n_cand, zmax});
    }
    __syncthreads();
    store_partial(acc, sh, w);
    sum_partials<NW>(sh, out);
  }
  const float tau = tau_u + zmax;
  if (tid == 0) {
    A.tau_out[bh] = tau; A.supp_out[bh] = supp;
    if (A.ex.solve_evals != nullptr) A.ex.solve_evals[bh] = evals;
  }

  if (block_extras) side_outputs<DENSE>(A, bh, n_cand, zr, zmax, sh);
}

// ------------------------------------------------------------------------------------------
// both passes in one launch: short per-head page lists
// ------------------------------------------------------------------------------------------
// A short list is decoded by ONE workgroup: it gathers the K pages, keeps the scores and their maxima in LDS and goes on
// to the threshold and the values there.  Two launches over such lists are hardly more than two launch latencies with a
// round trip of the scores through memory between them (4096-token float32 step: 7.6 + 12 us; 64 sequences of 8192
// tokens, 2048 lists of 11 pages: 26.5 + 14.2 us), and a workgroup that waits for its own rows overlaps the others of its
// compute unit, which launches cannot.  Against it stands the rate at which one compute unit reads K, about 75 GB/s:
// see rows_in_one_launch.  Scores are those of pass 1 bit for bit (the same products in the same order), and so are the
// results.
constexpr int kRowTokens = 4096;                   // longest list of the sixteen-wavefront workgroup
constexpr int kRowTokensMany = 2048;               // and of the four-wavefront one

// GROUP: the least number of tokens in a group, 64 where the page size divides 64, else at least 36 (one page of 36).
template <int NW, int TOKENS, int GROUP>
struct RowShared {
  static constexpr int kWaves = NW, kGroups = (TOKENS + GROUP - 1) / GROUP, kMaxGroups = kGroups;
  static constexpr bool kOverflows = false;
  static constexpr int kSegCap = (kGroups + kSegs - 1) / kSegs * 64;   // a segment holds all tokens of its groups
  union {                                          // the scores are dead once the candidates are listed
    alignas(16) float z[TOKENS];                   // read four at a time
    float obuf[kSegs][kD];
    struct { float list_u[kWaveList]; int32_t list_pos[kWaveList]; uint32_t list_row[kWaveList]; };
  };
  union {                                          // and the maxima before that
    uint2 seg[kSegs * kSegCap];
    float umax[TOKENS / 4];                        // per score unit: 16-token chunk, or page where PT is 0
  };
  float red[2][kSegs][3];
  int wcount[2][kSegs];
  int pre[kSegs + 1];
  float red1[NW];
  uint16_t glist[kGroups];
  float zmax, bound;
  int n_pass;
};

// PT: page size of a bf16 cache (16, 32, 64), 0: float32 (FMAs), or bf16 pages of any other size.
template <typename T, int PT, int NW, int TOKENS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 4 && PT ? (TOKENS > 1024 ? 5 : 6) : 4)))
void decode_row_kernel(const ScoreArgs S, const SolveArgs A) {
  __shared__ RowShared<NW, TOKENS, PT ? 64 : 36> sh;
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6);
  const int heads = S.Hq / S.Hkv;
  const int bh = group_on_one_xcd(blockIdx.x, gridDim.x, heads), b = bh / S.Hq, hkv = (bh - b * S.Hq) / heads;
  const int P = PT ? PT : S.P;
  const int n = uniform_load(S.seq_lens + b);
  const int n_slots = clampi(uniform_load(S.n_sel + bh), 0, S.cap);
  const float seed_z = A.ex.tau_seed != nullptr ? A.ex.tau_seed[bh] : NAN;
  const int gp = pmax_pages(P);
  constexpr int UPP = PT ? PT / 16 : 1;                   // score units per page
  const int n_units = n_slots * UPP;
  // lane l: the page of this wavefront's unit l (units w, w + NW, ...); 64 of them per batch
  for (int u0 = w; u0 < n_units; u0 += 64 * NW) {
    const int my_unit = min(u0 + NW * lane, n_units - 1);
    const int l_lp = clampi(S.page_idx[(size_t)bh * S.cap + my_unit / UPP], 0, S.Mmax - 1);
    const int l_phys = clampi(S.block_table[(size_t)b * S.Mmax + l_lp], 0, S.n_phys - 1);
    const int mine = min((n_units - u0 + NW - 1) / NW, 64);
    if constexpr (PT != 0) {
      const int m = lane & 15, j = lane >> 4, kq = m & 3, gl = m >> 2;      // as in decode_scores_mfma_kernel, G = 1
      const bf16_t* k_pool = (const bf16_t*)S.k_pool + gl * kD + (kq * 4 + j) * 8;
      const uint4 bq = *reinterpret_cast<const uint4*>((const bf16_t*)S.q + (size_t)bh * kD + kq * 32 + j * 8);
      auto request = [&](int i, uint4 (&a)[4]) {                            // past the end: the last unit again
        const int ic = min(i, mine - 1), t = (u0 + NW * ic) % UPP;
        const bf16_t* kc = k_pool + (((size_t)__builtin_amdgcn_readlane(l_phys, ic) * S.HkvPool + hkv) * PT + 16 * t) * kD;
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = *reinterpret_cast<const uint4*>(kc + s * 4 * kD);
      };
      auto consume = [&](int i, const uint4 (&a)[4]) {
        if (i >= mine) return;                                              // wave-uniform
        const int unit = u0 + NW * i, t = unit % UPP;
        const int tok0 = __builtin_amdgcn_readlane(l_lp, i) * PT + 16 * t + j;
        float zkeep = 0.f, mx = -INFINITY;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
          const f32x4_t c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[s]),
                                                                    __builtin_bit_cast(bf16x8_t, bq), zero, 0, 0, 0);
          const float v01 = (kq & 1) ? c[1] : c[0], v23 = (kq & 1) ? c[3] : c[2];
          float v = (kq & 2) ? v23 : v01;
          v += dpp_move<0xB1>(v);
          v += dpp_move<0x4E>(v);
          const float z = tok0 + 4 * s < n ? S.zscale * v : -INFINITY;
          if (s == kq) zkeep = z;
          mx = fmaxf(mx, z);
        }
        if (gl == 0) sh.z[16 * unit + 4 * kq + j] = zkeep;
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (lane == 0) sh.umax[unit] = mx;
      };
      uint4 a0[4], a1[4];
      request(0, a0);
      for (int i = 0; i < mine; i += 2) {
        request(i + 1, a1);
        __builtin_amdgcn_sched_barrier(0);
        consume(i, a0);
        request(i + 2, a0);
        __builtin_amdgcn_sched_barrier(0);
        consume(i + 1, a1);
      }
    } else {
      // as in decode_scores_steps_kernel, G = 1
      constexpr bool MFMA = sizeof(T) == 2;
      const int r = lane >> 4, c = lane & 15, kq = lane & 3, gl = (lane >> 2) & 3, j = r;
      const T* k_pool = (const T*)S.k_pool + (MFMA ? gl * kD + (kq * 4 + j) * 8 : r * kD + 8 * c);
      const T* qr = (const T*)S.q + (size_t)bh * kD;
      float coef[8];
      Raw8<T> bq;
      load_raw8(qr + (MFMA ? kq * 32 + j * 8 : 8 * c), bq);
      if constexpr (!MFMA) widen8(bq, coef);
      const int steps = P / 4, batches = (steps + 3) / 4, total = mine * batches;   // four steps = 16 tokens per batch
      auto request = [&](int i, Raw8<T> (&x)[4]) {
        const int ic = min(i, total - 1), pg = ic / batches, s0 = 4 * (ic - pg * batches);
        const T* kpage = k_pool + ((size_t)__builtin_amdgcn_readlane(l_phys, pg) * S.HkvPool + hkv) * P * kD;
#pragma unroll
        for (int s = 0; s < 4; ++s) load_raw8(kpage + (size_t)(4 * min(s0 + s, steps - 1)) * kD, x[s]);
      };
      float wmax = -INFINITY;
      auto consume = [&](int i, const Raw8<T> (&x)[4]) {
        if (i >= total) return;                                             // wave-uniform
        const int pg = i / batches, bt = i - pg * batches, unit = u0 + NW * pg;
        const int tok0 = __builtin_amdgcn_readlane(l_lp, pg) * P;
        const int keep = MFMA ? kq : c;                                     // the step whose score this lane stores
        float zkeep = -INFINITY;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int st = 4 * bt + s;
          float v = 0.f;
          if constexpr (MFMA) {
            const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4_t d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[s].a),
                                                                      __builtin_bit_cast(bf16x8_t, bq.a), zero, 0, 0, 0);
            const float v01 = (kq & 1) ? d[1] : d[0], v23 = (kq & 1) ? d[3] : d[2];
            v = (kq & 2) ? v23 : v01;
            v += dpp_move<0xB1>(v);
            v += dpp_move<0x4E>(v);
          } else {
            float xv[8];
            widen8(x[s], xv);
#pragma unroll
            for (int q = 0; q < 8; ++q) v = fmaf(coef[q], xv[q], v);
            v = row16_sum(v);
          }
          const float z = st < steps && tok0 + 4 * st + r < n ? S.zscale * v : -INFINITY;
          if (keep == s) zkeep = z;
          wmax = fmaxf(wmax, z);
        }
        if ((MFMA ? gl == 0 : c < 4) && 4 * bt + keep < steps) sh.z[unit * P + 4 * (4 * bt + keep) + r] = zkeep;
        if (bt == batches - 1) {
          wmax = fmaxf(wmax, __shfl_xor(wmax, 16));
          wmax = fmaxf(wmax, __shfl_xor(wmax, 32));
          if (lane == 0) sh.umax[unit] = wmax;
          wmax = -INFINITY;
        }
      };
      Raw8<T> x0[4], x1[4];
      request(0, x0);
      for (int i = 0; i < total; i += 2) {
        request(i + 1, x1);
        __builtin_amdgcn_sched_barrier(0);
        consume(i, x0);
        request(i + 2, x0);
        __builtin_amdgcn_sched_barrier(0);
        consume(i + 1, x1);
      }
    }
  }
  __syncthreads();
  const int upg = gp * UPP;                               // units per group of at most 64 tokens
  const RowRef R{b, bh, bh, hkv, n_slots * P, gp * P, (n_slots + gp - 1) / gp};
  if (w == 0) {
    auto group_max = [&](int g) {
      float mx = -INFINITY;
      for (int i = 0; i < upg; ++i) mx = fmaxf(mx, sh.umax[min(g * upg + i, max(n_units - 1, 0))]);
      return mx;
    };
    bound_groups<(decltype(sh)::kGroups + 63) / 64, true>(group_max, R.n_chunks, A.beta, A.ibeta, sh);
  }
  __syncthreads();
  const bool block_extras = A.ex.tau_ref != nullptr && (A.ex.kept_mass_ref != nullptr || A.ex.kept_supp_ref != nullptr);
  solve_bounded_row<T, false>(A, R, sh.z, seed_z, block_extras, sh);
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
// Workgroups per compute unit in a pass-1 launch; never more than the lists can hold items for, and independent of how full
// they are.  Eight are resident at a time; launching twice that (when there
// is that much work) measured 3-5 % faster than a grid of resident workgroups only -- a wavefront that starts fresh
// streams better than one that loops -- while workgroups that find no work cost about half a microsecond per
// thousand, which bounds what a list capacity far above the lists' lengths can cost.  Every workgroup reads the U
// lengths, so launches with many units get fewer.
// When every page is a candidate the launch is large whatever the lists hold, and one item per wavefront, left to
// the hardware's scheduling, is up to 4 % faster: such launches get up to 128 workgroups per compute unit (32 when the units
// are so many that reading their lengths is a cost of its own).  Of these come here what decode_windows.hip does not take:
// float32, other page sizes, shorter calls, more units.  Calls, us, 16 / 128: float32 2 x 131072 209.5 / 205.2, 64 x 4096 215.1 /
// 210.4, pages of 48 tokens 1 x 1048576 462 / 449, of 12 64 x 8192 241 / 232, 2 x 131072 122.9 / 122.9, bf16 1 x 32768 and 3 x 32768
// the same.
static int score_wgs_per_cu(int U, bool all_pages) {
  if (all_pages) return U <= 1024 ? 128 : 32;
  return U <= 256 ? 16 : 8;
}

template <int G, int MODE>
static void launch_scores(const Dims& dm, ScoreArgs sa, int32_t* pre_ws, hipStream_t st) {
  const int gp = pmax_pages(dm.P);
  const long long max_items = (long long)sa.U * (((MODE == kAllPages ? dm.Mmax : dm.cap) + gp - 1) / gp);
  long long wgs = (max_items + kScoreWaves - 1) / kScoreWaves;
  const long long wg_cap = (long long)device_compute_units() * score_wgs_per_cu(sa.U, MODE == kAllPages);
  if (wgs > wg_cap) wgs = wg_cap;
  if (wgs < 1) wgs = 1;
  const bool pre_global = sa.U > kUnitsLdsMax;
  // Lists are split over the XCDs as long as a wavefront's range is not longer than one and a half parts.  Where it spans
  // more, it takes the same part of the heads of a group one after the other, hundreds of megabytes of other reads apart, and
  // the pages they share are fetched again; unsplit, the heads meet in the cache all XCDs share.  Score pass, us, unsplit /
  // split, for heads that select the same, half the same and hardly the same pages (a tenth of a sequence):
  //   1024 units 246 / 125, 261 / 186, 253 / 231    1056 units 128 / 90, 129 / 121, 145 / 147    1536 units 390 / 360, 393 / 374, 422 / 433
  //   2048 units 501 / 453, 486 / 525, 606 / 583    4096 units 647 / 1204, 875 / 1202, 932 / 1261
  const bool split = MODE == kPerHead && dm.G > 1 && !pre_global && 3 * wgs * kScoreWaves >= 2ll * kXcds * sa.U;
  sa.parts = split ? kXcds : 1;
  if (split) wgs = (wgs + kXcds - 1) / kXcds * kXcds;
  dim3 grid((unsigned)wgs), block(kScoreThreads);
  const size_t lds = pre_global ? 0 : (size_t)(sa.U + 1) * sizeof(int);
  if (pre_global) {
    sa.pre_g = pre_ws;
    hipLaunchKernelGGL((unit_prefix_kernel<MODE>), dim3(1), dim3(1024), 0, st, sa, pre_ws);
  }
  // K of a large call over all pages, or over lists that the heads of a group share or that are one head's own, passes once
  // and goes past the caches (load16<true>).  Calls, us, kept / past the caches (before large bf16 calls over all pages moved to
  // decode_windows.hip): all pages of 1 x 1M tokens 473 / 427, 8 x
  // 256K in pages of 32 954 / 925, 2 x 128K for 64 heads 140.7 / 124.4, 2 x 128K in pages of 12 135.1 / 125.7, 2 x 32K (134
  // MB) 41.8 / 37.4; 1 x 32K 23.4 / 22.5 with four inputs in turn, 22.4 / 22.9 with three, which the last cache holds, 1 x
  // 4K 13.4 / 13.8.  Group steps, whose lists follow a stream of statistics, by the capacity, all that the host knows (it
  // is filled to half here): 134 MB 61.6 / 56.3, 86 MB 87 / 86, 67 MB 34.7 / 34.1, 17 MB 26.4 / 27.2.  float32 with both
  // loads of a row on whole lines (load_halves): 2 x 128K 229 / 208, on half lines 249.  Lists of heads without a group:
  // Gaussian steps of 4 x 128K 71.0 / 67.4, 8 x 32K 89.6 / 79.8, refined 4 x 32K 99.9 / 90.1, top-k by capacity 268 MB 69.8
  // / 63.8, 134 MB 44.3 / 43.2, 67 MB 33.9 / 33.7.  Lists per head of a group meet in the caches (16 x 16K Gaussian step
  // 253 / 324) and keep theirs.  The line is the capacity's, not the lists': lists of 4K tokens in a capacity of a million,
  // repeated, take 12.8 / 13.5 (on changing inputs 13.5 / 13.7); kernels with both loops, which choose by the lists, take 13.2
  // there but 31.3 for 28.8 over all pages of 4K tokens in that capacity.
  const long long k_bytes = (long long)sa.U * (MODE == kAllPages ? dm.Mmax : dm.cap) * dm.P * kD * (dm.dtype == EKV_F32 ? 4 : 2);
  const bool past_caches = (MODE != kPerHead || dm.G == 1) && k_bytes >= (MODE == kAllPages ? kStreamKBytes : kStreamListBytes);
  if constexpr (MODE == kAllPages)
    if (launch_scores_windows<G>(dm, sa, max_items, (size_t)k_bytes, st)) return;
#define EKV_SCORES_S(KERNEL, STREAM, ...)                                                                 \
  do {                                                                                                       \
    if (pre_global) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STREAM, true>), grid, block, lds, st, sa);     \
    else hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STREAM, false>), grid, block, lds, st, sa);               \
  } while (0)
#define EKV_SCORES(KERNEL, ...)                                                  \
  do {                                                                           \
    if (past_caches) EKV_SCORES_S(KERNEL, true, __VA_ARGS__);                     \
    else EKV_SCORES_S(KERNEL, false, __VA_ARGS__);                                \
  } while (0)
  if (dm.dtype == EKV_BF16 && dm.P == 16) EKV_SCORES(decode_scores_mfma_kernel, G, MODE, 16);
  else if (dm.dtype == EKV_BF16 && dm.P == 32) EKV_SCORES(decode_scores_mfma_kernel, G, MODE, 32);
  else if (dm.dtype == EKV_BF16 && dm.P == 64) EKV_SCORES(decode_scores_mfma_kernel, G, MODE, 64);
  else if (dm.dtype == EKV_BF16) EKV_SCORES(decode_scores_steps_kernel, bf16_t, G, MODE);
  else EKV_SCORES(decode_scores_steps_kernel, float, G, MODE);
#undef EKV_SCORES
#undef EKV_SCORES_S
}

// Pass 2: one workgroup per row; four wavefronts, and four rows to a compute unit, for many short rows.  A flat row outgrows
// their smaller LDS lists sooner and has a quarter of the wavefronts for its values, which shows while the compute units
// hold all rows at once.  Dense calls, us, support 40 / 2100 / 11 000 of 16K tokens (256 groups): 512 rows by sixteen
// wavefronts 130 / 189 / 378, by four 125 / 219 / 429, by the solve before the segments 135 / 247 / 411; 2048 rows 512 / 911 /
// 1557 before, by four 467 / 717 / 1474.  12 000 tokens (188 groups), 288 rows: 70 / 154 / 254 before, by four 59 / 151 / 252.
// One wavefront per row beyond two rows per compute unit, where a row has at most kOneGroups groups.  Whole grouped calls, us,
// four wavefronts against one: 2048 rows of 512 of 1024 tokens 35.1 / 23.6, of 1024 tokens with a support of 700 107 / 97.5,
// of 256 tokens, nearly all of them support, 49 / 30; 512 rows of 1024 tokens, support 700, 39.8 / 68, 288 rows 28 / 47.
// Only nearly full supports of 512-token lists are slower than in the kernel that solved from zmax - 1 with all scores in
// registers and agreed with the per-head decode to rounding only (2048 rows, support 440: 54.7 -> 58.3); peaked rows gain 20 %.
template <typename T, bool DENSE>
static void launch_solve(int rows, int n_chunks_max, const SolveArgs& so, hipStream_t st) {
  if constexpr (!DENSE)
    if (rows > 2 * device_compute_units() && n_chunks_max <= kOneGroups) {
      hipLaunchKernelGGL((decode_solve_one_kernel<T>), dim3(rows), dim3(64), 0, st, so);
      return;
    }
  const int cus = device_compute_units();
  if (rows > cus && n_chunks_max <= (rows > 2 * cus ? SolveSharedMany::kMaxGroups : SolveSharedMany::kMaxGroups / 4 * 3))
    hipLaunchKernelGGL((decode_solve_kernel<T, DENSE, SolveSharedMany>), dim3(rows), dim3(64 * SolveSharedMany::kWaves), 0, st, so);
  else
    hipLaunchKernelGGL((decode_solve_kernel<T, DENSE, SolveShared>), dim3(rows), dim3(64 * SolveShared::kWaves), 0, st, so);
}

// Short per-head lists, one workgroup each: sixteen wavefronts as long as every list has a compute unit to itself (the
// length of one list is what the call takes), else four, and three to six lists share a compute unit.
// One compute unit reads K at about 75 GB/s, so the line follows the bytes of a list; the host knows its capacity only, and
// a full list near the line of a few rows is a little faster in two launches, a half full one in one.  Decode calls on K that
// is in no cache, us, two launches / one, lists of the heads of a group the same, half the same, hardly the same:
//   32 half full lists of 2048 bf16 tokens 14.0 / 11.7, 14.4 / 12.2, 14.3 / 12.2, full 14.4 / 15.8, 14.8 / 15.8, 14.8 / 15.9
//   128 full lists of 4096 21.4 / 23.4, 26.2 / 24.1, 29.6 / 26.8    256 of them 30.7 / 23.4, 39.4 / 36.3, 46.7 / 43.9
//   512 full lists of 2048 31.4 / 22.9, 45.2 / 30.5, 50.7 / 40.7    2048 of them 182 / 81, 181 / 108, 209 / 151
// and 64 float32 lists of 1024 tokens, half full 19.2 / 12.6, full 20.3 / 16.4.  The heads of a group run on one XCD: dealt
// out in turn they fetched the pages they share into as many L2s (256 full lists of 4096: 45.6, 43.4, 44.2; before there was
// the one launch 35.5, 45.8, 52.1).
static bool rows_in_one_launch(const Dims& dm) {
  const int cus = device_compute_units(), rows = dm.B * dm.Hq;
  const long long tokens = (long long)dm.cap * dm.P;
  if (rows > cus) return tokens <= kRowTokensMany;
  const long long bytes = tokens * kD * (dm.dtype == EKV_F32 ? 4 : 2);
  return tokens <= kRowTokens && bytes <= (rows <= cus / 4 ? 512 << 10 : 1 << 20);
}
template <typename T, int PT>
static void launch_rows_T(const Dims& dm, const ScoreArgs& sa, const SolveArgs& so, hipStream_t st) {
  const int rows = dm.B * dm.Hq;
  if (rows <= device_compute_units())
    hipLaunchKernelGGL((decode_row_kernel<T, PT, 16, kRowTokens>), dim3(rows), dim3(1024), 0, st, sa, so);
  else if ((long long)dm.cap * dm.P <= kRowTokensMany / 2)
    hipLaunchKernelGGL((decode_row_kernel<T, PT, 4, kRowTokensMany / 2>), dim3(rows), dim3(256), 0, st, sa, so);
  else
    hipLaunchKernelGGL((decode_row_kernel<T, PT, 4, kRowTokensMany>), dim3(rows), dim3(256), 0, st, sa, so);
}
static void launch_rows(const Dims& dm, const ScoreArgs& sa, const SolveArgs& so, hipStream_t st) {
  if (dm.dtype == EKV_F32) launch_rows_T<float, 0>(dm, sa, so, st);
  else if (dm.P == 16) launch_rows_T<bf16_t, 16>(dm, sa, so, st);
  else if (dm.P == 32) launch_rows_T<bf16_t, 32>(dm, sa, so, st);
  else if (dm.P == 64) launch_rows_T<bf16_t, 64>(dm, sa, so, st);
  else launch_rows_T<bf16_t, 0>(dm, sa, so, st);
}

size_t decode_ws_carve(const Dims& dm, bool dense, void* base, DecodeWorkspace* ws) {
  const size_t slots = dense ? dm.Mmax : dm.cap;
  const size_t rows = (size_t)dm.B * dm.Hq;
  const size_t zstride = slots * dm.P;
  const int n_chunks_max = (int)((slots + pmax_pages(dm.P) - 1) / pmax_pages(dm.P));
  size_t n_slices = ((size_t)n_chunks_max + kFilterSliceChunks - 1) / kFilterSliceChunks;
  if (n_chunks_max <= kPreGroups || n_slices > (size_t)kFilterMaxSlices) n_slices = 0;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
  const size_t o_z = take(rows * zstride * sizeof(float));
  const size_t o_pm = take(rows * n_chunks_max * sizeof(float));
  const size_t o_pre = take((rows + 1) * sizeof(int32_t));
  // overflow list of a row whose candidates outgrow the solve's LDS list: (u, position) per entry
  const size_t spill_cap = zstride > (size_t)kListCap ? (zstride < (size_t)kSpillCap ? zstride : (size_t)kSpillCap) : 0;
  const size_t o_su = spill_cap ? take(rows * spill_cap * sizeof(float)) : 0;
  const size_t o_sp = spill_cap ? take(rows * spill_cap * sizeof(int32_t)) : 0;
  size_t o_fc = 0, o_fr = 0, o_fu = 0, o_fp = 0;
  if (n_slices) {
    o_fc = take(rows * n_slices * sizeof(int32_t));
    o_fr = take(rows * 2 * sizeof(float));
    o_fu = take(rows * n_slices * kFilterSliceCap * sizeof(float));
    o_fp = take(rows * n_slices * kFilterSliceCap * sizeof(int32_t));
  }
  if (ws != nullptr && base != nullptr) {
    char* p = (char*)base;
    ws->z = (float*)(p + o_z); ws->pmax = (float*)(p + o_pm); ws->unit_pre = (int32_t*)(p + o_pre);
    ws->zstride = zstride; ws->n_chunks_max = n_chunks_max; ws->n_slices_max = (int)n_slices;
    ws->spill_u = spill_cap ? (float*)(p + o_su) : nullptr;
    ws->spill_pos = spill_cap ? (int32_t*)(p + o_sp) : nullptr;
    ws->spill_cap = (int)spill_cap;
    ws->fcount = n_slices ? (int32_t*)(p + o_fc) : nullptr;
    ws->frow = n_slices ? (float*)(p + o_fr) : nullptr;
    ws->flist_u = n_slices ? (float*)(p + o_fu) : nullptr;
    ws->flist_pos = n_slices ? (int32_t*)(p + o_fp) : nullptr;
  }
  return off;
}

void launch_decode(const Dims& dm, bool dense, bool grouped, const void* q, const ekv_cache_view& c,
                   const int32_t* page_idx, const int32_t* n_sel, float* out, float* tau, int32_t* supp,
                   const ekv_decode_extras& ex, const DecodeWorkspace& ws, hipStream_t st) {
  ScoreArgs sa{q, c.k_pool, c.block_table, c.seq_lens, page_idx, n_sel, ws.z, ws.pmax,
               dm.Hq, dm.Hkv, dm.P, dm.Mmax, dm.cap, ws.n_chunks_max, c.n_phys_pages, ws.zstride, dm.a * dm.scale,
               dm.HkvPool, 0, nullptr, 1};
  SolveArgs so{c.v_pool, c.block_table, c.seq_lens, page_idx, n_sel, ws.z, ws.pmax, out, tau, supp, ex,
               dm.Hq, dm.Hkv, dm.P, dm.Mmax, dm.cap, ws.n_chunks_max, c.n_phys_pages, ws.zstride, dm.a, dm.beta, dm.ibeta};
  so.fcount = ws.fcount; so.frow = ws.frow; so.flist_u = ws.flist_u; so.flist_pos = ws.flist_pos;
  so.n_slices_max = ws.n_slices_max;
  so.grouped = grouped ? 1 : 0;
  so.HkvPool = dm.HkvPool;
  so.spill_u = ws.spill_u; so.spill_pos = ws.spill_pos; so.spill_cap = ws.spill_cap;
  FilterArgs fa{c.seq_lens, n_sel, ws.z, ws.pmax, ws.fcount, ws.frow, ws.flist_u, ws.flist_pos,
                dm.Hq, dm.Hkv, grouped ? 1 : 0, dm.P, ws.n_slices_max, dense ? dm.Mmax : dm.cap, ws.n_chunks_max,
                ws.zstride, dm.beta, dm.ibeta};
  dim3 fgrid(ws.n_slices_max, dm.B * dm.Hq), fblock(kFilterThreads);
  const int rows = dm.B * dm.Hq;
  if (dense) {
    sa.U = dm.B * dm.Hkv;
    switch (dm.G) {
      case 1: launch_scores<1, kAllPages>(dm, sa, ws.unit_pre, st); break;
      case 2: launch_scores<2, kAllPages>(dm, sa, ws.unit_pre, st); break;
      case 4: launch_scores<4, kAllPages>(dm, sa, ws.unit_pre, st); break;
      default: launch_scores<8, kAllPages>(dm, sa, ws.unit_pre, st); break;
    }
    if (ex.score_pass_only) return;
    if (ws.fcount != nullptr) {
      hipLaunchKernelGGL((filter_level_kernel<true>), dim3(dm.B * dm.Hq), fblock, 0, st, fa);
      hipLaunchKernelGGL((filter_compact_kernel<true>), fgrid, fblock, 0, st, fa);
    }
    if (dm.dtype == EKV_F32) launch_solve<float, true>(rows, ws.n_chunks_max, so, st);
    else launch_solve<bf16_t, true>(rows, ws.n_chunks_max, so, st);
  } else {
    if (grouped && dm.G > 1) {
      sa.U = dm.B * dm.Hkv;
      switch (dm.G) {
        case 2: launch_scores<2, kGroupList>(dm, sa, ws.unit_pre, st); break;
        case 4: launch_scores<4, kGroupList>(dm, sa, ws.unit_pre, st); break;
        default: launch_scores<8, kGroupList>(dm, sa, ws.unit_pre, st); break;
      }
    } else {                                    // G == 1: a group list is a per-head list
      sa.U = dm.B * dm.Hq;
      if (rows_in_one_launch(dm) && !ex.score_pass_only) { launch_rows(dm, sa, so, st); return; }
      launch_scores<1, kPerHead>(dm, sa, ws.unit_pre, st);
    }
    if (ex.score_pass_only) return;
    if (ws.fcount != nullptr) {
      hipLaunchKernelGGL((filter_level_kernel<false>), dim3(dm.B * dm.Hq), fblock, 0, st, fa);
      hipLaunchKernelGGL((filter_compact_kernel<false>), fgrid, fblock, 0, st, fa);
    }
    if (dm.dtype == EKV_F32) launch_solve<float, false>(rows, ws.n_chunks_max, so, st);
    else launch_solve<bf16_t, false>(rows, ws.n_chunks_max, so, st);
  }
}

}  // namespace ekv
