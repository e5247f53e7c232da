// Tiled gridder: each work item is a run of binned records of one uv-tile.  One
// wavefront owns the work item and accumulates its records in a private LDS copy of
// the tile plus an (S_max - 1)-cell halo on the high-x / high-y sides, then stores the
// copy to the work item's slot of a partial-tile buffer; tile_reduce_kernel adds the
// slots to the grid, one thread per cell in a fixed order (no atomics; the sum over the
// partial tiles does not depend on scheduling, though the order of records inside a bin,
// and so the FP32 rounding inside a partial tile, follows the binning's count atomics).
// The read-modify-write traffic of gridding therefore stays in LDS instead of going to
// HBM (the paper's CUDA gridder, Section 2.2, keeps one thread per kernel tap and
// baseline, sums that baseline's consecutive timestamps in a register and writes to the
// grid in global memory with an atomic add when it moves to the next baseline).
//
// Because the tile is private to one wavefront and its 64 lanes always touch 64
// distinct cells of a record's footprint, the accumulation is a plain LDS read, add and
// write: instructions of one wavefront reach LDS in order, so a later record sees the
// earlier record's update without atomics.  (LDS floating-point atomics on this chip
// retire at only a few lanes per clock; plain 64-bit reads and writes run at full
// LDS bandwidth.)  Tiles are small (16 or 32 cells) so that a CU holds many wavefronts,
// each with its own tile, to hide LDS and memory latency.
//
// Launch is persistent: enough wavefronts to fill every CU pull work items from queues in
// HBM until they are empty, which evens out the very uneven per-tile visibility counts of
// Earth-rotation tracks.  With a fixed support each lane handles one tap of every record per
// pass of 64 taps.  Records arrive 32 at a time in row-replicated registers, whose DPP
// broadcast rides in the instruction that uses a field: a record costs six vector
// instructions (one address add, four multiply-adds, half a table address and half a swap)
// where readlane broadcasts took eleven.  With FP32 arithmetic two records share a table
// load (one record per half wavefront, then a half-wavefront swap), and a group's loads stay
// one group of 16 records ahead of their use.
//
// What bounds it (5.6e7 records, 2048^2 grid, S = 8, 128 planes, 32-cell tiles): the taps' path
// from L2 through the L1 caches, whose data return is busy for 95 % of the launch and waits for
// L2 in 32 % of it.  A record's 512 bytes of taps come almost always from L2 (a tile holds
// fewer records of a plane than the plane has sub-kernels), 27 GB a launch at 20 TB/s.  1.53 ms with readlane broadcasts, 1.73 with DPP but loads left to the compiler's
// order, 1.40 with the loads held a group ahead and 16 records a group; with 16-cell tiles
// 1.33, and 1.05 if every tap hit L1.  Two half-wavefront gridders with a tile copy each
// (no swap, 25 instead of 32 clocks of issue a record) took 1.54 and 1.39 ms: LDS then holds
// half as many wavefronts, and issue no longer bounds the loop.
#pragma once

#include <algorithm>
#include <type_traits>

#include "wproj_tiled.h"

namespace wproj {
namespace {

__device__ inline float2 tab_load(const float2 *t, uint32_t i) { return t[i]; }
__device__ inline double2 tab_load(const double2 *t, uint32_t i) { return t[i]; }
__device__ inline float2 tab_load(const half2c *t, uint32_t i) {
  const half2c h = t[i];
  return make_float2((float)h.re, (float)h.im);
}

// FP64 table fetch through a buffer resource.
__device__ inline double2 tab_fetch(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0);
  const uint32_t w0 = v[0], w1 = v[1], w2 = v[2], w3 = v[3];
  const uint64_t re = (uint64_t)w0 | ((uint64_t)w1 << 32);
  const uint64_t im = (uint64_t)w2 | ((uint64_t)w3 << 32);
  return make_double2(__longlong_as_double((long long)re), __longlong_as_double((long long)im));
}
__device__ inline float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename Real> struct Cx;
template <> struct Cx<float> { using T = float2; };
template <> struct Cx<double> { using T = double2; };

// Table loads per group in one pass (8 pairs of records in FP32, 8 records in FP64), all
// issued before the first is consumed, so up to kGroup memory latencies overlap per
// wavefront.
constexpr int kGroup = 8;
// The same for the per-record-support path, whose table misses reach past L2.
constexpr int kVarGroup = 16;

// One tap of an FP32 or FP16 table loaded through a buffer resource (lane's byte offset
// in the vector offset, the sub-kernel's in the scalar offset), kept raw until use.
template <typename Tab> struct TapRaw;
template <> struct TapRaw<float2> {
  typedef uint32_t T __attribute__((ext_vector_type(2)));
  __device__ static T load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
  }
  __device__ static float2 value(const T &v) { return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1])); }
};
template <> struct TapRaw<half2c> {
  typedef uint32_t T;
  __device__ static T load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
  }
  __device__ static float2 value(const T &v) {
    half2c h;
    __builtin_memcpy(&h, &v, 4);
    return make_float2((float)h.re, (float)h.im);
  }
};
template <> struct TapRaw<double2> {  // the per-record-support fast path is FP32 only
  typedef double2 T;
};
constexpr int kMaxWavesPerBlock = 4;
// Support parameter of the kernel for large supports, and the rows from which it is taken.
constexpr int kLargeSupports = -1;
constexpr int64_t kManyLargeRows = 1 << 21;

// A row-carrying record (weight, row) turned into W V from the visibility it names; a
// negative weight marks a Hermitian-folded row, which enters as W conj(V).
template <typename Rec, typename C2>
__device__ inline void to_weighted(Rec &r, const C2 &v) {
  const auto wgt = r.wr;
  r.wr = fabs(wgt) * v.x;
  r.wi = wgt * v.y;
}

// One record's read-add-write of its 64-cell footprint (lane = tap) in the private tile.
template <typename C2, typename Real, typename Tap>
__device__ inline void accumulate(C2 *acc, int a, Real wr, Real wi, const Tap &t) {
  C2 v = acc[a];
  v.x = fmadd(wr, (Real)t.x, v.x);
  v.x = fmadd(-wi, (Real)t.y, v.x);
  v.y = fmadd(wr, (Real)t.y, v.y);
  v.y = fmadd(wi, (Real)t.x, v.y);
  acc[a] = v;
}

// The same with W V from row-replicated registers (record I of 16), on a held value.
template <int I, typename C2, typename Real, typename Tap>
__device__ inline void mac_bcast(C2 &v, Real wr, Real wi, const Tap &t) {
  fmac_bcast<I>(v.x, wr, t.x);
  fmsc_bcast<I>(v.x, wi, t.y);
  fmac_bcast<I>(v.y, wr, t.y);
  fmac_bcast<I>(v.y, wi, t.x);
}

// S = fixed support (0 = per-record support, kLargeSupports = per-record support, light).  PLANNED: the records are row-carrying
// (weight, row) and W V is formed from vis[row] as each record is loaded.  RUNS (paired
// fixed-support path only): while consecutive records of the work item share the
// footprint origin, each lane keeps its cell of the footprint in a register and writes it
// back to the tile only when the origin changes.  The multiply-adds and their order are
// those of the plain read-add-write, so the result is the same bit for bit.
template <typename Real, typename Rec, typename Tab, int S, bool PLANNED, bool RUNS = false>
__global__ void __launch_bounds__(64 * kMaxWavesPerBlock)
    tiled_grid_kernel(Geometry G, BinShape B, int pitch, int rows, int wave_lds,
                      const Tab *__restrict__ tab, uint32_t tab_bytes,
                      const Rec *__restrict__ rec, const WorkItem *__restrict__ items,
                      const uint32_t *__restrict__ order,
                      const uint32_t *__restrict__ n_items_ptr, uint32_t *queues, uint32_t n_queues,
                      typename Cx<Real>::T *__restrict__ partial,
                      const typename Cx<Real>::T *__restrict__ vis) {
  using C2 = typename Cx<Real>::T;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  C2 *acc = reinterpret_cast<C2 *>(smem_raw) + (size_t)wid * wave_lds;
  const uint32_t n_items = *n_items_ptr;
  const int area = rows * pitch;
  // LDS byte address of acc
  const uint32_t acc0 = lds_address(smem_raw) + (uint32_t)wid * (uint32_t)wave_lds * (uint32_t)sizeof(C2);
  const __amdgpu_buffer_rsrc_t tab_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)tab, (short)0, (int)tab_bytes, kBufferWord3);
  WorkQueue queue(queues, n_queues);

  for (;;) {
    uint32_t got = 0;
    if (lane == 0) got = queue.next();
    const uint32_t it = (uint32_t)__builtin_amdgcn_readlane((int)got, 0);
    if (it >= n_items) break;
    const uint32_t item = order[it];  // largest items first
    const WorkItem w = items[item];
    for (int i = lane; i < area; i += 64) acc[i] = C2{Real(0), Real(0)};
    const uint32_t n_rec = w.end - w.begin;
    // Records arrive with one coalesced load a batch (lanes i and 32 + i hold record i).
    constexpr bool kPaired = S > 0 && kPairedTab<Tab>;
    constexpr uint32_t kBatch = 32;
    const uint32_t slot = (uint32_t)lane & (kBatch - 1u);
    // Lanes past the last record load it again, so that no load hides behind a branch (the
    // compiler then knows how many are in flight); weigh gives them zero weight.
    auto load_rec = [&](uint32_t b, Rec &dst) { dst = rec[w.begin + min(b + slot, n_rec - 1u)]; };
    // row-carrying records: the visibilities they name
    auto load_vis = [&](const Rec &r, C2 &v) {
      if constexpr (PLANNED) v = vis[get_row(r)];
    };
    auto weigh = [&](uint32_t b, Rec &r, const C2 &v) {
      if constexpr (PLANNED) to_weighted(r, v);
      if (b + slot >= n_rec) r.wr = r.wi = Real(0);
    };
    auto load_batch = [&](uint32_t b, Rec &dst) {
      C2 v;
      load_rec(b, dst);
      load_vis(dst, v);
      weigh(b, dst, v);
    };

    if constexpr (kPaired) {
      // Fixed support, FP32 arithmetic: lane = tap, and records 2i and 2i + 1 share one load
      // of taps.
      using P = TapPair<Tab>;
      using Raw = typename P::Raw;
      constexpr int kPasses = pair_passes(S);
      constexpr int kPairs = kPasses == 1 ? kGroup : kPasses == 2 ? kGroup / 2 : kGroup / 4;  // per group
      constexpr int kGroups = 16 / kPairs;
      // Lanes j and 32 + j load entry pair j of records 2i and 2i + 1; after the swap, lane j
      // (< 32) holds tap 64q + j and lane 32 + j tap 64q + h + j of both records.  In full
      // passes that is tap 64q + lane, whose 64-bit LDS accesses the row pitch keeps free of
      // bank conflicts (pairs of adjacent taps would put each half wavefront on every second
      // column of eight rows, which no uniform pitch spreads over all banks).
      const int half = lane >> 5, j = lane & 31;
      uint32_t p_off[kPasses];  // LDS byte address of the lane's cell of a footprint at cell 0
      bool p_on[kPasses];
      uint32_t p_pair[kPasses];  // byte offset of the lane's entry pair inside a sub-kernel
#pragma unroll
      for (int q = 0; q < kPasses; ++q) {
        const int n_q = pair_taps(S, q), h_q = pair_half(S, q);
        const int t = 64 * q + (half ? h_q : 0) + j;
        p_on[q] = half ? j < n_q - h_q : j < h_q;
        p_off[q] = acc0 + (p_on[q] ? (uint32_t)((t / S) * pitch + t % S) * 8u : 0u);
        p_pair[q] = (uint32_t)(64 * q + (j < h_q ? 2 * j : 0)) * P::kTapBytes;
      }
      // The records carry their sub-kernel number above the LDS offset; a sub-kernel takes
      // pair_stride(S) entries of the pair-ordered table.
      constexpr uint32_t kSubBytes = (uint32_t)pair_stride(S) * P::kTapBytes;
      struct Batch {  // records 16 g .. 16 g + 15, row-replicated: LDS and table offsets, W V
        uint32_t cell[2], sub[2];
        float wr[2], wi[2];
      };
      auto unpack = [&](const Rec &r) {
        Batch o;
        replicate16((r.lds & kLdsMask) * 8u, o.cell);
        replicate16((r.lds >> kLdsBits) * kSubBytes, o.sub);
        replicate16(r.wr, o.wr);
        replicate16(r.wi, o.wi);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          // the upper half wavefront's sub-kernels moved down one record, so that one
          // broadcast gives records 2i and 2i + 1 to the two halves
          o.sub[g] = (uint32_t)__builtin_amdgcn_update_dpp((int)o.sub[g], (int)o.sub[g], 0x101, 0xC, 0xF, false);
          dpp_ready(o.cell[g], o.sub[g], o.wr[g], o.wi[g]);
        }
        return o;
      };
      auto fetch = [&](auto pair, const Batch &bt, Raw (&dst)[kPasses]) {
        constexpr int g = decltype(pair)::value / 8, i = 2 * (decltype(pair)::value % 8);
#pragma unroll
        for (int q = 0; q < kPasses; ++q) dst[q] = P::load(tab_rsrc, add_bcast<i>(bt.sub[g], p_pair[q]));
      };
      // RUNS: the lane's cells of the current origin (one per pass) and that origin's LDS
      // byte offset (wave-uniform; none before the first record)
      constexpr uint32_t kNone = 0xffffffffu;
      float2 held[kPasses];
      uint32_t held_base = kNone;
      auto put_back = [&]() {
#pragma unroll
        for (int q = 0; q < kPasses; ++q)
          if (held_base != kNone && p_on[q]) lds_write(held_base + p_off[q], held[q]);
      };
      auto add_record = [&](auto rec_no, const Batch &bt, const float2 (&t)[kPasses]) {
        constexpr int g = decltype(rec_no)::value / 16, i = decltype(rec_no)::value % 16;
        if constexpr (RUNS) {
          const uint32_t base = bcast(bt.cell[g], i);
          if (base != held_base) {  // a new origin: write the held cells back, load the new ones
            put_back();
#pragma unroll
            for (int q = 0; q < kPasses; ++q) lds_read(base + p_off[q], held[q]);
            held_base = base;
          }
#pragma unroll
          for (int q = 0; q < kPasses; ++q) mac_bcast<i>(held[q], bt.wr[g], bt.wi[g], t[q]);
        } else {
          uint32_t a[kPasses];
          float2 v[kPasses];
#pragma unroll
          for (int q = 0; q < kPasses; ++q) {
            a[q] = add_bcast<i>(bt.cell[g], p_off[q]);
            lds_read(a[q], v[q]);
          }
#pragma unroll
          for (int q = 0; q < kPasses; ++q) {
            mac_bcast<i>(v[q], bt.wr[g], bt.wi[g], t[q]);
            if (p_on[q]) lds_write(a[q], v[q]);
          }
        }
      };
      // Software pipeline: a group's taps load while the previous group is added, across
      // batches too; the next batch's records load a whole batch ahead (and, when they
      // name rows, the rows' visibilities load a batch ahead and the records two).  Loads
      // return in order, so the records are asked for after the taps of the group that
      // follows: waiting for those taps does not wait for the records.
      Rec nxt, nxt2;
      C2 vnext;
      load_rec(0, nxt);
      load_vis(nxt, vnext);
      weigh(0, nxt, vnext);
      Batch cur = unpack(nxt);
      load_rec(kBatch, nxt);
      Raw c[2][kPairs][kPasses];
      static_for<0, kPairs>([&](auto i) { fetch(i, cur, c[0][decltype(i)::value]); });
      if constexpr (PLANNED) load_rec(2 * kBatch, nxt2);
      for (uint32_t b = 0; b < n_rec; b += kBatch) {
        load_vis(nxt, vnext);
        Batch next;
        static_for<0, kGroups>([&](auto gi) {
          constexpr int gI = decltype(gi)::value;
          if constexpr (gI + 1 < kGroups) {
            static_for<0, kPairs>([&](auto i) {
              constexpr int pr = (gI + 1) * kPairs + decltype(i)::value;
              fetch(std::integral_constant<int, pr>{}, cur, c[(gI + 1) & 1][decltype(i)::value]);
            });
          } else {
            weigh(b + kBatch, nxt, vnext);
            next = unpack(nxt);
            static_for<0, kPairs>([&](auto i) { fetch(i, next, c[(gI + 1) & 1][decltype(i)::value]); });
            if constexpr (PLANNED) {
              nxt = nxt2;
              load_rec(b + 3 * kBatch, nxt2);
            } else {
              load_rec(b + 2 * kBatch, nxt);
            }
          }
          // the loads stay ahead of the additions (the scheduler would otherwise reuse each
          // tap register at once and issue every load late)
          __builtin_amdgcn_sched_barrier(0);
          static_for<0, kPairs>([&](auto i) {
            constexpr int pr = gI * kPairs + decltype(i)::value;
            // record by record (all passes of record 2i, then of 2i + 1): a cell that both
            // footprints cover through different passes takes its two updates in record
            // order
            float2 t0[kPasses], t1[kPasses];
#pragma unroll
            for (int q = 0; q < kPasses; ++q) P::split(c[gI & 1][decltype(i)::value][q], t0[q], t1[q]);
            add_record(std::integral_constant<int, 2 * pr>{}, cur, t0);
            add_record(std::integral_constant<int, 2 * pr + 1>{}, cur, t1);
          });
        });
        cur = next;
      }
      if constexpr (RUNS) put_back();
    } else if constexpr (S > 0) {
      // Direct-fetch path (fixed support, FP64): lane t handles tap t of every record, in
      // kPasses passes of 64 taps when S^2 > 64.  Table taps are loaded one group of
      // kGroupS records ahead of their use; the group shrinks as the passes grow, so the
      // prefetched taps stay within a fixed register budget.
      constexpr int kPasses = (S * S + 63) / 64;
      constexpr int kGroupS = kPasses == 1 ? kGroup : kPasses == 2 ? kGroup / 2 : kGroup / 4;
      constexpr int kGroups = (int)kBatch / kGroupS;
      uint32_t p_off[kPasses], p_tap[kPasses];  // byte offsets of the lane's cell and tap
      bool p_on[kPasses];
#pragma unroll
      for (int q = 0; q < kPasses; ++q) {
        const int t = q * 64 + lane;
        p_on[q] = t < S * S;
        p_off[q] = acc0 + (p_on[q] ? (uint32_t)((t / S) * pitch + t % S) * 16u : 0u);
        p_tap[q] = p_on[q] ? (uint32_t)t * 16u : 0u;
      }
      struct Batch {  // records 16 g .. 16 g + 15, row-replicated
        uint32_t cell[2], sub[2];
        double wr[2], wi[2];
      };
      auto unpack = [&](const Rec &r) {
        Batch o;
        replicate16((r.lds & kLdsMask) * 16u, o.cell);
        replicate16((r.lds >> kLdsBits) * (uint32_t)(S * S * 16), o.sub);
        replicate16(r.wr, o.wr);
        replicate16(r.wi, o.wi);
#pragma unroll
        for (int g = 0; g < 2; ++g) dpp_ready(o.cell[g], o.sub[g], o.wr[g], o.wi[g]);
        return o;
      };
      auto fetch = [&](auto k, const Batch &bt, double2 (&dst)[kPasses]) {
#pragma unroll
        for (int q = 0; q < kPasses; ++q)
          dst[q] = tab_fetch(tab_rsrc, add_bcast<decltype(k)::value % 16>(bt.sub[decltype(k)::value / 16], p_tap[q]));
      };
      Rec nxt;
      C2 vnext;
      load_rec(0, nxt);
      load_vis(nxt, vnext);
      weigh(0, nxt, vnext);
      Batch cur = unpack(nxt);
      load_rec(kBatch, nxt);
      double2 c[2][kGroupS][kPasses];
      static_for<0, kGroupS>([&](auto i) { fetch(i, cur, c[0][decltype(i)::value]); });
      for (uint32_t b = 0; b < n_rec; b += kBatch) {
        load_vis(nxt, vnext);
        Batch next;
        static_for<0, kGroups>([&](auto gi) {
          constexpr int gI = decltype(gi)::value;
          if constexpr (gI + 1 < kGroups) {
            static_for<0, kGroupS>([&](auto i) {
              constexpr int k = (gI + 1) * kGroupS + decltype(i)::value;
              fetch(std::integral_constant<int, k>{}, cur, c[(gI + 1) & 1][decltype(i)::value]);
            });
          } else {
            weigh(b + kBatch, nxt, vnext);
            next = unpack(nxt);
            static_for<0, kGroupS>([&](auto i) { fetch(i, next, c[(gI + 1) & 1][decltype(i)::value]); });
            load_rec(b + 2 * kBatch, nxt);
          }
          __builtin_amdgcn_sched_barrier(0);
          static_for<0, kGroupS>([&](auto ii) {
            constexpr int k = gI * kGroupS + decltype(ii)::value, g = k / 16, i = k % 16;
            double2 v[kPasses];
            uint32_t a[kPasses];
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
              a[q] = add_bcast<i>(cur.cell[g], p_off[q]);
              lds_read(a[q], v[q]);
            }
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
              mac_bcast<i>(v[q], cur.wr[g], cur.wi[g], c[gI & 1][decltype(ii)::value][q]);
              if (p_on[q]) lds_write(a[q], v[q]);
            }
          });
        });
        cur = next;
      }
    } else if constexpr (kHasTap<Rec> && std::is_same_v<Real, float> && S == 0) {
      // Per-record supports with FP32 arithmetic: lane t handles taps t, 64 + t, ... of a
      // record.  The lane's cells follow the support and are recomputed only when it changes (a
      // tile's records come plane by plane).  A batch whose supports all take one pass (S <= 8)
      // goes as with a fixed support: DPP broadcasts, taps loaded kVarGroup records ahead.  (Lanes
      // t >= S^2 load taps of the next sub-kernel; past the table's end a load gives zero.)
      // Other batches take kPasses passes, 2 (S <= 11) or 4 (S <= 16), their taps loaded
      // kVarGroup/kPasses records ahead; supports beyond 16 load their taps as they go.
      // 5.05e7 rows of S = 4 .. 16 on 4096^2 with an FP16 table: 1.84 ms; 3.94 with readlane
      // broadcasts and no loads ahead for S > 8, whose rows, 7 in 100, took 1.4 ms of it.  Held
      // to 128 registers (four wavefronts per SIMD instead of three) it spills: 2.01 ms.
      using Raw = typename TapRaw<Tab>::T;
      constexpr int kMaxPasses = 4;
      uint32_t s_cur = 0, p_off[kMaxPasses];
      bool p_on[kMaxPasses];
      auto set_support = [&](uint32_t Sn) {
        const float inv = 1.0f / (float)Sn;
#pragma unroll
        for (int q = 0; q < kMaxPasses; ++q) {
          // t / Sn by a float reciprocal: (t + 1/2) / Sn lies at least 1/(2 Sn) from an
          // integer, far beyond the rounding of this product
          const uint32_t t = 64 * q + (uint32_t)lane, kv = (uint32_t)(((float)t + 0.5f) * inv);
          p_on[q] = t < Sn * Sn;
          p_off[q] = acc0 + (p_on[q] ? (kv * (uint32_t)pitch + (t - kv * Sn)) * 8u : 0u);
        }
        s_cur = Sn;
      };
      const uint32_t vlane = (uint32_t)lane * (uint32_t)sizeof(Tab);
      struct Batch {  // records 16 g .. 16 g + 15, row-replicated: LDS and table offsets, W V
        uint32_t cell[2], sub[2];
        float wr[2], wi[2];
        uint32_t support, change;  // lane i's support; bit i: it may differ from the one before
      };
      auto unpack = [&](const Rec &r) {
        Batch o;
        o.support = (r.tap >> kTapBits) + 1u;
        // the support of the lane before, 0 for the first of each row of 16 lanes
        const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)o.support, 0x111, 0xF, 0xF, false);
        o.change = (uint32_t)__ballot(prev != o.support);
        replicate16((r.lds & kLdsMask) * 8u, o.cell);
        replicate16((r.tap & kTapMask) * (uint32_t)sizeof(Tab), o.sub);
        replicate16(r.wr, o.wr);
        replicate16(r.wi, o.wi);
        return o;
      };
      auto fetch_group = [&](auto gi, Batch &bt, Raw (&dst)[kVarGroup]) {
        constexpr int g = decltype(gi)::value;
        dpp_ready(bt.cell[g], bt.sub[g], bt.wr[g], bt.wi[g]);
        static_for<0, kVarGroup>([&](auto i) {
          dst[decltype(i)::value] = TapRaw<Tab>::load(tab_rsrc, add_bcast<decltype(i)::value>(bt.sub[g], vlane), 0);
        });
      };
      auto add_group = [&](auto gi, Batch &bt, const Raw (&src)[kVarGroup]) {
        constexpr int g = decltype(gi)::value;
        static_for<0, kVarGroup>([&](auto ii) {
          constexpr int i = decltype(ii)::value;
          if (bt.change >> (16 * g + i) & 1u) {
            const uint32_t Sr = bcast(bt.support, 16 * g + i);
            if (Sr != s_cur) set_support(Sr);
            dpp_ready(bt.cell[g], bt.sub[g], bt.wr[g], bt.wi[g]);
          }
          const uint32_t at = add_bcast<i>(bt.cell[g], p_off[0]);
          float2 v;
          lds_read(at, v);
          mac_bcast<i>(v, bt.wr[g], bt.wi[g], TapRaw<Tab>::value(src[i]));
          if (p_on[0]) lds_write(at, v);
        });
      };
      // records r (lane i: record i) in kPasses passes
      auto add_passes = [&](auto passes, const Rec &r, uint32_t left) {
        constexpr int kPasses = decltype(passes)::value, kAhead = kVarGroup / kPasses;
        auto fetch = [&](int j, Raw (&dst)[kAhead][kPasses]) {
#pragma unroll
          for (int i = 0; i < kAhead; ++i) {
            const uint32_t tp = bcast(r.tap, j + i), Sr = (tp >> kTapBits) + 1u;
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
              const uint32_t t = 64 * q + (uint32_t)lane;
              dst[i][q] = TapRaw<Tab>::load(tab_rsrc, t < Sr * Sr ? t * (uint32_t)sizeof(Tab) : 0u,
                                            (tp & kTapMask) * (uint32_t)sizeof(Tab));
            }
          }
        };
        auto add = [&](int j, const Raw (&src)[kAhead][kPasses]) {
#pragma unroll
          for (int i = 0; i < kAhead; ++i) {
            const uint32_t Sr = (bcast(r.tap, j + i) >> kTapBits) + 1u;
            if (Sr != s_cur) set_support(Sr);
            const uint32_t base = (bcast(r.lds, j + i) & kLdsMask) * 8u;
            const float rwr = bcast(r.wr, j + i), rwi = bcast(r.wi, j + i);
            float2 v[kPasses];
#pragma unroll
            for (int q = 0; q < kPasses; ++q) lds_read(base + p_off[q], v[q]);
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
              const float2 t = TapRaw<Tab>::value(src[i][q]);
              v[q].x = fmadd(rwr, t.x, v[q].x);
              v[q].x = fmadd(-rwi, t.y, v[q].x);
              v[q].y = fmadd(rwr, t.y, v[q].y);
              v[q].y = fmadd(rwi, t.x, v[q].y);
              if (p_on[q]) lds_write(base + p_off[q], v[q]);
            }
          }
        };
        Raw t0[kAhead][kPasses], t1[kAhead][kPasses];
        fetch(0, t0);
#pragma unroll 1
        for (int j = 0; j < (int)min(kBatch, left); j += 2 * kAhead) {
          fetch(j + kAhead, t1);
          __builtin_amdgcn_sched_barrier(0);
          add(j, t0);
          if (j + 2 * kAhead < (int)kBatch) fetch(j + 2 * kAhead, t0);
          __builtin_amdgcn_sched_barrier(0);
          add(j + kAhead, t1);
        }
      };
      Rec now, nxt;
      C2 vnext;
      load_batch(0, now);
      load_rec(kBatch, nxt);
      Batch cur = unpack(now);
      Raw c0[kVarGroup], c1[kVarGroup];
      if (__ballot(cur.support > 8u) == 0) fetch_group(std::integral_constant<int, 0>{}, cur, c0);
      for (uint32_t b = 0; b < n_rec; b += kBatch) {
        load_vis(nxt, vnext);
        const bool one_pass = __ballot(cur.support > 8u) == 0;
        if (one_pass) {
          fetch_group(std::integral_constant<int, 1>{}, cur, c1);
          __builtin_amdgcn_sched_barrier(0);
          add_group(std::integral_constant<int, 0>{}, cur, c0);
        } else if (__ballot(cur.support > 11u) == 0) {
          add_passes(std::integral_constant<int, 2>{}, now, n_rec - b);
        } else if (__ballot(cur.support > 16u) == 0) {
          add_passes(std::integral_constant<int, 4>{}, now, n_rec - b);
        } else {
#pragma unroll 1
          for (int j = 0; j < (int)min(kBatch, n_rec - b); ++j) {
            const uint32_t tp = bcast(now.tap, j);
            const int Sr = (int)(tp >> kTapBits) + 1, base = (int)(bcast(now.lds, j) & kLdsMask);
            const Real rwr = bcast(now.wr, j), rwi = bcast(now.wi, j);
            for (int t = lane; t < Sr * Sr; t += 64) {
              const int kv = t / Sr, ku = t - kv * Sr;
              accumulate(acc, base + kv * pitch + ku, rwr, rwi, tab_load(tab, (tp & kTapMask) + (uint32_t)t));
            }
          }
        }
        // the next batch's first taps load during this one's last group
        weigh(b + kBatch, nxt, vnext);
        now = nxt;
        Batch next = unpack(now);
        load_rec(b + 2 * kBatch, nxt);
        if (__ballot(next.support > 8u) == 0) fetch_group(std::integral_constant<int, 0>{}, next, c0);
        __builtin_amdgcn_sched_barrier(0);
        if (one_pass) add_group(std::integral_constant<int, 1>{}, cur, c1);
        cur = next;
      }
    } else if constexpr (kHasTap<Rec> && S == kLargeSupports) {
      // Large supports with FP32 arithmetic, taps loaded as they go: nothing held over records,
      // so that registers leave room for every wavefront whose tile copy LDS holds.
      Rec now, nxt, nxt2;
      C2 vnext;
      load_batch(0, now);
      load_rec(kBatch, nxt);
      for (uint32_t b = 0; b < n_rec; b += kBatch) {
        load_vis(nxt, vnext);
        load_rec(b + 2 * kBatch, nxt2);
#pragma unroll 1
        for (int j = 0; j < (int)min(kBatch, n_rec - b); ++j) {
          const uint32_t tp = bcast(now.tap, j);
          const int Sr = (int)(tp >> kTapBits) + 1, base = (int)(bcast(now.lds, j) & kLdsMask);
          const Real rwr = bcast(now.wr, j), rwi = bcast(now.wi, j);
          for (int t = lane; t < Sr * Sr; t += 64) {
            const int kv = t / Sr, ku = t - kv * Sr;
            accumulate(acc, base + kv * pitch + ku, rwr, rwi, tab_load(tab, (tp & kTapMask) + (uint32_t)t));
          }
        }
        weigh(b + kBatch, nxt, vnext);
        now = nxt;
        nxt = nxt2;
      }
    } else if constexpr (kHasTap<Rec>) {
      // General path (FP64; per-record support up to 32): records by wave-uniform loads,
      // each record's taps in passes of 64 lanes.
      for (uint32_t r = w.begin; r < w.end; ++r) {
        Rec rr = rec[r];
        if constexpr (PLANNED) to_weighted(rr, vis[get_row(rr)]);
        const uint32_t tp = rr.tap;
        const int Sr = S > 0 ? S : (int)(tp >> kTapBits) + 1;
        const uint32_t tb = tp & kTapMask;
        const int base = (int)(rr.lds & kLdsMask);
        for (int t = lane; t < Sr * Sr; t += 64) {
          const int kv = t / Sr, ku = t - kv * Sr;
          accumulate(acc, base + kv * pitch + ku, rr.wr, rr.wi, tab_load(tab, tb + t));
        }
      }
    }

    // flush: the work item's tile (with halo) goes to its own slot of the partial-tile
    // buffer with plain coalesced stores; tile_reduce_kernel adds the slots to the grid
    C2 *dst = partial + (size_t)item * rows * rows;
    for (int i = lane; i < rows * rows; i += 64) {
      const int ry = i / rows, rx = i - ry * rows;
      dst[i] = acc[ry * pitch + rx];
    }
  }
}

template <typename Real, typename Rec, typename Tab, int S, bool PLANNED, bool RUNS = false>
hipError_t launch_one(const wproj_kernels *k, const BinShape &B, const TileShape &ts,
                      const BinWorkspace &W, void *grid, const void *vis, hipStream_t s) {
  auto kern = tiled_grid_kernel<Real, Rec, Tab, S, PLANNED, RUNS>;
  // as many wavefronts per workgroup (up to 4) as their private tiles fit in LDS
  const int wpb = (int)std::max<size_t>(1, std::min<size_t>(kMaxWavesPerBlock, k->max_lds / ts.lds_bytes));
  const size_t lds = ts.lds_bytes * wpb;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * wpb, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipErrorInvalidConfiguration;
  const unsigned blocks = (unsigned)(k->n_cu * per_cu);
  const QueueRule &rule = S > 0 ? kFixedGridQueueRule : kGeneralGridQueueRule;
  const uint32_t n_queues = queue_count(k, rule, W, blocks, (int64_t)blocks * wpb);
  const int wave_lds = (int)(ts.lds_bytes / (2 * sizeof(Real)));
  // the paired fixed-support kernels read the pair-ordered table
  constexpr bool paired = S > 0 && kPairedTab<Tab>;
  if (paired && (!k->d_tab_pair || k->pair_stride != pair_stride(S))) return hipErrorInvalidValue;
  const int64_t n_sub = (int64_t)k->params.n_wplanes * k->params.oversample * k->params.oversample;
  const Tab *tab = (const Tab *)(paired ? k->d_tab_pair : k->d_tab);
  const int64_t tab_entries = paired ? n_sub * k->pair_stride : k->n_taps;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * wpb), lds, s, k->geo, B, ts.pitch,
                     ts.rows, wave_lds, tab, (uint32_t)(tab_entries * sizeof(Tab)),
                     (const Rec *)W.rec, W.items, W.order, W.choff + B.n_tiles, W.queues, n_queues, (typename Cx<Real>::T *)W.partial, (const typename Cx<Real>::T *)vis);
  return hipGetLastError();
}

template <typename Real, typename Rec, typename Tab, bool PLANNED, int S>
hipError_t dispatch_fixed(const wproj_kernels *k, const BinShape &B, const TileShape &ts,
                          const BinWorkspace &W, void *grid, const void *vis, hipStream_t s) {
  if constexpr (S > kMaxFixedSupport) {
    return hipErrorInvalidValue;  // pack_sub holds for kMinFixedSupport .. kMaxFixedSupport only
  } else {
    if (k->s_max == S) {
      if constexpr (kPairedTab<Tab>)
        if (k->params.accumulate_runs)
          return launch_one<Real, Rec, Tab, S, PLANNED, true>(k, B, ts, W, grid, vis, s);
      return launch_one<Real, Rec, Tab, S, PLANNED>(k, B, ts, W, grid, vis, s);
    }
    return dispatch_fixed<Real, Rec, Tab, PLANNED, S + 1>(k, B, ts, W, grid, vis, s);
  }
}

template <typename Real, typename Rec, typename Tab, bool PLANNED>
hipError_t dispatch_support(const wproj_kernels *k, const BinShape &B, const TileShape &ts,
                            const BinWorkspace &W, void *grid, const void *vis, hipStream_t s) {
  // a fixed support from kMinFixedSupport to kMaxFixedSupport has its own kernel, which
  // takes the sub-kernel from the packed LDS field (pack_sub is set exactly then);
  // per-plane supports take the general path
  if (B.pack_sub) {
    // FP32 W V records of a fixed support are the 12-byte packed form
    if constexpr (std::is_same_v<Rec, RecordF32> && !PLANNED)
      return dispatch_fixed<Real, RecordF32P, Tab, PLANNED, kMinFixedSupport>(k, B, ts, W, grid, vis, s);
    else
      return dispatch_fixed<Real, Rec, Tab, PLANNED, kMinFixedSupport>(k, B, ts, W, grid, vis, s);
  }
  // Supports above 16 alone over many rows: the kernel for mixed supports holds 188 registers with an
  // FP32 table (140 with FP16) and so 8 (12) wavefronts a CU, where LDS holds up to 16 copies of
  // 16-cell tiles.  Gridder call, mixed kernel and light one, S = 17, 16-cell tiles: 8.1e6 rows on
  // 2048^2 4.11 and 2.85 ms (FP16 2.61 and 2.31), on 4096^2 4.04 and 2.99, 4.0e6 on 2048^2 2.73 and
  // 1.90; S = 24 9.01 and 7.04; 32-cell tiles alike (4.0e6 rows 3.57 and 3.52).  Fewer rows go
  // either way (S = 17, 2.0e6 on 2048^2 1.25 and 1.25, with 8 planes 0.98 and 1.03; 1.0e6 on 512^2
  // 0.73 and 0.61, but S = 20 1.02 and 1.16).
  if constexpr (std::is_same_v<Real, float>)
    if (k->s_min > 16 && W.nvis > kManyLargeRows)
      return launch_one<Real, Rec, Tab, kLargeSupports, PLANNED>(k, B, ts, W, grid, vis, s);
  return launch_one<Real, Rec, Tab, 0, PLANNED>(k, B, ts, W, grid, vis, s);
}

template <typename Real, typename Rec, typename Tab>
hipError_t dispatch_planned(const wproj_kernels *k, const BinShape &B, const TileShape &ts,
                            const BinWorkspace &W, void *grid, const void *vis, hipStream_t s) {
  if (vis) return dispatch_support<Real, Rec, Tab, true>(k, B, ts, W, grid, vis, s);
  return dispatch_support<Real, Rec, Tab, false>(k, B, ts, W, grid, vis, s);
}

}  // namespace
}  // namespace wproj
