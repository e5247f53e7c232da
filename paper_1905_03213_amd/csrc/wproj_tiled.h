// Shapes and buffers of the binned (tiled) gridding path.
#pragma once

#include <type_traits>

#include "wproj_internal.h"

namespace wproj {

// Bits of Record::tap holding the first tap of the visibility's sub-kernel; the top
// bits hold S_p - 1.
constexpr int kTapBits = 26;
constexpr uint32_t kTapMask = (1u << kTapBits) - 1u;

// Bits of Record::lds holding the LDS offset; a tile copy has at most (64 + 31) x 104 =
// 9880 cells.  When BinShape::pack_sub is set, the bits above hold the sub-kernel number
// p O^2 + ov O + ou, so that with a uniform support S the first tap is that number times
// S^2 and the fixed-support gridders read one field instead of two.
constexpr int kLdsBits = 14;
constexpr uint32_t kLdsMask = (1u << kLdsBits) - 1u;
// Fixed supports with gridder kernels of their own.
constexpr int kMinFixedSupport = 3;
constexpr int kMaxFixedSupport = 16;

// Size classes of the largest-first work order (class c: items of more than
// (15 - c) / 16 of a chunk, down to the smallest).
constexpr int kOrderBuckets = 16;

// Work items are handed out largest first from kQueues queues, queue q holding items q, q + n,
// q + 2n, ... of that order: every worker (wavefront or workgroup) takes its next item with
// an atomic on its queue's head.  One head for all hands out only an item every 9 ns: 2.4 ms
// for the 2.6e5 tiles of 64 images of 1024^2 (16-cell tiles; 1.1 ms with 8, 16 or 32 heads,
// 1.14 with 128), and 0.42 ms instead of 0.28 for 1e7 rows on 16 layers of 2048^2.  Queues
// of their own for the small items, or a first item by the worker's number, measured slower
// (1.46 against 1.38 ms on 5.6e7 records), and so did workers that go on to another queue
// when theirs is empty (up to 50 us more, for the failed atomics of a launch's end).  Heads lie
// 128 bytes apart.
constexpr uint32_t kQueues = 16;
constexpr uint32_t kQueueStride = 32;
struct WorkQueue {
  uint32_t *head;
  uint32_t q, n_queues;  // n_queues <= workgroups, so that every queue is served
  __device__ WorkQueue(uint32_t *heads, uint32_t n) : q(blockIdx.x % n), n_queues(n) { head = heads + q * kQueueStride; }
  // one lane's call: the next item's place in the order (none is left when it is past the end)
  __device__ uint32_t next() { return atomicAdd(head, 1u) * n_queues + q; }
};
// With large sub-kernels one queue is better where its head is not busy: items are then handed
// out strictly in order, and items that run side by side share tables in the caches (16 queues
// drift apart).  Its cost is 9 ns for each item and each worker's last try, its gain a part of
// the time that the taps take, so the rule is the taps' bytes per take.  One queue's time over
// 16 queues', by kernel (least sub-kernel and bytes a take):
//   row-per-lane degridder  1536 B, 288 KB: FP64 S = 14 on 1024^2, 1.0e6 rows (420 KB) 0.97,
//     2048^2, 1.6e7 rows 0.97, 1.0e6 rows (170 KB) 1.01; S = 11 and 12, tile 32, 4.0e6 rows 0.95;
//     FP32 S = 16 0.98, on 64 images of 512^2 (118 KB) 0.99, S = 13 on 64 of 1024^2 (22 KB) 1.13;
//     smaller sub-kernels 1.00 to 1.1;
//   FP64 gridder            3072 B, 580 KB: S = 16 on 2048^2, 4.0e6 rows (790 KB) 0.92, 1.0e6
//     rows (210 KB) 1.14; S = 14 0.95 and 1.20; S = 12 1.01 at best, and no FP32 support gains;
//   general gridder         2048 B, 40 KB: FP64 S = 18 0.88 to 0.99, FP32 S = 20 0.92 to 0.98, but
//     1.03 and 1.08 for 2.1e4 rows on 1024^2 (19 and 12 KB).
// Per-plane supports count with their smallest, since most rows lie at small |w| (supports 4 to
// 16 on 2048^2, degridding a plan of 4.0e6 rows: FP32 392 us with one queue, 367 with 16).
struct QueueRule {
  int64_t tap_bytes, take_bytes;
};
constexpr QueueRule kDegridQueueRule{1536, 288 << 10}, kFixedGridQueueRule{3072, 580 << 10},
    kGeneralGridQueueRule{2048, 40 << 10};
struct BinWorkspace;
uint32_t queue_count(const wproj_kernels *k, const QueueRule &rule, const BinWorkspace &W, int64_t workgroups,
                     int64_t workers);

// Partial accumulators per image (weight sums) and per counter, spread by block index.
constexpr int kSlots = 256;

// One binned visibility: the LDS offset of its first cell inside its tile's private
// copy ((y0 - tile y0) pitch + (x0 - tile x0), optionally with the sub-kernel number
// above it), its sub-kernel (first tap | (S-1) << 26) and W V at the path's precision.
struct RecordF32 {
  uint32_t lds;
  uint32_t tap;
  float wr, wi;
};
struct RecordF64 {
  uint32_t lds;
  uint32_t tap;
  double wr, wi;
};
// The FP32 W V record of a fixed support whose sub-kernel number rides in `lds` (packed
// records): the first tap is that number times S^2, so no tap word is stored (12 bytes).
struct RecordF32P {
  uint32_t lds;
  float wr, wi;
};
template <typename Rec> constexpr bool kHasTap = !std::is_same_v<Rec, RecordF32P>;

// Row-carrying records (degridding and planned gridding) hold the visibility's weight in
// `wr` and its row in the low 32 bits of `wi` instead of W V.
__host__ __device__ inline void set_plan(RecordF32 &r, float w, uint32_t j) {
  r.wr = w;
  __builtin_memcpy(&r.wi, &j, 4);
}
__host__ __device__ inline void set_plan(RecordF64 &r, double w, uint32_t j) {
  r.wr = w;
  r.wi = 0.0;
  __builtin_memcpy(&r.wi, &j, 4);
}
__host__ __device__ inline uint32_t get_row(const RecordF32 &r) {
  uint32_t j;
  __builtin_memcpy(&j, &r.wi, 4);
  return j;
}
__host__ __device__ inline uint32_t get_row(const RecordF64 &r) {
  uint32_t j;
  __builtin_memcpy(&j, &r.wi, 4);
  return j;
}

// gfx9 buffer descriptor word 3: 32-bit data format, no swizzle
constexpr int kBufferWord3 = 0x00020000;

// Pair-ordered table (FP32 arithmetic).  The taps of a sub-kernel are cut into passes of 64;
// entries 2j and 2j + 1 of pass q are taps 64q + j and 64q + pair_half(S, q) + j.  One load
// brings two entries per lane, lanes 0-31 for the first record of a pair and lanes 32-63 for
// the second, so a pair of records costs one wide load instead of two narrow ones.  A swap
// of the upper half of the first entries with the lower half of the second entries
// (v_permlane32_swap, a VALU operation) then leaves every lane with one tap of both records.
constexpr int pair_passes(int S) { return (S * S + 63) / 64; }
constexpr int pair_taps(int S, int q) { return S * S - 64 * q < 64 ? S * S - 64 * q : 64; }
constexpr int pair_half(int S, int q) { return (pair_taps(S, q) + 1) / 2; }
// table entries per sub-kernel
constexpr int pair_stride(int S) { return 64 * (pair_passes(S) - 1) + 2 * pair_half(S, pair_passes(S) - 1); }

template <typename Tab> struct TapPair;
template <> struct TapPair<float2> {
  typedef uint32_t Raw __attribute__((ext_vector_type(4)));
  static constexpr uint32_t kTapBytes = 8;
  __device__ static Raw load(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0);
  }
  __device__ static void split(const Raw &v, float2 &first, float2 &second) {
    const uint32_t a_re = v[0], a_im = v[1], b_re = v[2], b_im = v[3];
    const auto re = __builtin_amdgcn_permlane32_swap(a_re, b_re, false, false);
    const auto im = __builtin_amdgcn_permlane32_swap(a_im, b_im, false, false);
    const uint32_t f_re = re[0], s_re = re[1], f_im = im[0], s_im = im[1];
    first = make_float2(__uint_as_float(f_re), __uint_as_float(f_im));
    second = make_float2(__uint_as_float(s_re), __uint_as_float(s_im));
  }
};
template <> struct TapPair<half2c> {
  typedef uint32_t Raw __attribute__((ext_vector_type(2)));
  static constexpr uint32_t kTapBytes = 4;
  __device__ static Raw load(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, 0);
  }
  __device__ static void split(const Raw &v, float2 &first, float2 &second) {
    const uint32_t a = v[0], b = v[1];
    const auto x = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    const uint32_t f = x[0], s = x[1];
    half2c hf, hs;
    __builtin_memcpy(&hf, &f, 4);
    __builtin_memcpy(&hs, &s, 4);
    first = make_float2((float)hf.re, (float)hf.im);
    second = make_float2((float)hs.re, (float)hs.im);
  }
};
template <typename Tab> constexpr bool kPairedTab = std::is_same_v<Tab, float2> || std::is_same_v<Tab, half2c>;

// Wave-uniform broadcast of lane j's value (v_readlane).
__device__ inline uint32_t bcast(uint32_t v, int j) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, j);
}
__device__ inline float bcast(float v, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
__device__ inline double bcast(double v, int j) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), j);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), j);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// A row-replicated register holds the same 16 values in each row of 16 lanes, so a DPP
// operand with row_newbcast:I reads value I in every lane: the multiply-add or address add
// that uses a record's field broadcasts it by itself, with no v_readlane before it.
// After the registers are replicated, dpp_ready covers the two wait states that a DPP read
// needs after a vector write (the assembler statements below hide the DPP read from the
// compiler's hazard handling; a CPU test looks for reads that come too early in the built
// kernels).  DPP reads nothing from a lane that is switched
// off, so these run with all 64 lanes on.
template <int I> __device__ inline uint32_t row_bcast(uint32_t v) {
  static_assert(I >= 0 && I < 16, "a row has 16 lanes");
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + I, 0xF, 0xF, true);
}
// s[I] + t, one instruction each (left to itself the compiler shares the broadcast of
// several sums in a register of its own, one instruction more)
template <int I> __device__ inline uint32_t add_bcast(uint32_t s, uint32_t t) {
  uint32_t d;
  asm("v_add_u32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(s), "v"(t), "n"(I));
  return d;
}
// d += s[I] t and d -= s[I] t, fused (one rounding), s row-replicated
template <int I> __device__ inline void fmac_bcast(float &d, float s, float t) {
  asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(t), "n"(I));
}
template <int I> __device__ inline void fmsc_bcast(float &d, float s, float t) {
  asm("v_fmac_f32_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(t), "n"(I));
}
template <int I> __device__ inline void fmac_bcast(double &d, double s, double t) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(t), "n"(I));
}
template <int I> __device__ inline void fmsc_bcast(double &d, double s, double t) {
  asm("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(t), "n"(I));
}
// v holds 32 values in each half wavefront (value i in lanes i and 32 + i): out[0] is
// values 0..15 and out[1] values 16..31, row-replicated.
__device__ inline void replicate16(uint32_t v, uint32_t (&out)[2]) {
  const auto h = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  out[0] = h[0];
  out[1] = h[1];
}
__device__ inline void replicate16(float v, float (&out)[2]) {
  uint32_t r[2];
  replicate16(__float_as_uint(v), r);
  out[0] = __uint_as_float(r[0]);
  out[1] = __uint_as_float(r[1]);
}
__device__ inline void replicate16(double v, double (&out)[2]) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  uint32_t lo[2], hi[2];
  replicate16((uint32_t)b, lo);
  replicate16((uint32_t)(b >> 32), hi);
  for (int g = 0; g < 2; ++g)
    out[g] = __longlong_as_double((long long)(((unsigned long long)hi[g] << 32) | lo[g]));
}

template <typename A, typename B, typename C, typename D>
__device__ inline void dpp_ready(A &a, B &b, C &c, D &d) {
  asm volatile("s_nop 1" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// f(std::integral_constant<int, 0>{}) ... f(std::integral_constant<int, N - 1>{}).
template <int I, int N, typename F> __device__ inline void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Complex cells at LDS byte addresses.
template <typename T> using LdsPtr = __attribute__((address_space(3))) T *;
typedef float Vec2f __attribute__((ext_vector_type(2)));
typedef double Vec2d __attribute__((ext_vector_type(2)));
__device__ inline uint32_t lds_address(void *p) { return (uint32_t)(uintptr_t)(LdsPtr<unsigned char>)(unsigned char *)p; }
__device__ inline void lds_read(uint32_t addr, float2 &v) {
  const Vec2f t = *(LdsPtr<Vec2f>)(uintptr_t)addr;
  v = make_float2(t.x, t.y);
}
__device__ inline void lds_read(uint32_t addr, double2 &v) {
  const Vec2d t = *(LdsPtr<Vec2d>)(uintptr_t)addr;
  v = make_double2(t.x, t.y);
}
__device__ inline void lds_write(uint32_t addr, const float2 &v) { *(LdsPtr<Vec2f>)(uintptr_t)addr = Vec2f{v.x, v.y}; }
__device__ inline void lds_write(uint32_t addr, const double2 &v) { *(LdsPtr<Vec2d>)(uintptr_t)addr = Vec2d{v.x, v.y}; }

// Binning geometry: tiles of `tile` cells, ntx x nty per image, kw keys per tile
// (n_wplanes when the plane is part of the key, else 1), 2^log2_rep counters per key.
struct BinShape {
  int tile;
  int log2_tile;     // tile = 1 << log2_tile
  int pitch;         // LDS row pitch (complex cells) of a tile's private copy
  int ntx, nty;
  int kw;
  int chunk;         // max records per work item
  int pack_sub;      // records carry the sub-kernel number in Record::lds (fixed support)
  int aggregate;     // the key pass aggregates counts per block in LDS (wproj_params::bin_aggregate)
  int stable;        // records keep input order inside a bin (wproj_params::stable_bins)
  int64_t n_tiles;   // n_images * ntx * nty
  int log2_rep;      // a key's visibilities are counted in 2^log2_rep counters, by the key pass's block
  int spread;        // neighbouring counters are stored on different cache lines (counter_place)
  uint32_t skew;     // spread: columns a row of counters is shifted by from the row before
  int64_t n_keys;    // n_tiles * kw
  int64_t n_counts;  // n_keys << log2_rep
};

// Words of a column of spread counters (counter_place).  (Columns of an odd number of cache
// lines, which fall on different memory channels, measured slower: 0.30 against 0.27 ms of
// binning for 4e6 rows on 1024^2.)
__host__ __device__ constexpr int64_t counter_column(int64_t n_counts) { return (n_counts + 255) / 256; }
// Words of the counter array.
constexpr int64_t counter_words(const BinShape &B) {
  return B.spread ? 256 * counter_column(B.n_counts) : B.n_counts;
}

struct WorkItem {
  uint32_t tile;   // img * (ntx * nty) + ty * ntx + tx
  uint32_t begin;  // record range
  uint32_t end;
};

// Workspace carve-up for one call (all device pointers).
struct BinWorkspace {
  uint32_t *slots;     // [3 nvis] (slot, key, record word) when pack_sub, else [4 nvis] (and tap word)
  void *rec;           // [nvis] RecordF32 / RecordF32P / RecordF64
  uint32_t *count;     // [counter_words]
  uint32_t *offset;    // [n_counts + 1]: a key's records start at offset[key << log2_rep]
  uint32_t *choff;     // [n_tiles + 1]; choff[n_tiles] = number of work items
  WorkItem *items;     // [max_items]
  uint32_t *scan_tmp;  // scan_temp_words of the scans, work_temp_words(n_tiles)
  uint32_t *queues;    // [kQueues * kQueueStride] heads of the work queues
  uint32_t *order;     // [max_items] work-item indices, largest items first
  uint32_t *order_cnt; // [2 * kOrderBuckets] per size class: item count, placement cursor
  int64_t nvis;        // rows of the call
  int64_t max_items;   // capacity of items, order and partial
  void *partial;       // [max_items][rows][rows] complex: each work item's accumulated tile
  // wslots, cslots, order_cnt and count follow each other and are cleared together at the start
  // of a binning (zero_words words before count)
  int64_t zero_words;
  double *wslots;      // [n_images][kSlots] partial weight sums
  unsigned long long *cslots;  // [3][kSlots] partial counters
  // stable binning only (null otherwise): radix-sort buffers
  uint32_t *sort_keys[2];  // [nvis] each: bin keys, ping-pong
  uint32_t *sort_vals[2];  // [nvis] each: visibility indices, ping-pong
  uint32_t *digit_count;   // [radix_digit_slots(nvis)] per-block digit counts, digit-major
  uint32_t *digit_off;     // [radix_digit_slots(nvis) + 1] their exclusive scan
};

// Entries of the per-block digit count array of the stable binning's radix sort.
int64_t radix_digit_slots(int64_t nvis);

int64_t scan_temp_words(int64_t n);
int64_t work_temp_words(int64_t n_tiles);  // block sums of the work list
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_exclusive_scan(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp,
                                 hipStream_t s);
// Bins visibilities for gridding (records carry W V) or, with vis == nullptr, into
// row-carrying records (weight and row: degridding, with wt == nullptr and weights taken
// as 1, and planned gridding).  zero_out (complex, nullable): rows that are not binned are
// set to 0 in it.
hipError_t launch_bin(const wproj_kernels *k, const BinShape &B, int64_t nvis, const double *uvw,
                      const void *vis, const void *wt, const int64_t *img_off, double *wsum,
                      int64_t *counters, const BinWorkspace &W, hipStream_t s, void *zero_out = nullptr);

// rows[i] = row of binned record i (row-carrying records), 0xffffffff past the last.
hipError_t launch_plan_rows(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W, int64_t nvis,
                            uint32_t *rows, hipStream_t s);

// LDS tile geometry of the tiled gridder for a handle.
struct TileShape {
  int tile;   // T
  int rows;   // T + S_max - 1
  int pitch;  // >= rows, padded for conflict-free rows of taps
  size_t lds_bytes;
};
TileShape tile_shape(const wproj_kernels *k, int tile);
// Row pitch (complex cells) of the degridder's tile copy when records are binned for
// degridding only: the smallest odd pitch >= T + S_max - 1.
int degrid_pitch(const wproj_kernels *k, int tile);
// Fills k->d_tab_pair from k->d_tab.
hipError_t launch_pair_table(const wproj_kernels *k, hipStream_t s);
// The tile gridder into the work items' partial tiles, then their sum into the grid.
// With vis != nullptr the records are row-carrying (a plan), W V is formed from vis and the
// queue heads are cleared here (a single call's binning clears them).
hipError_t launch_tiled_grid(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W,
                             void *grid, hipStream_t s, const void *vis = nullptr);
hipError_t launch_tiled_grid_f16(const wproj_kernels *k, const BinShape &B, const TileShape &ts, const BinWorkspace &W,
                                 void *grid, const void *vis, hipStream_t s);
hipError_t launch_tiled_grid_f64(const wproj_kernels *k, const BinShape &B, const TileShape &ts, const BinWorkspace &W,
                                 void *grid, const void *vis, hipStream_t s);
hipError_t launch_tile_reduce(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W,
                              void *grid, hipStream_t s);
// Whether launch_tiled_degrid takes the one-tap-per-lane degridder (FP32 arithmetic and
// tables, packed records of a fixed support up to 8, the pair-ordered table); its
// records are binned with the gridder's row pitch.
bool tap_lane_degrid(const wproj_kernels *k, const BinShape &B);
// planned: vis_out and the queue heads are cleared here; a single call's binning does both.
hipError_t launch_tiled_degrid(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W,
                               const void *model_grid, void *vis_out, int64_t nvis, bool planned, hipStream_t s);

// Rows regrouped by baseline (Eqs. 5 and 6): a stable counting sort over blocks of
// rows_per_block rows, n_keys = n_ant (n_ant + 1) / 2 baseline numbers + 1 for rows with
// an invalid antenna ID.
struct RegroupShape {
  uint32_t n_keys;
  int64_t rows_per_block;
  int64_t n_blocks;
  int64_t n_counts;  // n_keys * n_blocks
};
RegroupShape regroup_shape(int64_t n_rows, int32_t n_ant);
int64_t regroup_workspace_bytes(const RegroupShape &r);
hipError_t launch_regroup(const RegroupShape &r, int64_t n_rows, const int32_t *ant1,
                          const int32_t *ant2, int32_t n_ant, int64_t *perm, int64_t *start,
                          int64_t *counts, void *workspace, hipStream_t s);
hipError_t launch_channel_order(int64_t n_keys, int32_t n_chan, const int64_t *perm,
                                const int64_t *start, const int64_t *counts, int64_t *vis_perm,
                                hipStream_t s);
hipError_t launch_gather_rows(int64_t n_rows, int64_t row_bytes, const int64_t *perm,
                              int64_t n_src_rows, const void *src, void *dst, int64_t *bad,
                              hipStream_t s);

}  // namespace wproj
