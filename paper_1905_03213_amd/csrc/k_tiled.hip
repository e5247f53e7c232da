// Tiled gridder: FP32 tables, the partial-tile reduce, the pair-ordered table and the
// dispatch on precision (the gridder itself is in tiled_grid.h; one file per precision, so
// that they compile side by side).
#include "tiled_grid.h"

namespace wproj {
namespace {

// Adds the partial tiles to the grid.  A thread takes two cells of a column and sums, in
// FP64, every work item's partial value for each of them: the items of the cell's own tile
// and those of the tiles to its left/above whose halo reaches it (items of tile t are
// contiguous in the work list: [choff[t], choff[t + 1])).  Each cell has exactly one writer,
// so the grid update needs no atomics and the result does not depend on scheduling.
constexpr int kReduceAhead = 6;

template <typename Real>
__global__ void __launch_bounds__(256)
    tile_reduce_kernel(Geometry G, BinShape B, int rows, const typename Cx<Real>::T *__restrict__ partial,
                       const uint32_t *__restrict__ choff, Real *grid) {
  using C2 = typename Cx<Real>::T;
  // blockIdx.x * 256 + threadIdx.x is the column; a thread takes rows 2 blockIdx.y and
  // 2 blockIdx.y + 1 (one tile row, since tiles have an even side), whose work items and
  // their offsets it looks up once; blockIdx.z steps through the grids
  const int X = (int)(blockIdx.x * 256 + threadIdx.x), Y = 2 * (int)blockIdx.y;
  if (X >= G.n) return;
  const int64_t cells = (int64_t)G.n * G.n;
  const int T = B.tile;
  const int tx = X >> B.log2_tile, ty = Y >> B.log2_tile, lx = X & (T - 1), ly = Y & (T - 1);
  for (int img = (int)blockIdx.z; img < G.n_grids; img += (int)gridDim.z) {
    double sr0 = 0.0, si0 = 0.0, sr1 = 0.0, si1 = 0.0;
    for (int dy = 0; dy <= ty && ly + dy * T < rows; ++dy) {
      const bool second = ly + 1 + dy * T < rows;  // row Y + 1 is inside this tile's copy too
      for (int dx = 0; dx <= tx && lx + dx * T < rows; ++dx) {
        const int64_t tile = ((int64_t)img * B.nty + (ty - dy)) * B.ntx + (tx - dx);
        const int off = (ly + dy * T) * rows + (lx + dx * T);
        const uint32_t i1 = choff[tile + 1];
        uint32_t i = choff[tile];
        const int64_t stride = (int64_t)rows * rows;
        // kReduceAhead items' values load before the first is added: a tile of many items
        // otherwise waits for memory once an item (1024^2, 4e6 rows in items of 512: 144 us,
        // 64 with 4 ahead, 55 with 6, 51 with 8, 45 with 16, which costs tiles of one item
        // 40 % by its registers)
        for (; i + kReduceAhead <= i1; i += kReduceAhead) {
          const C2 *p = partial + (int64_t)i * stride + off;
          const int below = second ? rows : 0;
          C2 v0[kReduceAhead], v1[kReduceAhead];
#pragma unroll
          for (int k = 0; k < kReduceAhead; ++k) {
            v0[k] = p[k * stride];
            v1[k] = p[k * stride + below];
          }
#pragma unroll
          for (int k = 0; k < kReduceAhead; ++k) {
            sr0 += (double)v0[k].x;
            si0 += (double)v0[k].y;
            if (second) {
              sr1 += (double)v1[k].x;
              si1 += (double)v1[k].y;
            }
          }
        }
        for (; i < i1; ++i) {
          const C2 *p = partial + (int64_t)i * stride + off;
          const C2 v0 = p[0];
          sr0 += (double)v0.x;
          si0 += (double)v0.y;
          if (second) {
            const C2 v1 = p[rows];
            sr1 += (double)v1.x;
            si1 += (double)v1.y;
          }
        }
      }
    }
    C2 *g = reinterpret_cast<C2 *>(grid) + (cells * img + (int64_t)Y * G.n + X);
    if (sr0 != 0.0 || si0 != 0.0) {
      C2 v = g[0];
      v.x = (Real)((double)v.x + sr0);
      v.y = (Real)((double)v.y + si0);
      g[0] = v;
    }
    if (sr1 != 0.0 || si1 != 0.0) {
      C2 v = g[G.n];
      v.x = (Real)((double)v.x + sr1);
      v.y = (Real)((double)v.y + si1);
      g[G.n] = v;
    }
  }
}

template <typename Real>
hipError_t launch_reduce(const wproj_kernels *k, const BinShape &B, const TileShape &ts,
                         const BinWorkspace &W, void *grid, hipStream_t s) {
  const dim3 grid3((unsigned)((k->params.n + 255) / 256), (unsigned)(k->params.n / 2),
                   (unsigned)std::min<int64_t>(k->geo.n_grids, 65535));
  hipLaunchKernelGGL(tile_reduce_kernel<Real>, grid3, dim3(256), 0,
                     s, k->geo, B, ts.rows, (const typename Cx<Real>::T *)W.partial, W.choff,
                     (Real *)grid);
  return hipGetLastError();
}

// Fills the pair-ordered table: one thread per entry.  Entry 2j of pass q is tap 64q + j and
// entry 2j + 1 tap 64q + h + j, h = pair_half(S, q), or zero where that tap does not exist.
template <typename Tab>
__global__ void __launch_bounds__(256)
    pair_table_kernel(const Tab *__restrict__ src, int64_t n_sub, int S, int stride, Tab *__restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_sub * stride) return;
  const int64_t sub = i / stride;
  const int e = (int)(i - sub * stride);
  const int q = e / 64, jj = (e - 64 * q) >> 1;
  const int n_q = pair_taps(S, q), h = pair_half(S, q);
  const bool second = e & 1;
  Tab v{};
  if (second ? jj < n_q - h : jj < h) v = src[sub * S * S + 64 * q + (second ? h : 0) + jj];
  dst[i] = v;
}

}  // namespace

hipError_t launch_pair_table(const wproj_kernels *k, hipStream_t s) {
  const int S = k->s_max;
  const int64_t n_sub = (int64_t)k->params.n_wplanes * k->params.oversample * k->params.oversample;
  const int64_t total = n_sub * k->pair_stride;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (k->params.precision == WPROJ_F32)
    hipLaunchKernelGGL(pair_table_kernel<float2>, dim3(blocks), dim3(256), 0, s, (const float2 *)k->d_tab,
                       n_sub, S, (int)k->pair_stride, (float2 *)k->d_tab_pair);
  else
    hipLaunchKernelGGL(pair_table_kernel<half2c>, dim3(blocks), dim3(256), 0, s, (const half2c *)k->d_tab,
                       n_sub, S, (int)k->pair_stride, (half2c *)k->d_tab_pair);
  return hipGetLastError();
}

TileShape tile_shape(const wproj_kernels *k, int tile) {
  // One wavefront's private tile: rows = T + S_max - 1 complex cells per side.  The row
  // pitch (in complex cells) is odd-multiple-of-8 so that the 4 rows of 8 taps a half
  // wavefront touches fall on different LDS banks for 64-bit accesses.
  TileShape t;
  t.tile = tile;
  t.rows = tile + k->s_max - 1;
  int pitch = t.rows;
  while ((pitch & 15) != 8) ++pitch;
  t.pitch = pitch;
  const size_t real = k->params.precision == WPROJ_F64 ? 8 : 4;
  t.lds_bytes = 2 * (size_t)t.rows * t.pitch * real;  // per wavefront
  return t;
}

uint32_t queue_count(const wproj_kernels *k, const QueueRule &rule, const BinWorkspace &W, int64_t workgroups,
                     int64_t workers) {
  const int64_t taps = (int64_t)k->s_min * k->s_min * (int64_t)k->tap_bytes;
  const int64_t takes = W.max_items + workers;
  if (taps >= rule.tap_bytes && W.nvis * taps >= takes * rule.take_bytes) return 1;
  return (uint32_t)std::min<int64_t>(kQueues, workgroups);
}

int degrid_pitch(const wproj_kernels *k, int tile) { return (tile + k->s_max - 1) | 1; }

hipError_t launch_tiled_grid(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W,
                             void *grid, hipStream_t s, const void *vis) {
  const TileShape ts = tile_shape(k, B.tile);
  if (vis) {
    const hipError_t e = launch_fill_u32(W.queues, kQueues * kQueueStride, 0u, s);
    if (e != hipSuccess) return e;
  }
  switch (k->params.precision) {
    case WPROJ_F64:
      return launch_tiled_grid_f64(k, B, ts, W, grid, vis, s);
    case WPROJ_F32:
      return dispatch_planned<float, RecordF32, float2>(k, B, ts, W, grid, vis, s);
    default:
      return launch_tiled_grid_f16(k, B, ts, W, grid, vis, s);
  }
}

hipError_t launch_tile_reduce(const wproj_kernels *k, const BinShape &B, const BinWorkspace &W,
                              void *grid, hipStream_t s) {
  const TileShape ts = tile_shape(k, B.tile);
  if (k->params.precision == WPROJ_F64) return launch_reduce<double>(k, B, ts, W, grid, s);
  return launch_reduce<float>(k, B, ts, W, grid, s);
}

}  // namespace wproj
