// The image transforms for grid sides that are powers of two from 128 to 4096: 2D transforms
// in two passes over memory, with what surrounds them (the Hermitian part, the grid
// correction, the sum over w-stacking layers) done in the same passes.  Other sides, and few
// small w-stacking layers (own_fft), go through rocFFT (api.hip).
//
// Bound by HBM: each pass reads and writes the data once, where rocFFT's passes and those of
// the Hermitian part and the correction around them are five or more.  Transform and
// correction together, rocFFT's way and here: 64 FP32 images of 1024^2 745 and 277 us (1.34 GB
// in two passes, 4.9 TB/s; the column pass asks for the half spectrum E twice, the second time
// served by the caches); one of 2048^2 74 and 33 us in FP32, 96 and 47 us in FP64; FP64
// image -> grid of 2048^2 120 and 50 us; FP32 4096^2 201 and 111 us; FP64 256^2 23 and 15 us;
// 16 FP32 w-stacking layers of 2048^2 984 and 384 us.
//
// grid -> image is Re IDFT(G).  Row pass: rows ky and -ky of G are transformed along x by the
// same threads and combined to E[ky][x] = F[ky][x] + conj(F[-ky][x]), ky = 0 .. n/2, whose
// transform along y is real; half the data.  Column pass: two neighbouring columns E1, E2 go
// through one complex transform as E1 + i E2 (the rows beyond n/2 are conjugates of the
// others), which leaves one real column in each part; the correction is applied on the way
// out.  image -> grid runs backwards: two real rows per complex transform, columns
// 0 .. n/2 transformed, and the other columns of the grid written as their conjugates.  In
// FP64 only: chi^2 of FP32 predictions, an FP64 sum, shows a transform's rounding (1.2e-7 off
// either way, 1e-8 apart), and stays as it was.
//
// A sequence of N values is transformed by N/16 threads, 16 values each, in two or three
// Stockham passes of radix 16 or 8 (thread t holds values t + q N/16, q = 0..15, at both
// ends), exchanged through LDS a component at a time, which halves the LDS a sequence takes.
// Twiddle factors come from a table laid out pass by pass as the threads read it, computed
// in double precision.
#include <math.h>

#include <algorithm>
#include <vector>

#include "wproj_internal.h"

namespace wproj {
namespace {

template <typename Real> struct CplxOf;
template <> struct CplxOf<float> { using T = float2; };
template <> struct CplxOf<double> { using T = double2; };
// Two image pixels, stored at once: the image is aligned to one.
template <typename Real> struct Pair { Real v[2]; };

constexpr int radix_of(int n, int p) {
  return n == 512 ? 8 : p == 0 ? 16 : n == 128 || n == 1024 || (n == 2048 && p == 2) ? 8 : 16;
}
constexpr int passes_of(int n) { return n <= 256 ? 2 : 3; }

// Entries of the twiddle table: pass p (after Ns values are combined, radix R) holds
// exp(-2 pi i k j / (Ns R)) at k Ns + j, j < Ns, k < R; the first pass needs none.
constexpr int twiddle_base(int n, int p) {
  int base = 0, ns = radix_of(n, 0);
  for (int q = 1; q < p; ++q) {
    base += ns * radix_of(n, q);
    ns *= radix_of(n, q);
  }
  return base;
}

template <int SIGN, typename C2> __device__ inline C2 mul(const C2 &a, const C2 &w) {  // a w or a conj(w)
  C2 r;
  if constexpr (SIGN < 0) {
    r.x = a.x * w.x - a.y * w.y;
    r.y = a.x * w.y + a.y * w.x;
  } else {
    r.x = a.x * w.x + a.y * w.y;
    r.y = a.y * w.x - a.x * w.y;
  }
  return r;
}
template <typename C2> __device__ inline C2 add(const C2 &a, const C2 &b) {
  C2 r;
  r.x = a.x + b.x;
  r.y = a.y + b.y;
  return r;
}
template <typename C2> __device__ inline C2 sub(const C2 &a, const C2 &b) {
  C2 r;
  r.x = a.x - b.x;
  r.y = a.y - b.y;
  return r;
}
template <int SIGN, typename C2> __device__ inline C2 turn(const C2 &a) {  // a exp(SIGN pi i / 2)
  C2 r;
  r.x = SIGN < 0 ? a.y : -a.y;
  r.y = SIGN < 0 ? -a.x : a.x;
  return r;
}

template <int SIGN, typename C2> __device__ inline void dft4(C2 &a, C2 &b, C2 &c, C2 &d) {
  const C2 s = add(a, c), t = sub(a, c), u = add(b, d), v = turn<SIGN>(sub(b, d));
  a = add(s, u);
  b = add(t, v);
  c = sub(s, u);
  d = sub(t, v);
}

// DFT of 8 or 16 values in place, in natural order.
template <int R, int SIGN, typename C2> __device__ inline void dft(C2 *x) {
  using Real = decltype(x->x);
  constexpr double kCos16[16] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
                                 0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
                                 -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173,
                                 0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613};
  constexpr int M = R / 4;  // inner sums over x[M n1 + n2]
  C2 y[R];
#pragma unroll
  for (int n2 = 0; n2 < M; ++n2) {
    C2 a = x[n2], b = x[M + n2], c = x[2 * M + n2], d = x[3 * M + n2];
    dft4<SIGN>(a, b, c, d);
    y[n2] = a;
    y[M + n2] = b;
    y[2 * M + n2] = c;
    y[3 * M + n2] = d;
  }
#pragma unroll
  for (int k1 = 1; k1 < 4; ++k1)
#pragma unroll
    for (int n2 = 1; n2 < M; ++n2) {
      const int e = (k1 * n2 * (16 / R)) & 15;  // exp(-2 pi i e / 16)
      C2 w;
      w.x = (Real)kCos16[e];
      w.y = (Real)kCos16[(e + 4) & 15];  // -sin
      y[k1 * M + n2] = mul<SIGN>(y[k1 * M + n2], w);
    }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    if constexpr (M == 4) {
      dft4<SIGN>(y[4 * k1], y[4 * k1 + 1], y[4 * k1 + 2], y[4 * k1 + 3]);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) x[k1 + 4 * k2] = y[4 * k1 + k2];
    } else {
      x[k1] = add(y[2 * k1], y[2 * k1 + 1]);
      x[k1 + 4] = sub(y[2 * k1], y[2 * k1 + 1]);
    }
  }
}

// Place of value i of a sequence in its LDS buffer (padded against bank conflicts) and the
// words a sequence takes (8 mod 64 apart, so that neighbouring sequences use other banks).
__device__ inline int lds_at(int i) { return i + (i >> 4); }
constexpr int seq_words(int n) { return (n + n / 16) / 64 * 64 + ((n + n / 16) % 64 ? 64 : 0) + 8; }

// Value q of a thread's 16 stands at v[(q % M) R + q / M] of a pass of radix R, M = 16/R.
template <int R> __device__ constexpr int reg_of(int q) { return (q % (16 / R)) * R + q / (16 / R); }

// DFT of one sequence (sign SIGN) held 16 values a thread: on entry v[reg_of<first radix>(q)]
// = value t + q N/16, on return v[reg_of<last radix>(q)] = value t + q N/16 of the transform.
// seq: the sequence's LDS buffer; every thread of the workgroup calls this together.
template <int N, int SIGN, typename Real, typename C2>
__device__ inline void fft_sequence(C2 (&v)[16], int t, Real *seq, const C2 *__restrict__ tw) {
  constexpr int TN = N / 16;
  auto pass = [&](auto pass_no) {
    constexpr int p = decltype(pass_no)::value, R = radix_of(N, p), M = 16 / R;
    constexpr int Ns = p == 0 ? 1 : p == 1 ? radix_of(N, 0) : radix_of(N, 0) * radix_of(N, 1);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = t + m * TN;
      if constexpr (p > 0) {
        const C2 *w = tw + twiddle_base(N, p) + (j & (Ns - 1));
#pragma unroll
        for (int k = 1; k < R; ++k) v[m * R + k] = mul<SIGN>(v[m * R + k], w[k * Ns]);
      }
      dft<R, SIGN>(&v[m * R]);
    }
    if constexpr (p + 1 < passes_of(N)) {
      constexpr int R2 = radix_of(N, p + 1);
      auto exchange = [&](auto part) {
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int j = t + m * TN;
          const int at = (j / Ns) * (Ns * R) + (j & (Ns - 1));
#pragma unroll
          for (int k = 0; k < R; ++k) seq[lds_at(at + k * Ns)] = decltype(part)::value ? v[m * R + k].y : v[m * R + k].x;
        }
        __syncthreads();
      };
      Real re[16];
      exchange(std::integral_constant<int, 0>{});
#pragma unroll
      for (int q = 0; q < 16; ++q) re[reg_of<R2>(q)] = seq[lds_at(t + q * TN)];
      exchange(std::integral_constant<int, 1>{});
#pragma unroll
      for (int q = 0; q < 16; ++q) v[reg_of<R2>(q)].y = seq[lds_at(t + q * TN)];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q].x = re[q];
    }
  };
  pass(std::integral_constant<int, 0>{});
  pass(std::integral_constant<int, 1>{});
  if constexpr (passes_of(N) == 3) pass(std::integral_constant<int, 2>{});
}

template <int N> constexpr int kFirst = radix_of(N, 0);
template <int N> constexpr int kLast = radix_of(N, passes_of(N) - 1);

constexpr int kColThreads = 512;
constexpr int kMaxGridY = 65535;

// Sequences per workgroup.  Rows: 256 threads, one wavefront for the sides that give few
// workgroups.  Columns: 16 where 64 KiB of LDS hold them, at most kColThreads threads.
template <int N> constexpr int kRowSeqs = N >= 4096 ? 1 : N >= 512 ? 4096 / N : 1024 / N;
constexpr int col_seqs(int n, int real_bytes) {
  int c = 16;
  while (c > 1 && (c * (n / 16) > kColThreads || c * seq_words(n) * real_bytes > 65536)) c /= 2;
  return c;
}
template <typename Real, int N> constexpr int kCols = col_seqs(N, sizeof(Real));

// The group of columns a workgroup takes.  Workgroups go to the 8 XCDs in turn; neighbouring
// columns, which share lines of memory, go to one XCD and its L2 (4096^2 in FP32, whose groups
// are 32 bytes wide: both passes 179 us in launch order, 110 so; 2048^2 FP64 59 and 47 us).
__device__ inline int column_group() {
  const unsigned b = blockIdx.x, g = gridDim.x / 8;
  return (int)(b < 8 * g ? (b % 8) * g + b / 8 : b);
}

// ---- grid -> image (no w-stacking) ----

template <typename Real, int N>
__global__ void __launch_bounds__((kRowSeqs<N> * (N / 16)))
    g2i_rows_kernel(const typename CplxOf<Real>::T *__restrict__ G, typename CplxOf<Real>::T *__restrict__ E,
                    const typename CplxOf<Real>::T *__restrict__ tw) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16;
  __shared__ Real lds[kRowSeqs<N> * seq_words(N)];
  const int t = threadIdx.x % TN, s = threadIdx.x / TN;
  Real *seq = lds + s * seq_words(N);
  const int ky = (int)blockIdx.x * kRowSeqs<N> + s;
  const bool on = ky <= N / 2;
  const int row = on ? ky : 0, mirror = row == 0 ? 0 : N - row;
  const C2 *g = G + (int64_t)blockIdx.y * N * N;
  C2 a[16], b[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) a[reg_of<kFirst<N>>(q)] = g[(int64_t)row * N + t + q * TN];
#pragma unroll
  for (int q = 0; q < 16; ++q) b[reg_of<kFirst<N>>(q)] = g[(int64_t)mirror * N + t + q * TN];
  fft_sequence<N, 1>(a, t, seq, tw);
  fft_sequence<N, 1>(b, t, seq, tw);
  if (!on) return;
  C2 *e = E + ((int64_t)blockIdx.y * (N / 2 + 1) + ky) * N;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const C2 x = a[reg_of<kLast<N>>(q)], y = b[reg_of<kLast<N>>(q)];
    C2 r;
    r.x = x.x + y.x;
    r.y = x.y - y.y;
    e[t + q * TN] = r;
  }
}

template <typename Real, int N>
__global__ void __launch_bounds__((kCols<Real, N> * (N / 16)))
    g2i_cols_kernel(const typename CplxOf<Real>::T *__restrict__ E, const typename CplxOf<Real>::T *__restrict__ tw,
                    const double *__restrict__ kappa, const double *__restrict__ wsum, Real *__restrict__ img) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16, C = kCols<Real, N>;
  __shared__ Real lds[C * seq_words(N)];
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int xs = 2 * (column_group() * C + c);  // columns xs and xs + 1
  const C2 *e = E + (int64_t)blockIdx.y * (N / 2 + 1) * N + xs;
  C2 v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int ky = t + q * TN;
    const bool upper = ky > N / 2;
    const C2 *p = e + (int64_t)(upper ? N - ky : ky) * N;
    C2 a = p[0], b = p[1];
    if (upper) {
      a.y = -a.y;
      b.y = -b.y;
    }
    C2 z;
    z.x = a.x - b.y;
    z.y = a.y + b.x;
    v[reg_of<kFirst<N>>(q)] = z;
  }
  fft_sequence<N, 1>(v, t, lds + c * seq_words(N), tw);
  double scale = 0.5;  // E holds twice the Hermitian part
  if (wsum != nullptr) {
    const double s = wsum[blockIdx.y];
    scale = s != 0.0 ? scale / s : 0.0;
  }
  const int x = xs + N / 2 < N ? xs + N / 2 : xs - N / 2;
  const double k0 = kappa[x] * scale, k1 = kappa[x + 1] * scale;
  Real *out = img + (int64_t)blockIdx.y * N * N + x;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int ys = t + q * TN, y = ys + N / 2 < N ? ys + N / 2 : ys - N / 2;
    const C2 r = v[reg_of<kLast<N>>(q)];
    const double ky = (y & 1) ? -kappa[y] : kappa[y];  // the sign (-1)^(x + y); x is even
    Pair<Real> o;
    o.v[0] = (Real)((double)r.x * (ky * k0));
    o.v[1] = (Real)(-(double)r.y * (ky * k1));
    *reinterpret_cast<Pair<Real> *>(out + (int64_t)y * N) = o;
  }
}

// ---- grids -> image with w-stacking ----

// The layers' centres are symmetric about w = 0 (layer L - 1 - l is the mirror of l), so for
// real images the partner's phase is the conjugate, and Re(F_l e^(i phi) + F_l' e^(-i phi)) =
// Re((F_l + conj F_l') e^(i phi)): one column transform and one phase for two layers.  Row pass:
// E_l[ky] = F_l[ky] + conj(F_l'[-ky]) over row ky of layer l < L/2, which only the threads that
// write it read.  A middle layer is its own partner; its rows ky and -ky are done together.
// (16 layers of 2048^2: 187 us for 0.8 GB, the rate of a copy.)
template <typename Real, int N>
__global__ void __launch_bounds__((kRowSeqs<N> * (N / 16)))
    stack_rows_kernel(int n_layers, typename CplxOf<Real>::T *__restrict__ G,
                      const typename CplxOf<Real>::T *__restrict__ tw) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16;
  __shared__ Real lds[kRowSeqs<N> * seq_words(N)];
  const int t = threadIdx.x % TN, s = threadIdx.x / TN;
  Real *seq = lds + s * seq_words(N);
  const int half = (n_layers + 1) / 2, l = (int)blockIdx.y % half, partner = n_layers - 1 - l;
  const int ky = (int)blockIdx.x * kRowSeqs<N> + s, mirror = (N - ky) & (N - 1);
  const bool on = l != partner || ky <= N / 2;
  C2 *g = G + (int64_t)(blockIdx.y / half) * n_layers * N * N;
  C2 *ga = g + ((int64_t)l * N + ky) * N, *gb = g + ((int64_t)partner * N + mirror) * N;
  C2 a[16] = {}, b[16] = {};
  if (on) {
#pragma unroll
    for (int q = 0; q < 16; ++q) a[reg_of<kFirst<N>>(q)] = ga[t + q * TN];
#pragma unroll
    for (int q = 0; q < 16; ++q) b[reg_of<kFirst<N>>(q)] = gb[t + q * TN];
  }
  fft_sequence<N, 1>(a, t, seq, tw);
  fft_sequence<N, 1>(b, t, seq, tw);
  if (!on) return;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const C2 x = a[reg_of<kLast<N>>(q)], y = b[reg_of<kLast<N>>(q)];
    C2 r;
    r.x = x.x + y.x;
    r.y = x.y - y.y;
    ga[t + q * TN] = r;
    r.y = -r.y;
    if (l == partner && mirror != ky) gb[t + q * TN] = r;
  }
}

// Columns of an image's combined layers along y, one after the other: the image is
// Re(sum over l of E_l exp(+2 pi i w_l (n - 1))) kappa kappa / sumW, so nothing but the image
// is written.  Bound by the phases' FP64 sines and by its barriers (8 combined layers of
// 2048^2: 207 us, memory alone 50); held to 128 registers, for twice the wavefronts, it spills
// and takes as long.
template <typename Real, int N>
__global__ void __launch_bounds__((kCols<Real, N> * (N / 16)))
    g2i_stack_cols_kernel(Geometry geo, const typename CplxOf<Real>::T *__restrict__ E,
                          const typename CplxOf<Real>::T *__restrict__ tw, const double *__restrict__ kappa,
                          const double *__restrict__ wsum, Real *__restrict__ img) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16, C = kCols<Real, N>;
  __shared__ Real lds[C * seq_words(N)];
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int xs = column_group() * C + c, x = xs + N / 2 < N ? xs + N / 2 : xs - N / 2;
  const int L = geo.n_layers;
  const uint32_t at = (uint32_t)(t * N + xs);
  double acc[16], nm1[16];
  bool inside[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int ys = t + q * TN, y = ys + N / 2 < N ? ys + N / 2 : ys - N / 2;
    acc[q] = nm1[q] = 0.0;
    inside[q] = n_minus_1(geo, x, y, nm1[q]);
  }
  for (int l = 0; l < (L + 1) / 2; ++l) {
    const C2 *e = E + ((int64_t)blockIdx.y * L + l) * N * N;
    C2 v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[reg_of<kFirst<N>>(q)] = (e + (int64_t)q * TN * N)[at];
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(tw));  // else all twiddle factors are kept in registers over the loop
#endif
    fft_sequence<N, 1>(v, t, lds + c * seq_words(N), tw);
    const bool middle = l == L - 1 - l;
    const double wl = middle ? 0.0 : 2.0 * layer_centre(geo, l), weight = middle ? 0.5 : 1.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const C2 r = v[reg_of<kLast<N>>(q)];
      double sn, cs;
      sincospi(wl * nm1[q], &sn, &cs);
      acc[q] += weight * ((double)r.x * cs - (double)r.y * sn);
      __builtin_amdgcn_sched_barrier(0);  // one phase at a time, or the registers don't hold
    }
  }
  double scale = kappa[x];
  if (wsum != nullptr) {
    const double s = wsum[blockIdx.y];
    scale = s != 0.0 ? scale / s : 0.0;
  }
  Real *out = img + (int64_t)blockIdx.y * N * N + x;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int ys = t + q * TN, y = ys + N / 2 < N ? ys + N / 2 : ys - N / 2;
    const double v = ((x + y) & 1) ? -acc[q] : acc[q];
    out[(int64_t)y * N] = inside[q] ? (Real)(v * (kappa[y] * scale)) : (Real)0;
  }
}

// ---- image -> grid (no w-stacking) ----

// Rows y1 = 2 s and y1 + 1 of the corrected, shifted, sign-flipped image as one complex
// sequence; H[row][kx], kx = 0 .. N/2, in rows of N/2 + 1.
template <typename Real, int N>
__global__ void __launch_bounds__((kRowSeqs<N> * (N / 16)))
    i2g_rows_kernel(const Real *__restrict__ img, const double *__restrict__ kappa,
                    const typename CplxOf<Real>::T *__restrict__ tw, typename CplxOf<Real>::T *__restrict__ H) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16;
  __shared__ Real lds[kRowSeqs<N> * seq_words(N)];
  const int t = threadIdx.x % TN, s = threadIdx.x / TN;
  Real *seq = lds + s * seq_words(N);
  const int r0 = 2 * ((int)blockIdx.x * kRowSeqs<N> + s);  // shifted rows r0, r0 + 1
  const int y = r0 + N / 2 < N ? r0 + N / 2 : r0 - N / 2;
  const Real *p = img + ((int64_t)blockIdx.y * N + y) * N;
  const double k0 = kappa[y], k1 = kappa[y + 1];
  C2 v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int xs = t + q * TN, x = xs + N / 2 < N ? xs + N / 2 : xs - N / 2;
    const double kx = (xs & 1) ? -kappa[x] : kappa[x];  // (-1)^(xs + row); r0 is even
    C2 z;
    z.x = (Real)((double)p[x] * (kx * k0));
    z.y = (Real)(-(double)p[N + x] * (kx * k1));
    v[reg_of<kFirst<N>>(q)] = z;
  }
  fft_sequence<N, -1>(v, t, seq, tw);
  // Z[k] and Z[-k] give the two rows: F1 = (Z[k] + conj Z[-k]) / 2, F2 = (Z[k] - conj Z[-k]) / 2i
  C2 m[16];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) seq[lds_at(t + q * TN)] = v[reg_of<kLast<N>>(q)].x;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) m[q].x = seq[lds_at((N - (t + q * TN)) & (N - 1))];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) seq[lds_at(t + q * TN)] = v[reg_of<kLast<N>>(q)].y;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) m[q].y = seq[lds_at((N - (t + q * TN)) & (N - 1))];
  C2 *h = H + ((int64_t)blockIdx.y * N + r0) * (N / 2 + 1);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int kx = t + q * TN;
    if (kx > N / 2) continue;
    const C2 z = v[reg_of<kLast<N>>(q)];
    C2 f1, f2;
    f1.x = Real(0.5) * (z.x + m[q].x);
    f1.y = Real(0.5) * (z.y - m[q].y);
    f2.x = Real(0.5) * (z.y + m[q].y);
    f2.y = Real(0.5) * (m[q].x - z.x);
    h[kx] = f1;
    h[N / 2 + 1 + kx] = f2;
  }
}

template <typename Real, int N>
__global__ void __launch_bounds__((kCols<Real, N> * (N / 16)))
    i2g_cols_kernel(const typename CplxOf<Real>::T *__restrict__ H, const typename CplxOf<Real>::T *__restrict__ tw,
                    typename CplxOf<Real>::T *__restrict__ G) {
  using C2 = typename CplxOf<Real>::T;
  constexpr int TN = N / 16, C = kCols<Real, N>;
  __shared__ Real lds[C * seq_words(N)];
  const int c = threadIdx.x % C, t = threadIdx.x / C;
  const int kx = column_group() * C + c;
  const bool on = kx <= N / 2;
  const C2 *h = H + (int64_t)blockIdx.y * N * (N / 2 + 1) + (on ? kx : 0);
  C2 v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) v[reg_of<kFirst<N>>(q)] = h[(int64_t)(t + q * TN) * (N / 2 + 1)];
  fft_sequence<N, -1>(v, t, lds + c * seq_words(N), tw);
  if (!on) return;
  C2 *g = G + (int64_t)blockIdx.y * N * N;
  const bool mirrored = kx > 0 && kx < N / 2;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int ky = t + q * TN;
    C2 z = v[reg_of<kLast<N>>(q)];
    g[(int64_t)ky * N + kx] = z;
    z.y = -z.y;
    if (mirrored) g[(int64_t)((N - ky) & (N - 1)) * N + N - kx] = z;
  }
}

template <typename Real, int N>
hipError_t g2i(const wproj_kernels *k, void *grid, void *half, void *image, const double *wsum, hipStream_t s) {
  using C2 = typename CplxOf<Real>::T;
  const C2 *tw = (const C2 *)k->d_twiddle;
  constexpr int C = kCols<Real, N>;
  const dim3 row_block(kRowSeqs<N> * (N / 16)), col_block(C * (N / 16));
  for (int i = 0; i < k->geo.n_images; i += kMaxGridY) {
    const unsigned m = (unsigned)std::min(kMaxGridY, k->geo.n_images - i);
    const double *ws = wsum ? wsum + i : nullptr;
    Real *img = (Real *)image + (int64_t)i * N * N;
    if (k->params.w_mode == WPROJ_W_STACK) {
      const int L = k->geo.n_layers;
      C2 *g = (C2 *)grid + (int64_t)i * L * N * N;
      const int half = (L + 1) / 2, step = kMaxGridY / half;  // images per launch
      for (int j = 0; j < (int)m; j += step)
        hipLaunchKernelGGL((stack_rows_kernel<Real, N>),
                           dim3(N / kRowSeqs<N>, (unsigned)(half * std::min(step, (int)m - j))), row_block, 0, s, L,
                           g + (int64_t)j * L * N * N, tw);
      hipLaunchKernelGGL((g2i_stack_cols_kernel<Real, N>), dim3(N / C, m), col_block, 0, s, k->geo, g, tw, k->d_kappa,
                         ws, img);
    } else {
      C2 *e = (C2 *)half + (int64_t)i * N * (N / 2 + 1);
      hipLaunchKernelGGL((g2i_rows_kernel<Real, N>), dim3((N / 2 + kRowSeqs<N>) / kRowSeqs<N>, m), row_block, 0, s,
                         (const C2 *)grid + (int64_t)i * N * N, e, tw);
      hipLaunchKernelGGL((g2i_cols_kernel<Real, N>), dim3(N / 2 / C, m), col_block, 0, s, e, tw, k->d_kappa, ws, img);
    }
  }
  return hipGetLastError();
}

template <typename Real, int N>
hipError_t i2g(const wproj_kernels *k, const void *image, void *half, void *grid, hipStream_t s) {
  using C2 = typename CplxOf<Real>::T;
  const C2 *tw = (const C2 *)k->d_twiddle;
  constexpr int C = kCols<Real, N>;
  constexpr int pairs = N / 2;
  for (int i = 0; i < k->geo.n_images; i += kMaxGridY) {
    const unsigned m = (unsigned)std::min(kMaxGridY, k->geo.n_images - i);
    C2 *h = (C2 *)half + (int64_t)i * N * (N / 2 + 1);
    hipLaunchKernelGGL((i2g_rows_kernel<Real, N>), dim3(pairs / kRowSeqs<N>, m), dim3(kRowSeqs<N> * (N / 16)), 0, s,
                       (const Real *)image + (int64_t)i * N * N, k->d_kappa, tw, h);
    hipLaunchKernelGGL((i2g_cols_kernel<Real, N>), dim3((N / 2 + C) / C, m), dim3(C * (N / 16)), 0, s, h, tw,
                       (C2 *)grid + (int64_t)i * N * N);
  }
  return hipGetLastError();
}

template <typename F> hipError_t for_side(int n, F &&f) {
  switch (n) {
    case 128: return f(std::integral_constant<int, 128>{});
    case 256: return f(std::integral_constant<int, 256>{});
    case 512: return f(std::integral_constant<int, 512>{});
    case 1024: return f(std::integral_constant<int, 1024>{});
    case 2048: return f(std::integral_constant<int, 2048>{});
    case 4096: return f(std::integral_constant<int, 4096>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Which handles transform by themselves.  Without w-stacking: every side that has kernels.  With
// it, the column pass goes through an image's layers one after the other in n/16 columns a
// workgroup at the most, so few small images leave most of the chip idle, where rocFFT and a
// pass over the pixels take all layers side by side.  rocFFT's way and here, us, for 12 FP32
// layers: 22 and 42 for one image of 256^2, 37 and 47 for 4, 99 and 63 for 15; 49 and 76 for one
// of 512^2, 120 and 89 for 3; 140 and 84 for one of 1024^2.  For one layer: 16 and 25 for one of
// 512^2, 22 and 26 for 2, 28 and 27 for 3.  FP64 alike (3 images of 512^2: 33 and 31 with one
// layer, 129 and 105 with 12).  The line is 3 2^18 pixels of images.
constexpr int64_t kMinStackPixels = 3ll << 18;
bool own_fft(const wproj_params &p) {
  if (p.n < 128 || p.n > 4096 || (p.n & (p.n - 1)) != 0) return false;
  return p.w_mode != WPROJ_W_STACK || (int64_t)p.n_images * p.n * p.n >= kMinStackPixels;
}

std::vector<double> twiddle_table(int n) {
  std::vector<double> w(2 * (size_t)twiddle_base(n, passes_of(n)));
  int ns = radix_of(n, 0);
  for (int p = 1; p < passes_of(n); ++p) {
    const int R = radix_of(n, p), base = twiddle_base(n, p);
    for (int k = 0; k < R; ++k)
      for (int j = 0; j < ns; ++j) {
        const double a = -2.0 * M_PI * (double)(k * j) / (double)(ns * R);
        w[2 * (size_t)(base + k * ns + j)] = cos(a);
        w[2 * (size_t)(base + k * ns + j) + 1] = sin(a);
      }
    ns *= R;
  }
  return w;
}

hipError_t launch_grid_to_image(const wproj_kernels *k, void *grid, void *half, void *image, const double *wsum,
                                hipStream_t s) {
  return for_side(k->params.n, [&](auto n) {
    constexpr int N = decltype(n)::value;
    return k->params.precision == WPROJ_F64 ? g2i<double, N>(k, grid, half, image, wsum, s)
                                            : g2i<float, N>(k, grid, half, image, wsum, s);
  });
}

hipError_t launch_image_to_grid(const wproj_kernels *k, const void *image, void *half, void *grid, hipStream_t s) {
  return for_side(k->params.n, [&](auto n) {
    constexpr int N = decltype(n)::value;
    return i2g<double, N>(k, image, half, grid, s);
  });
}

}  // namespace wproj
