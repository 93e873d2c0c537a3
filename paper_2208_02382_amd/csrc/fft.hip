// Free-space Poisson solve by Hockney's zero-padded FFT convolution (padded lengths M_a = 2 n_a),
// with a hand-written FFT built from LDS radix-4/2/3 stages.
//
// Green spectrum.  The cyclic Green array is real and even along every axis, so its DFT is real
// and even: Ghat(k) depends on (fold(kx), fold(ky), fold(kz)) only, fold(k) = min(k, M - k).
// It is computed on the (n_x+1)(n_y+1)(n_z+1) cell averages by three even-real DFT passes (one
// per axis; two real lines ride in one complex FFT of the even extension), in float64, then
// scaled by 1/(4 pi eps0 Mx My Mz) and stored in the grid's precision.
//
// Solve, on the half spectrum W[Mz][My][Kx] (Kx = n_x + 1):
//   r2c_x   real charge rows (y < n_y, z < n_z) -> half spectra, through a complex FFT of length
//           n_x of the even/odd-packed row and the standard split;
//   c2c y   forward along y for the planes z < n_z only (the others are zero);
//   zconv   along z: forward FFT of the n_z non-zero inputs, product with Ghat, inverse FFT, and
//           only the n_z + 2 output rows on nodes -1..n_z are written back;
//   c2c y   inverse along y for those rows, writing the n_y + 2 rows on nodes -1..n_y;
//   c2r_x   inverse real transform of those rows, writing phi on nodes -1..n_x directly.
// The field is then E' = -grad phi by centred differences (k_grad).
//
// FFT engines: fft_reg.hpp holds the lines in registers (the lengths it lists: 16..256 of the
// usual grids); any other length 2^a 3^b <= 512 runs the engine below, where a workgroup holds
// LB lines of length L in LDS (LB L <= 4096 complex values, at most 64 KB) and runs a Stockham
// self-sorting decimation-in-time FFT (Govindaraju et al., SC'08 formulation) in place: each
// stage reads its butterfly inputs to registers, barriers, writes the outputs.  Lines along y
// and z are batched along x, so every row load is a run of consecutive complex values.  Twiddles
// come from a per-axis table exp(-2 pi i t/M) computed with sincospi; a half-length transform
// reads every second entry.
#include <algorithm>

#include "fft_reg.hpp"
#include "internal.hpp"

namespace pic {

namespace {

constexpr int kLdsElems = 4096;  // complex values per workgroup (64 KB for complex double)

// One Stockham stage of radix R over LB lines of length M (line stride M + 1): butterfly bf
// (line l, j < M/R, k = j mod Ns) reads buf[l, j + r M/R], applies the twiddles
// exp(-+2 pi i r k / (Ns R)) and the radix-R DFT, and writes buf[l, (j / Ns) Ns R + k + r Ns].
// Each thread takes up to two butterflies; inputs are read before the barrier and outputs
// written after it.
template <typename T, int DIR, int R>
__device__ __forceinline__ void fft_stage(Cx<T>* buf, int LB, int M, int Ns,
                                          const typename TwT<T>::type* tw, int tws) {
  const int MR = M / R;
  const int nbf = LB * MR;
  const int NT = blockDim.x;
  Cx<T> v[2][R];
  int ob[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int bf = threadIdx.x + q * NT;
    ob[q] = -1;
    if (bf < nbf) {
      const int l = bf / MR, j = bf - l * MR;
      const int k = j % Ns;
      const Cx<T>* src = buf + l * (M + 1) + j;
      const int tstep = k * (M / (Ns * R)) * tws;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        Cx<T> a = src[r * MR];
        if (r && tstep) {
          const auto w = tw[r * tstep];
          a = cmul(a, Cx<T>{(T)w.x, DIR < 0 ? (T)w.y : (T)-w.y});
        }
        v[q][r] = a;
      }
      dft<T, DIR, R>(v[q]);
      ob[q] = l * (M + 1) + (j / Ns) * Ns * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (ob[q] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) buf[ob[q] + r * Ns] = v[q][r];
    }
  __syncthreads();
}

// In-place LDS FFT of LB lines of length ax.M (line l at buf[l (M + 1)]: the padding of one
// element per line spreads the transposed loads and stores of y and z lines over the LDS
// banks).  Twiddle exp(-2 pi i t/M) is tw[t * tws] (tws = 2 when the table belongs to a
// transform twice as long).  Requires blockDim.x >= LB M / 4.  Ends with a barrier.
template <typename T, int DIR>
__device__ void fft_lds(Cx<T>* buf, int LB, const FftAxis& ax, const typename TwT<T>::type* tw,
                        int tws) {
  // the planner's radix order: all factors 4, then 2, then 3 (derived from M here, so that
  // no array is indexed at run time)
  const int M = ax.M;
  int m = M, Ns = 1;
  while (m % 4 == 0) {
    fft_stage<T, DIR, 4>(buf, LB, M, Ns, tw, tws);
    Ns *= 4;
    m /= 4;
  }
  while (m % 2 == 0) {
    fft_stage<T, DIR, 2>(buf, LB, M, Ns, tw, tws);
    Ns *= 2;
    m /= 2;
  }
  while (m % 3 == 0) {
    fft_stage<T, DIR, 3>(buf, LB, M, Ns, tw, tws);
    Ns *= 3;
    m /= 3;
  }
}

// Copies `count` twiddles into LDS right after the LB lines of buf (LB (M + 1) elements), so
// that the stages read them from LDS instead of global memory; ordered before the first stage
// by the barrier that ends the caller's load phase.
template <typename T>
__device__ __forceinline__ const typename TwT<T>::type* stage_twiddles(
    Cx<T>* buf, int LB, int M, const typename TwT<T>::type* __restrict__ tw, int count) {
  auto* twl = reinterpret_cast<typename TwT<T>::type*>(buf + LB * (M + 1));
  for (int t = threadIdx.x; t < count; t += blockDim.x) twl[t] = tw[t];
  return twl;
}

// Fills the LB lines of length M in LDS (line l at buf[l (M + 1)]) from global memory, element
// p of line l from addr(p, l) where ok(p, l) holds and zero elsewhere; consecutive threads take
// consecutive lines, which are consecutive in memory.  A thread issues its loads four at a time
// before it stores any of them to LDS, the addresses of elements that are not loaded replaced by
// `safe` (any valid address) and the values by zero, so that no branch surrounds a load: a load
// inside a branch is waited for at the branch's join, which would put the latencies of a
// thread's loads one after another.
template <typename T, typename Addr, typename Ok>
__device__ __forceinline__ void load_lines(Cx<T>* buf, int LB, int M, const Cx<T>* safe,
                                           Addr addr, Ok ok) {
  const int total = LB * M, nt = (int)blockDim.x;
  for (int i0 = (int)threadIdx.x; i0 < total; i0 += 4 * nt) {
    Cx<T> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      const int p = idx / LB, l = idx - p * LB;
      const bool use = idx < total && ok(p, l);
      const Cx<T> x = ld(use ? addr(p, l) : safe);
      v[u] = use ? x : Cx<T>{0, 0};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      if (idx < total) {
        const int p = idx / LB, l = idx - p * LB;
        buf[l * (M + 1) + p] = v[u];
      }
    }
  }
}

// cyclic index of the ghost-inclusive position p = 0..n+1 (node p - 1): M - 1 for p = 0
__device__ __forceinline__ int ghost_src(int p, int M) { return p == 0 ? M - 1 : p - 1; }

// Three uses of the same passes.  MODE 0 (Poisson solve): the source lives on nodes 0..n-1 and
// the result is kept on nodes -1..n.  MODE 1 (transposed solve of the reverse sweep): the
// source lives on nodes -1..n (node -1 at cyclic index M - 1) and the result is kept on nodes
// 0..n-1.  MODE 2 (direct field): source and result on nodes 0..n-1.  All are exact: every
// source-to-output offset lies in [-n, n].
template <int MODE>
__device__ __forceinline__ bool src_nonzero(int p, int n, int M) {
  return MODE != 1 ? p < n : (p <= n || p == M - 1);
}
template <int MODE>
__device__ __forceinline__ int out_count(int n) { return MODE == 0 ? n + 2 : n; }
template <int MODE>
__device__ __forceinline__ int out_src(int q, int M) { return MODE == 0 ? ghost_src(q, M) : q; }
__device__ __forceinline__ int fold(int k, int M) { return k <= M / 2 ? k : M - k; }

// ------------------------------------------------------------------------------ Green spectrum

// Even-real DFT along one axis of the float64 array gd[(k (ny+1) + j)(nx+1) + i] in place:
// line values g_0..g_n are extended to length M = 2n by g_t = g_{M-t}, transformed, and the
// real outputs k = 0..n stored.  Complex line c carries real lines a = 2c (real part) and
// a = 2c + 1 (imaginary part); line a starts at a*sa + b*sb, elements at stride st.
// ODD: the odd extension g_t = -g_{M-t} (g_n = 0, an offset no output node reaches), whose
// transform is i S_k with S real; S is stored (the factor i is applied by the product).  For
// a packed pair Z = A + i B with A = i S_A, B = i S_B: S_A = Im Z, S_B = -Re Z.
template <bool ODD>
__device__ __forceinline__ void green_dft_body(double* __restrict__ gd, FftAxis ax,
                                                         const double2* __restrict__ tw,
                                                         int64_t st, int64_t sa, int64_t sb,
                                                         int na, int LB, int bx, int by, int nbx) {
  extern __shared__ unsigned char smem_raw[];
  Cx<double>* buf = reinterpret_cast<Cx<double>*>(smem_raw);
  const int M = ax.M, n = M / 2;
  const int c0 = bx * LB;  // first complex line of this block
  double* base = gd + (int64_t)by * sb;
  // consecutive threads take consecutive elements of a line where the line is contiguous in
  // memory (st == 1), else consecutive lines (contiguous across lines)
  const bool efast = st == 1;
  for (int idx = threadIdx.x; idx < LB * M; idx += blockDim.x) {
    int p, l;
    if (efast) {
      l = idx / M;
      p = idx - l * M;
    } else {
      p = idx / LB;
      l = idx - p * LB;
    }
    const int t = p <= n ? p : M - p;
    const double sgn = ODD ? (p < n ? 1.0 : (p == n ? 0.0 : -1.0)) : 1.0;
    const int a0 = 2 * (c0 + l), a1 = a0 + 1;
    double re = a0 < na ? base[(int64_t)a0 * sa + (int64_t)t * st] : 0.0;
    double im = a1 < na ? base[(int64_t)a1 * sa + (int64_t)t * st] : 0.0;
    buf[l * (M + 1) + p] = Cx<double>{sgn * re, sgn * im};
  }
  const double2* twl = stage_twiddles(buf, LB, M, tw, M);
  __syncthreads();
  fft_lds<double, -1>(buf, LB, ax, twl, 1);
  for (int idx = threadIdx.x; idx < LB * (n + 1); idx += blockDim.x) {
    int p, l;
    if (efast) {
      l = idx / (n + 1);
      p = idx - l * (n + 1);
    } else {
      p = idx / LB;
      l = idx - p * LB;
    }
    const int a0 = 2 * (c0 + l), a1 = a0 + 1;
    const Cx<double> v = buf[l * (M + 1) + p];
    if (a0 < na) base[(int64_t)a0 * sa + (int64_t)p * st] = ODD ? v.y : v.x;
    if (a1 < na) base[(int64_t)a1 * sa + (int64_t)p * st] = ODD ? -v.x : v.y;
  }
}

__device__ __forceinline__ void green_even_dft_body(double* __restrict__ gd, FftAxis ax,
                                                    const double2* __restrict__ tw, int64_t st,
                                                    int64_t sa, int64_t sb, int na, int LB,
                                                    int bx, int by, int nbx) {
  green_dft_body<false>(gd, ax, tw, st, sa, sb, na, LB, bx, by, nbx);
}

template <bool ODD>
__global__ __launch_bounds__(1024) void k_green_dft(double* __restrict__ gd, FftAxis ax,
                                                    const double2* __restrict__ tw, int64_t st,
                                                    int64_t sa, int64_t sb, int na, int LB) {
  green_dft_body<ODD>(gd, ax, tw, st, sa, sb, na, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

template <typename T>
__device__ __forceinline__ void green_finish_body(const Geom* __restrict__ g,
                                                      const double* __restrict__ gd,
                                                      T* __restrict__ gh, int64_t total,
                                                      double scale, int bx, int by, int nbx) {
  if (g->status) return;
  for (int64_t t = bx * 256ll + threadIdx.x; t < total; t += (int64_t)nbx * 256)
    gh[t] = (T)(gd[t] * scale);
}

template <typename T>
__global__ __launch_bounds__(256) void k_green_finish(const Geom* __restrict__ g,
                                                      const double* __restrict__ gd,
                                                      T* __restrict__ gh, int64_t total,
                                                      double scale) {
  green_finish_body<T>(g, gd, gh, total, scale, blockIdx.x, blockIdx.y, gridDim.x);
}

// ------------------------------------------------------------------------------ solve passes

// Forward real transform of the source rows into the half spectrum W[z][y][0..n_x], z and y
// cyclic.  MODE 0: rows (y < n_y, z < n_z) of the charge src[z][y][x] (length n_x).  MODE 1:
// rows (yy < n_y + 2, zz < n_z + 2) of the ghost-inclusive source src[zz][yy][xx]
// (length n_x + 2, node xx - 1), stored at cyclic rows (ghost_src(zz), ghost_src(yy)).
// Packed z_j = x_{2j} + i x_{2j+1}, j < n_x, complex FFT of length n_x (ax), then
// X_k = E_k + W^k O_k, E_k = (Z_k + conj Z_{n-k})/2, O_k = (Z_k - conj Z_{n-k})/(2i),
// W = exp(-2 pi i / M_x), k = 0..n_x.
template <typename T, int MODE>
__device__ __forceinline__ void r2c_x_body(const Geom* __restrict__ g,
                                                const T* __restrict__ src, Cx<T>* __restrict__ W,
                                                FftAxis ax, const typename TwT<T>::type* __restrict__ tw,
                                                int nx, int ny, int nz, int Kx, int My, int LB, int bx, int by, int nbx) {
  extern __shared__ unsigned char smem_raw[];
  Cx<T>* buf = reinterpret_cast<Cx<T>*>(smem_raw);
  if (g->status) return;
  const int H = ax.M;  // = nx
  const int M = 2 * H;
  const int rows = MODE == 0 ? ny : ny + 2;
  const int len = MODE == 0 ? nx : nx + 2;
  const int y0 = bx * LB, z = by;
  const int nl = min(LB, rows - y0);
  const T* s0 = src + ((int64_t)z * rows + y0) * len;
  // four elements per thread at a time, their loads issued before any is stored and with no
  // branch around a load (out-of-range addresses replaced by the row's start, values by zero)
  const int total = LB * H, nt = (int)blockDim.x;
  for (int i0 = (int)threadIdx.x; i0 < total; i0 += 4 * nt) {
    T vr[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      const int l = idx / H, j = idx - l * H;
      const bool row_ok = idx < total && l < nl;
      const T* row = s0 + (int64_t)(row_ok ? l : 0) * len;
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        const int t = 2 * j + h2;  // cyclic position
        int at = -1;               // its element in the source row, if any
        if (MODE == 0) {
          if (t < nx) at = t;
        } else {
          if (t <= nx) at = t + 1;
          else if (t == M - 1) at = 0;
        }
        const bool use = row_ok && at >= 0;
        const T val = row[use ? at : 0];
        vr[u][h2] = use ? val : T(0);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      if (idx < total) {
        const int l = idx / H, j = idx - l * H;
        buf[l * (H + 1) + j] = Cx<T>{vr[u][0], vr[u][1]};
      }
    }
  }
  const auto* twl = stage_twiddles(buf, LB, H, tw, M);
  __syncthreads();
  fft_lds<T, -1>(buf, LB, ax, twl, 2);
  const int cz = MODE == 0 ? z : ghost_src(z, 2 * nz);
  for (int idx = threadIdx.x; idx < LB * (H + 1); idx += blockDim.x) {
    const int l = idx / (H + 1), k = idx - l * (H + 1);
    if (l >= nl) continue;
    const int cy = MODE == 0 ? y0 + l : ghost_src(y0 + l, My);
    const Cx<T> zk = buf[l * (H + 1) + (k % H)];
    const Cx<T> zc = cconj(buf[l * (H + 1) + ((H - k) % H)]);
    const Cx<T> e = {(T)0.5 * (zk.x + zc.x), (T)0.5 * (zk.y + zc.y)};
    const Cx<T> dif = csub(zk, zc);
    const Cx<T> o = {(T)0.5 * dif.y, (T)-0.5 * dif.x};  // dif / (2i)
    const auto w = tw[k];                              // exp(-2 pi i k / M_x)
    W[((int64_t)cz * My + cy) * Kx + k] = cadd(e, cmul(Cx<T>{(T)w.x, (T)w.y}, o));
  }
}

template <typename T, int MODE>
__global__ __launch_bounds__(1024) void k_r2c_x(const Geom* __restrict__ g,
                                                const T* __restrict__ src, Cx<T>* __restrict__ W,
                                                FftAxis ax, const typename TwT<T>::type* __restrict__ tw,
                                                int nx, int ny, int nz, int Kx, int My, int LB) {
  r2c_x_body<T, MODE>(g, src, W, ax, tw, nx, ny, nz, Kx, My, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

// Complex line FFT in place along y (element stride Kx) for lines a = kx (stride 1) on the
// planes b = blockIdx.y.  STAGE 0 (forward): the planes holding source rows -- z < n_z
// (MODE 0) or the cyclic rows of nodes -1..n_z (MODE 1) -- with the source's non-zero inputs
// only, all M outputs stored.  STAGE 1 (inverse): the planes b < out_count(n_z) written by the
// z pass, all M inputs, the out_count(n_y) kept rows stored at positions q from out_src(q).
template <typename T, int DIR, int MODE, int STAGE>
__device__ __forceinline__ void c2c_y_body(const Geom* __restrict__ g, Cx<T>* __restrict__ W,
                                                FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int Kx, int ny, int nz, int LB, int bx, int by, int nbx) {
  extern __shared__ unsigned char smem_raw[];
  Cx<T>* buf = reinterpret_cast<Cx<T>*>(smem_raw);
  if (g->status) return;
  const int M = ax.M;
  const int a0 = bx * LB;
  const int nl = min(LB, Kx - a0);
  const int plane = (STAGE == 0 && MODE == 1) ? ghost_src(by, 2 * nz) : (int)by;
  Cx<T>* base = W + (int64_t)plane * M * Kx + a0;
  load_lines<T>(
      buf, LB, M, base, [&](int p, int l) { return base + (int64_t)p * Kx + l; },
      [&](int p, int l) { return l < nl && (STAGE == 1 || src_nonzero<MODE>(p, ny, M)); });
  const auto* twl = stage_twiddles(buf, LB, M, tw, M);
  __syncthreads();
  fft_lds<T, DIR>(buf, LB, ax, twl, 1);
  const int nout = STAGE == 0 ? M : out_count<MODE>(ny);
  for (int idx = threadIdx.x; idx < LB * nout; idx += blockDim.x) {
    const int q = idx / LB, l = idx - q * LB;
    if (l < nl)
      base[(int64_t)q * Kx + l] = buf[l * (M + 1) + (STAGE == 0 ? q : out_src<MODE>(q, M))];
  }
}

template <typename T, int DIR, int MODE, int STAGE>
__global__ __launch_bounds__(1024) void k_c2c_y(const Geom* __restrict__ g, Cx<T>* __restrict__ W,
                                                FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int Kx, int ny, int nz, int LB) {
  c2c_y_body<T, DIR, MODE, STAGE>(g, W, ax, tw, Kx, ny, nz, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

// Along z (element stride My Kx) for lines a = kx, b = ky: forward FFT of the source's
// non-zero inputs, product with Ghat(fold kz, fold ky, kx) (gh[(fz (ny+1) + fy)(nx+1) + kx]),
// inverse FFT, and the out_count(n_z) kept rows written back in place.
// IMAG: the kernel spectrum is i gh (an odd field kernel, see green_dft_body), odd along axis
// `odd`: its spectrum is odd there too, so the folded value changes sign for k_y > n_y
// (odd = 1) or k_z > n_z (odd = 2); along x only k_x <= n_x is stored, no fold.  W2: where the
// kept rows go (W itself for the potential).
template <typename T, int MODE, bool IMAG = false>
__device__ __forceinline__ void zconv_body(const Geom* __restrict__ g, Cx<T>* W,
                                                const T* __restrict__ gh, FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int Kx, int My, int ny, int nz, int LB, int bx, int by, int nbx,
                                                Cx<T>* W2 = nullptr, int odd = -1) {
  extern __shared__ unsigned char smem_raw[];
  Cx<T>* buf = reinterpret_cast<Cx<T>*>(smem_raw);
  if (g->status) return;
  const int M = ax.M;
  const int a0 = bx * LB, ky = by;
  const int nl = min(LB, Kx - a0);
  const int64_t sz = (int64_t)My * Kx;
  Cx<T>* base = W + (int64_t)ky * Kx + a0;
  Cx<T>* obase = (W2 ? W2 : W) + (int64_t)ky * Kx + a0;
  load_lines<T>(
      buf, LB, M, base, [&](int p, int l) { return base + (int64_t)p * sz + l; },
      [&](int p, int l) { return l < nl && src_nonzero<MODE>(p, nz, M); });
  const auto* twl = stage_twiddles(buf, LB, M, tw, M);
  const int fy = fold(ky, My);
  const T* grow = gh + (int64_t)fy * Kx + a0;
  const int64_t gplane = (int64_t)(ny + 1) * Kx;
  const bool flip_y = IMAG && odd == 1 && ky > ny;
  const int total = LB * M, nt = (int)blockDim.x;
  __syncthreads();
  fft_lds<T, -1>(buf, LB, ax, twl, 1);
  // the kernel spectrum of the thread's first 4 elements (all of them with the launches'
  // shapes, LB M <= 4 blockDim.x), loaded together without a branch around a load (loading it
  // before the transform would hold 8 more registers through it and halve the resident blocks)
  T gs[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int idx = (int)threadIdx.x + u * nt;
    const int p = idx / LB, l = idx - p * LB;
    const bool use = idx < total && l < nl;
    gs[u] = grow[use ? (int64_t)fold(p, M) * gplane + l : 0];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int idx = (int)threadIdx.x + u * nt;
    const int p = idx / LB, l = idx - p * LB;
    if (idx < total && l < nl) {
      T s = gs[u];
      if (IMAG && (flip_y || (odd == 2 && p > nz))) s = -s;
      Cx<T> v = buf[l * (M + 1) + p];
      buf[l * (M + 1) + p] = IMAG ? Cx<T>{-v.y * s, v.x * s} : Cx<T>{v.x * s, v.y * s};
    }
  }
  // elements past 4 blockDim.x (none with the launches' shapes) load their spectrum here
  for (int idx = (int)threadIdx.x + 4 * nt; idx < total; idx += nt) {
    const int p = idx / LB, l = idx - p * LB;
    if (l < nl) {
      T s = grow[(int64_t)fold(p, M) * gplane + l];
      if (IMAG && (flip_y || (odd == 2 && p > nz))) s = -s;
      Cx<T> v = buf[l * (M + 1) + p];
      buf[l * (M + 1) + p] = IMAG ? Cx<T>{-v.y * s, v.x * s} : Cx<T>{v.x * s, v.y * s};
    }
  }
  __syncthreads();
  fft_lds<T, +1>(buf, LB, ax, twl, 1);
  for (int idx = threadIdx.x; idx < LB * out_count<MODE>(nz); idx += blockDim.x) {
    const int q = idx / LB, l = idx - q * LB;
    if (l < nl) obase[(int64_t)q * sz + l] = buf[l * (M + 1) + out_src<MODE>(q, M)];
  }
}

template <typename T, int MODE>
__global__ __launch_bounds__(1024) void k_zconv(const Geom* __restrict__ g, Cx<T>* __restrict__ W,
                                                const T* __restrict__ gh, FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int Kx, int My, int ny, int nz, int LB) {
  zconv_body<T, MODE>(g, W, gh, ax, tw, Kx, My, ny, nz, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

// direct field: forward z FFT of W (kept intact for the next component), product with i gh,
// inverse z FFT, the n_z node rows into W2 [n_z][2 n_y][n_x + 1]
template <typename T>
__global__ __launch_bounds__(1024) void k_zconv_field(const Geom* __restrict__ g,
                                                      Cx<T>* __restrict__ W,
                                                      const T* __restrict__ gh, FftAxis ax,
                                                      const typename TwT<T>::type* __restrict__ tw,
                                                      int Kx, int My, int ny, int nz, int LB,
                                                      Cx<T>* __restrict__ W2, int odd) {
  zconv_body<T, 2, true>(g, W, gh, ax, tw, Kx, My, ny, nz, LB, blockIdx.x, blockIdx.y, gridDim.x,
                         W2, odd);
}

// Inverse real transform of the kept rows (yy < out_count(n_y), zz < out_count(n_z)) of W,
// writing the result on the kept x-nodes (MODE 0: -1..n_x into phi[(nz+2)][(ny+2)][(nx+2)];
// MODE 1: 0..n_x-1 into an [nz][ny][nx] array): Z_k = (X_k + conj X_{n-k}) + i exp(+2 pi i k/M_x)(X_k - conj X_{n-k}),
// k < n = n_x, inverse complex FFT of length n_x, x_{2j} = Re z_j, x_{2j+1} = Im z_j.
template <typename T, int MODE>
__device__ __forceinline__ void c2r_x_body(const Geom* __restrict__ g,
                                                const Cx<T>* __restrict__ W, T* __restrict__ phi,
                                                FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int nx, int ny, int Kx, int My, int LB, int bx, int by, int nbx) {
  extern __shared__ unsigned char smem_raw[];
  Cx<T>* buf = reinterpret_cast<Cx<T>*>(smem_raw);
  if (g->status) return;
  const int H = ax.M;  // = nx
  const int M = 2 * H;
  const int py = out_count<MODE>(ny);
  const int r0 = bx * LB, zz = by;
  const int nl = min(LB, py - r0);
  const Cx<T>* src = W + ((int64_t)zz * My + r0) * Kx;
  // four elements per thread at a time, their loads issued before any is used and with no
  // branch around a load (rows past the block's last read as row 0, their values not used)
  const int total = LB * H, nt = (int)blockDim.x;
  for (int i0 = (int)threadIdx.x; i0 < total; i0 += 4 * nt) {
    Cx<T> xk[4], xh[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      const int l = idx / H, k = idx - l * H;
      const bool ok = idx < total && l < nl;
      const Cx<T>* row = src + (int64_t)(ok ? l : 0) * Kx;
      const int kk = ok ? k : 0;
      xk[u] = ld(row + kk);
      xh[u] = ld(row + (H - kk));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = i0 + u * nt;
      if (idx < total) {
        const int l = idx / H, k = idx - l * H;
        const auto w = tw[k];
        Cx<T> v = {0, 0};
        if (l < nl) {
          const Cx<T> xc = cconj(xh[u]);
          const Cx<T> winv = {(T)w.x, (T)-w.y};  // exp(+2 pi i k / M_x)
          const Cx<T> d = cmul(winv, csub(xk[u], xc));
          v = cadd(cadd(xk[u], xc), Cx<T>{-d.y, d.x});  // + i d
        }
        buf[l * (H + 1) + k] = v;
      }
    }
  }
  const auto* twl = stage_twiddles(buf, LB, H, tw, M);
  __syncthreads();
  fft_lds<T, +1>(buf, LB, ax, twl, 2);
  const int px = out_count<MODE>(nx);
  T* dst = phi + ((int64_t)zz * py + r0) * px;
  for (int idx = threadIdx.x; idx < LB * px; idx += blockDim.x) {
    const int l = idx / px, q = idx - l * px;
    if (l < nl) {
      const int t = out_src<MODE>(q, M);
      const Cx<T> zj = buf[l * (H + 1) + (t >> 1)];
      dst[(int64_t)l * px + q] = (t & 1) ? zj.y : zj.x;
    }
  }
}

template <typename T, int MODE>
__global__ __launch_bounds__(1024) void k_c2r_x(const Geom* __restrict__ g,
                                                const Cx<T>* __restrict__ W, T* __restrict__ phi,
                                                FftAxis ax,
                                                const typename TwT<T>::type* __restrict__ tw,
                                                int nx, int ny, int Kx, int My, int LB) {
  c2r_x_body<T, MODE>(g, W, phi, ax, tw, nx, ny, Kx, My, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

// E'[c][k][j][i] = -(phi(n + e_c) - phi(n - e_c)) / (2 h_c), rest-frame spacings
template <typename T>
__device__ __forceinline__ void grad_body(const Geom* __restrict__ g, const T* __restrict__ phi,
                                              T* __restrict__ E, int nx, int ny, int nz, int bx, int by, int nbx) {
  if (g->status) return;
  const int px = nx + 2, py = ny + 2;
  const int64_t total = (int64_t)nx * ny * nz;
  const T cx = (T)(1.0 / (2.0 * g->h_rest[0]));
  const T cy = (T)(1.0 / (2.0 * g->h_rest[1]));
  const T cz = (T)(1.0 / (2.0 * g->h_rest[2]));
  const int64_t sy = px, sz = (int64_t)px * py;
  for (int64_t t = bx * 256ll + threadIdx.x; t < total; t += (int64_t)nbx * 256) {
    const Idx3 q3 = split3(t, nx, ny);
    const int i = q3.x, j = q3.y, k = q3.z;
    int64_t c = (int64_t)(k + 1) * sz + (int64_t)(j + 1) * sy + (i + 1);
    E[t] = -(phi[c + 1] - phi[c - 1]) * cx;
    E[total + t] = -(phi[c + sy] - phi[c - sy]) * cy;
    E[2 * total + t] = -(phi[c + sz] - phi[c - sz]) * cz;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_grad(const Geom* __restrict__ g, const T* __restrict__ phi,
                                              T* __restrict__ E, int nx, int ny, int nz) {
  grad_body<T>(g, phi, E, nx, ny, nz, blockIdx.x, blockIdx.y, gridDim.x);
}


// --------------------------------------------------------------- passes in registers
// One launch covers one beam (args) or a batch (beam = blockIdx.y).  Lines are numbered through
// all planes, so only the last workgroup of a beam can hold fewer lines than fit.  What bounds
// them is the traffic of W (34 MB over the three passes that touch it at 64^3, from the caches)
// and, on small grids, one workgroup's chain of loads, transform and stores.  Float64, us per
// launch, runtime-length engine / registers, at 64^3 and 128^3: r2c 13.7 / 6.0 and 36 / 15, y
// 13.7 / 8.0 and 45 / 35, z 37 / 10.5 and 163 / 45, y inverse 14.1 / 9.4 and 46 / 32, c2r
// 12.0 / 5.4 and 33 / 19, one axis of the kernel spectrum 13 / 7 and 30 / 22; the z pass of 256
// batched beams 3118 / 731.

// MODE, IMAG and ODD of the kernels above as run-time values
struct FftArgs {
  const Geom* g;
  int nx, ny, nz;
  int mode;
  int odd;          // zconv: axis along which the kernel spectrum is odd (IMAG), else -1
  const void* src;  // r2c: source rows
  void* W;
  void* W2;         // zconv: where the kept rows go
  const void* gh;
  void* dst;        // c2r: result rows
  const void* tw[3];
};

template <typename T>
__device__ __forceinline__ const typename TwT<T>::type* tw_of(const FftPlan& p, int a);
template <>
__device__ __forceinline__ const double2* tw_of<double>(const FftPlan& p, int a) { return p.tw[a]; }
template <>
__device__ __forceinline__ const float2* tw_of<float>(const FftPlan& p, int a) { return p.twf[a]; }

// the arguments of beam blockIdx.y of a batch (a Poisson solve in place), or those given
template <typename T>
__device__ __forceinline__ FftArgs beam_args(const FftArgs& args, const BeamDev* beams) {
  if (!beams) return args;
  const BeamDev& d = beams[blockIdx.y];
  FftArgs a;
  a.g = d.geom;
  a.nx = d.c.nx;
  a.ny = d.c.ny;
  a.nz = d.c.nz;
  a.mode = 0;
  a.odd = -1;
  a.src = d.rho;
  a.W = d.W;
  a.W2 = d.W;
  a.gh = d.Gh;
  a.dst = d.phi;
  for (int q = 0; q < 3; ++q) a.tw[q] = tw_of<T>(d.plan, q);
  return a;
}
template <typename T>
__device__ __forceinline__ const typename TwT<T>::type* tw_arg(const FftArgs& a, int axis) {
  return reinterpret_cast<const typename TwT<T>::type*>(a.tw[axis]);
}

__host__ __device__ __forceinline__ int mode_out(int mode, int n) { return mode == 0 ? n + 2 : n; }
__host__ __device__ __forceinline__ int mode_src(int mode, int n) { return mode == 1 ? n + 2 : n; }
// output position of cyclic index t on the kept nodes, -1 if it is not kept
__device__ __forceinline__ int mode_out_pos(int mode, int t, int n, int M) {
  if (mode != 0) return t < n ? t : -1;
  return t <= n ? t + 1 : (t == M - 1 ? 0 : -1);
}
__device__ __forceinline__ bool mode_src_nonzero(int mode, int p, int n, int M) {
  return mode != 1 ? p < n : (p <= n || p == M - 1);
}

// see r2c_x_body; H = n_x
template <typename T, int H>
__device__ __forceinline__ void r2c_reg(const FftArgs& a, Cx<T>* buf, int blk) {
  constexpr int LB = line_count<H>(), TPL = line_threads<H>(), M = 2 * H;
  const int mode = a.mode;
  const int ry = mode_src(mode, a.ny), len = mode_src(mode, H);
  const int rows = ry * mode_src(mode, a.nz);
  if (blk * LB >= rows) return;
  int l, j;
  line_pos<H, false>(&l, &j);
  const int row = min(blk * LB + l, rows - 1);
  const bool ok = blk * LB + l < rows;
  const T* s = (const T*)a.src + (int64_t)row * len;
  const auto* tw = tw_arg<T>(a, 0);
  auto elem = [&](int t) {  // element t of the zero-padded row
    int at = -1;
    if (mode != 1) {
      if (t < H) at = t;
    } else {
      if (t <= H) at = t + 1;
      else if (t == M - 1) at = 0;
    }
    const T v = s[at >= 0 ? at : 0];
    return at >= 0 ? v : T(0);
  };
  line_fft<T, -1, H, false, 2>(
      buf, l, j, tw, [&](int p) { return Cx<T>{elem(2 * p), elem(2 * p + 1)}; },
      [&](auto& v) {
        __syncthreads();
        each_output<T, H>(v, j, [&](int p, Cx<T> x) { buf[lds_at<H, false>(l, p)] = x; });
        __syncthreads();
      });
  const int z = row / ry, y = row - z * ry;
  const int My = 2 * a.ny;
  const int cz = mode == 1 ? ghost_src(z, 2 * a.nz) : z;
  const int cy = mode == 1 ? ghost_src(y, My) : y;
  Cx<T>* out = (Cx<T>*)a.W + ((int64_t)cz * My + cy) * (H + 1);
#pragma unroll
  for (int k0 = 0; k0 <= H; k0 += TPL) {
    const int k = k0 + j;
    if (k > H || !ok) continue;
    const Cx<T> zk = buf[lds_at<H, false>(l, k == H ? 0 : k)];
    const Cx<T> zc = cconj(buf[lds_at<H, false>(l, k == 0 ? 0 : H - k)]);
    const Cx<T> e = {(T)0.5 * (zk.x + zc.x), (T)0.5 * (zk.y + zc.y)};
    const Cx<T> dif = csub(zk, zc);
    const Cx<T> o = {(T)0.5 * dif.y, (T)-0.5 * dif.x};  // dif / (2i)
    const auto w = tw[k];                              // exp(-2 pi i k / M_x)
    out[k] = cadd(e, cmul(Cx<T>{(T)w.x, (T)w.y}, o));
  }
}

// see c2c_y_body; M = 2 n_y
template <typename T, int M, int DIR>
__device__ __forceinline__ void c2c_y_reg(const FftArgs& a, Cx<T>* buf, int blk) {
  constexpr int LB = line_count<M>();
  const int Kx = a.nx + 1, mode = a.mode;
  const int planes = DIR < 0 ? mode_src(mode, a.nz) : mode_out(mode, a.nz);
  const int lines = Kx * planes;
  if (blk * LB >= lines) return;
  int l, j;
  line_pos<M, true>(&l, &j);
  const int g = min(blk * LB + l, lines - 1);
  const bool ok = blk * LB + l < lines;
  int b = g / Kx;
  const int x = g - b * Kx;
  if (DIR < 0 && mode == 1) b = ghost_src(b, 2 * a.nz);
  Cx<T>* base = (Cx<T>*)(DIR < 0 ? a.W : a.W2) + (int64_t)b * M * Kx + x;
  line_fft<T, DIR, M, true, 1>(
      buf, l, j, tw_arg<T>(a, 1),
      [&](int p) {
        const bool use = DIR > 0 || mode_src_nonzero(mode, p, M / 2, M);
        const Cx<T> v = ld(use ? base + (int64_t)p * Kx : base);
        return use ? v : Cx<T>{0, 0};
      },
      [&](auto& v) {
        each_output<T, M>(v, j, [&](int p, Cx<T> x) {
          const int q = DIR < 0 ? p : mode_out_pos(mode, p, M / 2, M);
          if (ok && q >= 0) base[(int64_t)q * Kx] = x;
        });
      });
}

// see zconv_body; M = 2 n_z
template <typename T, int M, bool IMAG>
__device__ __forceinline__ void zconv_reg(const FftArgs& a, Cx<T>* buf, int blk) {
  constexpr int LB = line_count<M>();
  const int Kx = a.nx + 1, My = 2 * a.ny, mode = a.mode;
  const int lines = Kx * My;
  if (blk * LB >= lines) return;
  int l, j;
  line_pos<M, true>(&l, &j);
  const int g = min(blk * LB + l, lines - 1);
  const bool ok = blk * LB + l < lines;
  const int ky = g / Kx, kx = g - ky * Kx;
  const int64_t sz = lines;
  const Cx<T>* base = (const Cx<T>*)a.W + g;
  Cx<T>* obase = (Cx<T>*)a.W2 + g;
  const T* grow = (const T*)a.gh + (int64_t)fold(ky, My) * Kx + kx;
  const int64_t gplane = (int64_t)(a.ny + 1) * Kx;
  // signs of the folded spectrum past the Nyquist index: of this line, and along it.  As factors: of
  // `if (flip_y || (odd == 2 && p > n_z)) s = -s` clang 22 (ROCm 7.2) drops the negation where two
  // branches lead to it.  Its LLVM IR still has it; in the machine code -s is computed ahead of the
  // branches into the register that the other branch then overwrites with s, and the block that
  // negates is left empty (`s_and_saveexec` followed by the `s_or` that undoes it).  The z component
  // was then 1 to 30 % off at every z length whose last radix is even.
  const T sign_y = IMAG && a.odd == 1 && ky > a.ny ? T(-1) : T(1);
  const T sign_z = IMAG && a.odd == 2 ? T(-1) : T(1);
  const auto* tw = tw_arg<T>(a, 2);
  using FWD = typename RadicesOf<M>::fwd;
  using INV = typename ReverseRadices<FWD>::type;
  line_fft<T, -1, M, true, 1>(
      buf, l, j, tw,
      [&](int p) {
        const bool use = mode_src_nonzero(mode, p, M / 2, M);
        const Cx<T> v = ld(use ? base + (int64_t)p * sz : base);
        return use ? v : Cx<T>{0, 0};
      },
      [&](auto& v) {
        constexpr int Q = sizeof(v) / sizeof(v[0]), R = sizeof(v[0]) / sizeof(v[0][0]);
        constexpr int TPL = line_threads<M>(), NS = M / R;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int jb = j + q * TPL < NS ? j + q * TPL : 0;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int p = jb + r * NS;
            T s = grow[(int64_t)fold(p, M) * gplane];
            if constexpr (IMAG) s *= sign_y * (p > M / 2 ? sign_z : T(1));
            const Cx<T> x = v[q][r];
            v[q][r] = IMAG ? Cx<T>{-x.y * s, x.x * s} : Cx<T>{x.x * s, x.y * s};
          }
        }
        Stages<T, +1, M, true, 1, 1, false, INV>::run(v, buf, l, j, tw, [&](auto& w) {
          each_output<T, M>(w, j, [&](int p, Cx<T> x) {
            const int q = mode_out_pos(mode, p, M / 2, M);
            if (ok && q >= 0) obase[(int64_t)q * sz] = x;
          });
        });
      });
}

// Sums of three convolutions of one source against one grid, without forming them: with psi and Q
// already transformed along x and y (a.W, a source on nodes -1..n; a.W2, one on nodes 0..n-1), the
// z transforms of a line of each and acc[b] += sum over the line's k_z of
// ghat_b Re(psihat conj(Qhat)), times 2 for the lines that stand for k_x and -k_x too (Parseval).
// gh: three spectra, the stride apart, scaled as for zconv; all even.
template <typename T, int M>
__device__ __forceinline__ void zdot_reg(const FftArgs& a, int64_t gstride, Cx<T>* buf, int blk,
                                         double (&acc)[3]) {
  constexpr int LB = line_count<M>();
  const int Kx = a.nx + 1, My = 2 * a.ny;
  const int lines = Kx * My;
  if (blk * LB >= lines) return;
  int l, j;
  line_pos<M, true>(&l, &j);
  const int g = min(blk * LB + l, lines - 1);
  const int ky = g / Kx, kx = g - ky * Kx;
  const double weight = blk * LB + l < lines ? (kx == 0 || kx == a.nx ? 1.0 : 2.0) : 0.0;
  const int64_t sz = lines;
  const Cx<T>* psi = (const Cx<T>*)a.W + g;
  const Cx<T>* q0 = (const Cx<T>*)a.W2 + g;
  const T* grow = (const T*)a.gh + (int64_t)fold(ky, My) * Kx + kx;
  const int64_t gplane = (int64_t)(a.ny + 1) * Kx;
  const auto* tw = tw_arg<T>(a, 2);
  line_fft<T, -1, M, true, 1>(
      buf, l, j, tw,
      [&](int p) {
        const bool use = mode_src_nonzero(1, p, M / 2, M);
        const Cx<T> v = ld(use ? psi + (int64_t)p * sz : psi);
        return use ? v : Cx<T>{0, 0};
      },
      [&](auto& vp) {
        __syncthreads();  // the second transform's first exchange writes what the first's last read
        line_fft<T, -1, M, true, 1>(
            buf, l, j, tw,
            [&](int p) {
              const bool use = p < M / 2;
              const Cx<T> v = ld(use ? q0 + (int64_t)p * sz : q0);
              return use ? v : Cx<T>{0, 0};
            },
            [&](auto& vq) {
              constexpr int Q = sizeof(vp) / sizeof(vp[0]);
              constexpr int R = sizeof(vp[0]) / sizeof(vp[0][0]);
              constexpr int TPL = line_threads<M>(), NS = M / R;
#pragma unroll
              for (int q = 0; q < Q; ++q) {
                const int jb = j + q * TPL;
                if (jb >= NS) continue;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                  const Cx<T> x = vp[q][r], y = vq[q][r];
                  const double d = weight * ((double)x.x * y.x + (double)x.y * y.y);
                  const T* s = grow + (int64_t)fold(jb + r * NS, M) * gplane;
                  for (int b = 0; b < 3; ++b) acc[b] += (double)s[b * gstride] * d;
                }
              }
            });
      });
  __syncthreads();
}

// see c2r_x_body; H = n_x
template <typename T, int H>
__device__ __forceinline__ void c2r_reg(const FftArgs& a, Cx<T>* buf, int blk) {
  constexpr int LB = line_count<H>(), M = 2 * H;
  const int mode = a.mode;
  const int py = mode_out(mode, a.ny), px = mode_out(mode, H);
  const int rows = py * mode_out(mode, a.nz);
  if (blk * LB >= rows) return;
  int l, j;
  line_pos<H, false>(&l, &j);
  const int row = min(blk * LB + l, rows - 1);
  const bool ok = blk * LB + l < rows;
  const int z = row / py, y = row - z * py;
  const Cx<T>* src = (const Cx<T>*)a.W2 + ((int64_t)z * 2 * a.ny + y) * (H + 1);
  T* dst = (T*)a.dst + (int64_t)row * px;
  const auto* tw = tw_arg<T>(a, 0);
  line_fft<T, +1, H, false, 2>(
      buf, l, j, tw,
      [&](int k) {
        const Cx<T> xk = ld(src + k), xc = cconj(ld(src + (H - k)));
        const auto w = tw[k];
        const Cx<T> d = cmul(Cx<T>{(T)w.x, (T)-w.y}, csub(xk, xc));  // exp(+2 pi i k / M_x)
        return cadd(cadd(xk, xc), Cx<T>{-d.y, d.x});                 // + i d
      },
      [&](auto& v) {
        each_output<T, H>(v, j, [&](int p, Cx<T> x) {
          const int q0 = mode_out_pos(mode, 2 * p, H, M);
          const int q1 = mode_out_pos(mode, 2 * p + 1, H, M);
          if (ok && q0 >= 0) dst[q0] = x.x;
          if (ok && q1 >= 0) dst[q1] = x.y;
        });
      });
}

template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_reg_r2c(FftArgs args, const BeamDev* beams) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const FftArgs a = beam_args<T>(args, beams);
  if (a.g->status) return;
  with_line_length(a.nx, [&](auto len) {
    r2c_reg<T, decltype(len)::value>(a, reinterpret_cast<Cx<T>*>(smem_raw), blockIdx.x);
  });
}
template <typename T, int DIR>
__global__ __launch_bounds__(kFftThreads) void k_reg_y(FftArgs args, const BeamDev* beams) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const FftArgs a = beam_args<T>(args, beams);
  if (a.g->status) return;
  with_line_length(2 * a.ny, [&](auto len) {
    c2c_y_reg<T, decltype(len)::value, DIR>(a, reinterpret_cast<Cx<T>*>(smem_raw), blockIdx.x);
  });
}
template <typename T, bool IMAG>
__global__ __launch_bounds__(kFftThreads) void k_reg_z(FftArgs args, const BeamDev* beams) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const FftArgs a = beam_args<T>(args, beams);
  if (a.g->status) return;
  with_line_length(2 * a.nz, [&](auto len) {
    zconv_reg<T, decltype(len)::value, IMAG>(a, reinterpret_cast<Cx<T>*>(smem_raw), blockIdx.x);
  });
}
// partial[blk 3 + b] = the block's share of the three sums of zdot_reg
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_reg_zdot(FftArgs a, int64_t gstride,
                                                          double* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double sh[kFftThreads / 64][3];
  double acc[3] = {0.0, 0.0, 0.0};
  if (a.g->status == 0)
    with_line_length(2 * a.nz, [&](auto len) {
      constexpr int M = decltype(len)::value;
      const int blocks = ((a.nx + 1) * 2 * a.ny + line_count<M>() - 1) / line_count<M>();
      for (int blk = blockIdx.x; blk < blocks; blk += gridDim.x)
        zdot_reg<T, M>(a, gstride, reinterpret_cast<Cx<T>*>(smem_raw), blk, acc);
    });
  for (int b = 0; b < 3; ++b) {
    for (int off = 32; off > 0; off >>= 1) acc[b] += __shfl_xor(acc[b], off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][b] = acc[b];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int w = 0; w < kFftThreads / 64; ++w) t += sh[w][threadIdx.x];
    partial[blockIdx.x * 3 + threadIdx.x] = t;
  }
}
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_reg_c2r(FftArgs args, const BeamDev* beams) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const FftArgs a = beam_args<T>(args, beams);
  if (a.g->status) return;
  with_line_length(a.nx, [&](auto len) {
    c2r_reg<T, decltype(len)::value>(a, reinterpret_cast<Cx<T>*>(smem_raw), blockIdx.x);
  });
}

// One axis of the kernel spectrum (see green_dft_body): lines of gd along `axis`, two real lines
// per complex one.  gh != nullptr (the last axis): the result times `scale` goes there in the
// grid's precision instead of back into gd.
struct GreenArgs {
  const Geom* g;
  double* gd;
  void* gh;
  double scale;
  int nx, ny, nz;
  int odd;
  const double2* tw;
  int64_t stride;  // several kernels of one grid (blockIdx.y): from one to the next, gd and gh
};

__host__ __device__ __forceinline__ double green_scale(int nx, int ny, int nz) {
  return 1.0 / (4.0 * 3.14159265358979323846 * 8.8541878128e-12 * (8.0 * nx * ny * nz));
}

template <typename T, int M, int AXIS>
__device__ __forceinline__ void green_reg(const GreenArgs& a, Cx<double>* buf, int blk) {
  constexpr int LB = line_count<M>(), n = M / 2;
  constexpr bool LFAST = AXIS != 0;
  const int ex = a.nx + 1, ey = a.ny + 1, ez = a.nz + 1;
  // real lines per plane, planes, element / line / plane strides
  const int na = AXIS == 0 ? ey : (AXIS == 1 ? ex : ex * ey);
  const int planes = AXIS == 2 ? 1 : ez;
  const int64_t st = AXIS == 0 ? 1 : (AXIS == 1 ? ex : (int64_t)ex * ey);
  const int64_t sa = AXIS == 0 ? ex : 1, sb = (int64_t)ex * ey;
  const int ncx = (na + 1) / 2, lines = ncx * planes;
  if (blk * LB >= lines) return;
  int l, j;
  line_pos<M, LFAST>(&l, &j);
  const int g = min(blk * LB + l, lines - 1);
  const bool ok0 = blk * LB + l < lines;
  const int b = AXIS == 2 ? 0 : g / ncx;
  const int c = g - b * ncx;
  const bool ok1 = ok0 && 2 * c + 1 < na;
  const int64_t o0 = b * sb + 2 * (int64_t)c * sa, o1 = 2 * c + 1 < na ? o0 + sa : o0;
  const bool odd = a.odd != 0;
  line_fft<double, -1, M, LFAST, 1>(
      buf, l, j, a.tw,
      [&](int p) {
        const int t = p <= n ? p : M - p;
        const double sgn = odd ? (p < n ? 1.0 : (p == n ? 0.0 : -1.0)) : 1.0;
        return Cx<double>{sgn * a.gd[o0 + t * st], sgn * a.gd[o1 + t * st]};
      },
      [&](auto& v) {
        // in place: the same workgroup has read the line's values by here, all of them before
        // the first exchange
        each_output<double, M>(v, j, [&](int p, Cx<double> x) {
          if (p > n) return;
          const double r0 = odd ? x.y : x.x, r1 = odd ? -x.x : x.y;
          if (a.gh) {
            T* gh = (T*)a.gh;
            if (ok0) gh[o0 + p * st] = (T)(r0 * a.scale);
            if (ok1) gh[o1 + p * st] = (T)(r1 * a.scale);
          } else {
            if (ok0) a.gd[o0 + p * st] = r0;
            if (ok1) a.gd[o1 + p * st] = r1;
          }
        });
      });
}

template <typename T, int AXIS>
__global__ __launch_bounds__(kFftThreads) void k_reg_green(GreenArgs args, const BeamDev* beams) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  GreenArgs a = args;
  if (beams) {
    const BeamDev& d = beams[blockIdx.y];
    a.g = d.geom;
    a.gd = d.Gd;
    a.nx = d.c.nx;
    a.ny = d.c.ny;
    a.nz = d.c.nz;
    a.gh = AXIS == 2 ? d.Gh : nullptr;
    a.scale = green_scale(a.nx, a.ny, a.nz);
    a.odd = 0;
    a.tw = d.plan.tw[AXIS];
  } else if (gridDim.y > 1) {
    a.gd += blockIdx.y * a.stride;
    if (a.gh) a.gh = (T*)a.gh + blockIdx.y * a.stride;
  }
  if (a.g->status) return;
  with_line_length(2 * (AXIS == 0 ? a.nx : (AXIS == 1 ? a.ny : a.nz)), [&](auto len) {
    green_reg<T, decltype(len)::value, AXIS>(a, reinterpret_cast<Cx<double>*>(smem_raw),
                                             blockIdx.x);
  });
}

// ------------------------------------------------------------------------ batched wrappers
// beam = blockIdx.z; lines per workgroup as in shape_for, per beam; blocks beyond a beam's
// extent exit.

__device__ __forceinline__ bool reg_length(int M) {
  return with_line_length(M, [](auto) {});
}

__device__ __forceinline__ int lines_per_block(int L, int lines) {
  int lb = kLdsElems / (L + 1);
  if (lb < 1) lb = 1;
  return lb > lines ? lines : lb;
}

__global__ __launch_bounds__(1024) void k_green_even_dft_batch(const BeamDev* __restrict__ beams,
                                                               int axis) {
  const BeamDev& d = beams[blockIdx.z];
  if (d.geom->status || reg_length(d.plan.full[axis].M)) return;
  const int ex = d.c.nx + 1, ey = d.c.ny + 1, ez = d.c.nz + 1;
  int64_t st, sa, sb;
  int na, nplanes;
  if (axis == 0) {
    st = 1; sa = ex; sb = (int64_t)ex * ey; na = ey; nplanes = ez;
  } else if (axis == 1) {
    st = ex; sa = 1; sb = (int64_t)ex * ey; na = ex; nplanes = ez;
  } else {
    st = (int64_t)ex * ey; sa = 1; sb = 0; na = ex * ey; nplanes = 1;
  }
  const int ncx = (na + 1) / 2;
  const int LB = lines_per_block(d.plan.full[axis].M, ncx);
  if ((int)blockIdx.x >= (ncx + LB - 1) / LB || (int)blockIdx.y >= nplanes) return;
  green_even_dft_body(d.Gd, d.plan.full[axis], d.plan.tw[axis], st, sa, sb, na, LB, blockIdx.x,
                      blockIdx.y, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(256) void k_green_finish_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.y];
  if (reg_length(d.plan.full[2].M)) return;
  const int64_t total = (int64_t)(d.c.nx + 1) * (d.c.ny + 1) * (d.c.nz + 1);
  const double scale = green_scale(d.c.nx, d.c.ny, d.c.nz);
  green_finish_body<T>(d.geom, d.Gd, (T*)d.Gh, total, scale, blockIdx.x, 0, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_r2c_x_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.z];
  if (reg_length(d.plan.half_x.M)) return;
  const int nx = d.c.nx, ny = d.c.ny, nz = d.c.nz;
  const int LB = lines_per_block(d.plan.half_x.M, ny);
  if ((int)blockIdx.x >= (ny + LB - 1) / LB || (int)blockIdx.y >= nz) return;
  r2c_x_body<T, 0>(d.geom, (const T*)d.rho, (Cx<T>*)d.W, d.plan.half_x, tw_of<T>(d.plan, 0), nx,
                   ny, nz, nx + 1, 2 * ny, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

template <typename T, int DIR, int STAGE>
__global__ __launch_bounds__(1024) void k_c2c_y_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.z];
  if (reg_length(d.plan.full[1].M)) return;
  const int Kx = d.c.nx + 1, ny = d.c.ny, nz = d.c.nz;
  const int LB = lines_per_block(d.plan.full[1].M, Kx);
  const int planes = STAGE == 0 ? nz : nz + 2;
  if ((int)blockIdx.x >= (Kx + LB - 1) / LB || (int)blockIdx.y >= planes) return;
  c2c_y_body<T, DIR, 0, STAGE>(d.geom, (Cx<T>*)d.W, d.plan.full[1], tw_of<T>(d.plan, 1), Kx, ny,
                               nz, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_zconv_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.z];
  if (reg_length(d.plan.full[2].M)) return;
  const int Kx = d.c.nx + 1, My = 2 * d.c.ny;
  const int LB = lines_per_block(d.plan.full[2].M, Kx);
  if ((int)blockIdx.x >= (Kx + LB - 1) / LB || (int)blockIdx.y >= My) return;
  zconv_body<T, 0>(d.geom, (Cx<T>*)d.W, (const T*)d.Gh, d.plan.full[2], tw_of<T>(d.plan, 2), Kx,
                   My, d.c.ny, d.c.nz, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_c2r_x_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.z];
  if (reg_length(d.plan.half_x.M)) return;
  const int nx = d.c.nx, ny = d.c.ny, nz = d.c.nz;
  const int LB = lines_per_block(d.plan.half_x.M, ny + 2);
  if ((int)blockIdx.x >= (ny + 2 + LB - 1) / LB || (int)blockIdx.y >= nz + 2) return;
  c2r_x_body<T, 0>(d.geom, (const Cx<T>*)d.W, (T*)d.phi, d.plan.half_x, tw_of<T>(d.plan, 0), nx,
                   ny, nx + 1, 2 * ny, LB, blockIdx.x, blockIdx.y, gridDim.x);
}

__global__ void k_twiddles(double2* tw, float2* twf, int M) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= M) return;
  double s, c;
  sincospi(2.0 * (double)t / (double)M, &s, &c);
  tw[t] = make_double2(c, -s);
  twf[t] = make_float2((float)c, (float)-s);
}

int grid_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 16384) b = 16384;
  return (int)(b < 1 ? 1 : b);
}

// lines per workgroup and threads for transforms of length L over `lines` lines
void shape_for(int L, int lines, int* LB, int* NT) {
  int lb = kLdsElems / (L + 1);
  if (lb < 1) lb = 1;
  if (lb > lines) lb = lines;
  int nt = (lb * L + 3) / 4;
  nt = ((nt + 63) / 64) * 64;
  if (nt > 1024) nt = 1024;
  if (nt < 64) nt = 64;
  *LB = lb;
  *NT = nt;
}

template <typename T>
const typename TwT<T>::type* table(const FftPlan& p, int a);
template <>
const double2* table<double>(const FftPlan& p, int a) { return p.tw[a]; }
template <>
const float2* table<float>(const FftPlan& p, int a) { return p.twf[a]; }

}  // namespace

hipError_t launch_twiddles(double2* tw, float2* twf, int M, hipStream_t s) {
  hipLaunchKernelGGL(k_twiddles, dim3((M + 255) / 256), dim3(256), 0, s, tw, twf, M);
  return hipGetLastError();
}

namespace {
// launch shape of the register transforms of a length: lines per workgroup and LDS; false if
// the length has none
template <typename T>
bool reg_shape(int M, bool lfast, int* lb, size_t* lds) {
  return with_line_length(M, [&](auto len) {
    constexpr int V = decltype(len)::value;
    *lb = line_count<V>();
    *lds = sizeof(Cx<T>) * (size_t)(lfast ? lds_elems<V, true>() : lds_elems<V, false>());
  });
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// real lines per plane and planes of one axis of an octant array
void green_lines(int axis, int nx, int ny, int nz, int* na, int* planes) {
  const int ex = nx + 1, ey = ny + 1, ez = nz + 1;
  *na = axis == 0 ? ey : (axis == 1 ? ex : ex * ey);
  *planes = axis == 2 ? 1 : ez;
}

template <typename T>
void launch_reg_green(int axis, dim3 grid, size_t lds, const GreenArgs& a, const BeamDev* beams,
                      hipStream_t s) {
  const dim3 nt(kFftThreads);
  if (axis == 0)
    hipLaunchKernelGGL((k_reg_green<double, 0>), grid, nt, lds, s, a, beams);
  else if (axis == 1)
    hipLaunchKernelGGL((k_reg_green<double, 1>), grid, nt, lds, s, a, beams);
  else
    hipLaunchKernelGGL((k_reg_green<T, 2>), grid, nt, lds, s, a, beams);
}

// One DFT pass of an octant kernel with the runtime-length engine
template <typename T>
hipError_t kernel_spectrum_axis(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                double* gd, T* gh, int a, bool odd, hipStream_t s) {
  const int ex = nx + 1, ey = ny + 1, ez = nz + 1;
  int na, planes, LB, NT;
  green_lines(a, nx, ny, nz, &na, &planes);
  const int ncx = (na + 1) / 2;
  // (element stride, line stride a, plane stride b)
  const int64_t cfg[3][3] = {{1, ex, (int64_t)ex * ey},
                             {ex, 1, (int64_t)ex * ey},
                             {(int64_t)ex * ey, 1, 0}};
  shape_for(p.full[a].M, ncx, &LB, &NT);
  const dim3 grid(ceil_div(ncx, LB), planes);
  const size_t lds = (size_t)LB * (p.full[a].M + 1) * sizeof(Cx<double>) +
                     (size_t)p.full[a].M * sizeof(double2);
  if (odd)
    hipLaunchKernelGGL(k_green_dft<true>, grid, dim3(NT), lds, s, gd, p.full[a], p.tw[a],
                       cfg[a][0], cfg[a][1], cfg[a][2], na, LB);
  else
    hipLaunchKernelGGL(k_green_dft<false>, grid, dim3(NT), lds, s, gd, p.full[a], p.tw[a],
                       cfg[a][0], cfg[a][1], cfg[a][2], na, LB);
  PIC_TRY(hipGetLastError());
  if (a == 2) {
    const int64_t total = (int64_t)ex * ey * ez;
    hipLaunchKernelGGL((k_green_finish<T>), dim3(grid_for(total)), dim3(256), 0, s, g, gd, gh,
                       total, green_scale(nx, ny, nz));
  }
  return hipGetLastError();
}

// The three even/odd DFT passes of `count` octant kernels gd, consecutive (odd_axis: -1 for even
// kernels), and the scaled conversion into gh.  The register transforms take all of them in one
// launch per axis: one kernel's lines of a 64^3 grid fill a third of the chip, and its three
// h-derivatives' nine launches of 6.5 us became three of 9 us.
template <typename T>
hipError_t kernel_spectrum(const Geom* g, const FftPlan& p, int nx, int ny, int nz, double* gd,
                           T* gh, int odd_axis, hipStream_t s, int count = 1) {
  const int ex = nx + 1, ey = ny + 1, ez = nz + 1;
  const double scale = green_scale(nx, ny, nz);
  const int64_t total = (int64_t)ex * ey * ez;
  for (int a = 0; a < 3; ++a) {
    int na, planes, LB;
    green_lines(a, nx, ny, nz, &na, &planes);
    const int ncx = (na + 1) / 2;  // complex lines (two real lines each)
    size_t lds;
    if (reg_shape<double>(p.full[a].M, a != 0, &LB, &lds)) {
      const GreenArgs ga{g,  gd, a == 2 ? (void*)gh : nullptr, scale, nx, ny, nz, a == odd_axis,
                         p.tw[a], total};
      launch_reg_green<T>(a, dim3(ceil_div(ncx * planes, LB), count), lds, ga, nullptr, s);
      PIC_TRY(hipGetLastError());
      continue;
    }
    for (int q = 0; q < count; ++q)
      PIC_TRY(kernel_spectrum_axis<T>(g, p, nx, ny, nz, gd + q * total, gh + q * total, a,
                                      a == odd_axis, s));
  }
  return hipSuccess;
}
}  // namespace

template <typename T>
hipError_t launch_green_field_spectrum(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                       double2* hcorners, double* gd3, T* gh3, hipStream_t s) {
  PIC_TRY(launch_igf_field(g, nx, ny, nz, hcorners, gd3, s));
  const int64_t total = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
  for (int a = 0; a < 3; ++a)
    PIC_TRY(kernel_spectrum<T>(g, p, nx, ny, nz, gd3 + a * total, gh3 + a * total, a, s));
  return hipSuccess;
}

template <typename T>
hipError_t launch_green_dh_spectra(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                   bool field, double2* dc, double* gd, T* gh, hipStream_t s) {
  PIC_TRY(launch_igf_dh(g, nx, ny, nz, field, dc, gd, s));
  if (!field) return kernel_spectrum<T>(g, p, nx, ny, nz, gd, gh, -1, s, 3);
  const int64_t total = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
  // kernel (a, b) = f = 3 a + b in gd; its spectrum at 3 b + a, so that the three of one b
  // are consecutive, as the transposed field solve reads them
  for (int f = 0; f < 9; ++f)
    PIC_TRY(kernel_spectrum<T>(g, p, nx, ny, nz, gd + f * total,
                               gh + (3 * (f % 3) + f / 3) * total, f / 3, s));
  return hipSuccess;
}

template <typename T>
hipError_t launch_green_spectrum(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                 double2* corners, double* gd, T* gh, hipStream_t s) {
  PIC_TRY(launch_igf_corners(g, nx, ny, nz, corners, s));
  PIC_TRY(launch_igf_cells(g, nx, ny, nz, corners, gd, s));
  return kernel_spectrum<T>(g, p, nx, ny, nz, gd, gh, -1, s);
}


namespace {

// The passes of a solve, each with the register transforms where its line length has them and
// the runtime-length engine elsewhere (modes as in MODE; 1 and 2 keep the same outputs, 0 and 2
// read the same inputs).
template <typename T>
hipError_t pass_r2c(const FftArgs& a, const FftPlan& p, hipStream_t s) {
  const int rows_y = mode_src(a.mode, a.ny), rows_z = mode_src(a.mode, a.nz);
  int LB, NT;
  size_t lds;
  if (reg_shape<T>(a.nx, false, &LB, &lds)) {
    hipLaunchKernelGGL((k_reg_r2c<T>), dim3(ceil_div(rows_y * rows_z, LB)), dim3(kFftThreads),
                       lds, s, a, nullptr);
    return hipGetLastError();
  }
  shape_for(p.half_x.M, rows_y, &LB, &NT);
  lds = (size_t)LB * (p.half_x.M + 1) * sizeof(Cx<T>) +
        (size_t)p.full[0].M * sizeof(typename TwT<T>::type);
  const dim3 grid(ceil_div(rows_y, LB), rows_z);
  if (a.mode == 1)
    hipLaunchKernelGGL((k_r2c_x<T, 1>), grid, dim3(NT), lds, s, a.g, (const T*)a.src, (Cx<T>*)a.W,
                       p.half_x, table<T>(p, 0), a.nx, a.ny, a.nz, a.nx + 1, 2 * a.ny, LB);
  else
    hipLaunchKernelGGL((k_r2c_x<T, 0>), grid, dim3(NT), lds, s, a.g, (const T*)a.src, (Cx<T>*)a.W,
                       p.half_x, table<T>(p, 0), a.nx, a.ny, a.nz, a.nx + 1, 2 * a.ny, LB);
  return hipGetLastError();
}

template <typename T, int DIR>
hipError_t pass_y(const FftArgs& a, const FftPlan& p, hipStream_t s) {
  const int Kx = a.nx + 1;
  const int planes = DIR < 0 ? mode_src(a.mode, a.nz) : mode_out(a.mode, a.nz);
  int LB, NT;
  size_t lds;
  if (reg_shape<T>(2 * a.ny, true, &LB, &lds)) {
    hipLaunchKernelGGL((k_reg_y<T, DIR>), dim3(ceil_div(Kx * planes, LB)), dim3(kFftThreads), lds,
                       s, a, nullptr);
    return hipGetLastError();
  }
  shape_for(p.full[1].M, Kx, &LB, &NT);
  lds = (size_t)LB * (p.full[1].M + 1) * sizeof(Cx<T>) +
        (size_t)p.full[1].M * sizeof(typename TwT<T>::type);
  const dim3 grid(ceil_div(Kx, LB), planes);
  Cx<T>* W = (Cx<T>*)(DIR < 0 ? a.W : a.W2);
  constexpr int STAGE = DIR < 0 ? 0 : 1;
  if ((DIR < 0 && a.mode == 1) || (DIR > 0 && a.mode != 0))
    hipLaunchKernelGGL((k_c2c_y<T, DIR, 1, STAGE>), grid, dim3(NT), lds, s, a.g, W, p.full[1],
                       table<T>(p, 1), Kx, a.ny, a.nz, LB);
  else
    hipLaunchKernelGGL((k_c2c_y<T, DIR, 0, STAGE>), grid, dim3(NT), lds, s, a.g, W, p.full[1],
                       table<T>(p, 1), Kx, a.ny, a.nz, LB);
  return hipGetLastError();
}

template <typename T>
hipError_t pass_z(const FftArgs& a, const FftPlan& p, hipStream_t s) {
  const int Kx = a.nx + 1, My = 2 * a.ny;
  int LB, NT;
  size_t lds;
  if (reg_shape<T>(2 * a.nz, true, &LB, &lds)) {
    const dim3 grid(ceil_div(Kx * My, LB));
    if (a.odd >= 0)
      hipLaunchKernelGGL((k_reg_z<T, true>), grid, dim3(kFftThreads), lds, s, a, nullptr);
    else
      hipLaunchKernelGGL((k_reg_z<T, false>), grid, dim3(kFftThreads), lds, s, a, nullptr);
    return hipGetLastError();
  }
  shape_for(p.full[2].M, Kx, &LB, &NT);
  lds = (size_t)LB * (p.full[2].M + 1) * sizeof(Cx<T>) +
        (size_t)p.full[2].M * sizeof(typename TwT<T>::type);
  const dim3 grid(ceil_div(Kx, LB), My);
  Cx<T>* W = (Cx<T>*)a.W;
  const T* gh = (const T*)a.gh;
  if (a.odd >= 0)
    hipLaunchKernelGGL((k_zconv_field<T>), grid, dim3(NT), lds, s, a.g, W, gh, p.full[2],
                       table<T>(p, 2), Kx, My, a.ny, a.nz, LB, (Cx<T>*)a.W2, a.odd);
  else if (a.mode == 1)
    hipLaunchKernelGGL((k_zconv<T, 1>), grid, dim3(NT), lds, s, a.g, W, gh, p.full[2],
                       table<T>(p, 2), Kx, My, a.ny, a.nz, LB);
  else
    hipLaunchKernelGGL((k_zconv<T, 0>), grid, dim3(NT), lds, s, a.g, W, gh, p.full[2],
                       table<T>(p, 2), Kx, My, a.ny, a.nz, LB);
  return hipGetLastError();
}

template <typename T>
hipError_t pass_c2r(const FftArgs& a, const FftPlan& p, hipStream_t s) {
  const int out_y = mode_out(a.mode, a.ny), out_z = mode_out(a.mode, a.nz);
  int LB, NT;
  size_t lds;
  if (reg_shape<T>(a.nx, false, &LB, &lds)) {
    hipLaunchKernelGGL((k_reg_c2r<T>), dim3(ceil_div(out_y * out_z, LB)), dim3(kFftThreads), lds,
                       s, a, nullptr);
    return hipGetLastError();
  }
  shape_for(p.half_x.M, out_y, &LB, &NT);
  lds = (size_t)LB * (p.half_x.M + 1) * sizeof(Cx<T>) +
        (size_t)p.full[0].M * sizeof(typename TwT<T>::type);
  const dim3 grid(ceil_div(out_y, LB), out_z);
  if (a.mode == 0)
    hipLaunchKernelGGL((k_c2r_x<T, 0>), grid, dim3(NT), lds, s, a.g, (const Cx<T>*)a.W2,
                       (T*)a.dst, p.half_x, table<T>(p, 0), a.nx, a.ny, a.nx + 1, 2 * a.ny, LB);
  else
    hipLaunchKernelGGL((k_c2r_x<T, 1>), grid, dim3(NT), lds, s, a.g, (const Cx<T>*)a.W2,
                       (T*)a.dst, p.half_x, table<T>(p, 0), a.nx, a.ny, a.nx + 1, 2 * a.ny, LB);
  return hipGetLastError();
}

template <typename T>
FftArgs fft_args(const Geom* g, const FftPlan& p, int nx, int ny, int nz, int mode, void* W,
                 void* W2) {
  return FftArgs{g, nx, ny, nz, mode, -1, nullptr, W, W2, nullptr, nullptr,
                 {table<T>(p, 0), table<T>(p, 1), table<T>(p, 2)}};
}

// mode 0: phi (nodes -1..n) from rho (nodes 0..n-1); mode 1: chi (nodes 0..n-1) from a source
// on nodes -1..n.  src/dst layouts as in k_r2c_x and k_c2r_x.
template <typename T>
hipError_t run_passes(const Geom* g, const FftPlan& p, int nx, int ny, int nz, int mode,
                      const T* src, void* W, const T* gh, T* dst, hipStream_t s) {
  FftArgs a = fft_args<T>(g, p, nx, ny, nz, mode, W, W);
  a.src = src;
  a.gh = gh;
  a.dst = dst;
  PIC_TRY(pass_r2c<T>(a, p, s));
  PIC_TRY((pass_y<T, -1>(a, p, s)));
  PIC_TRY(pass_z<T>(a, p, s));
  PIC_TRY((pass_y<T, +1>(a, p, s)));
  return pass_c2r<T>(a, p, s);
}

// one field component's convolution: the z pass of W with i Khat_a (odd along axis a) into W2
// and the inverse y and x passes into dst (nodes 0..n-1)
template <typename T>
hipError_t field_component(FftArgs a, const FftPlan& p, int axis, const T* gh, T* dst,
                           hipStream_t s) {
  a.odd = axis;
  a.gh = gh;
  a.dst = dst;
  PIC_TRY(pass_z<T>(a, p, s));
  PIC_TRY((pass_y<T, +1>(a, p, s)));
  return pass_c2r<T>(a, p, s);
}

}  // namespace

template <typename T>
hipError_t launch_solve(const Geom* g, const FftPlan& p, int nx, int ny, int nz, const T* rho,
                        void* Wv, const T* gh, T* phi, T* E, hipStream_t s) {
  PIC_TRY(run_passes<T>(g, p, nx, ny, nz, 0, rho, Wv, gh, phi, s));
  if (!E) return hipSuccess;  // the gather-kick differences phi itself
  const int64_t ng = (int64_t)nx * ny * nz;
  hipLaunchKernelGGL((k_grad<T>), dim3(grid_for(ng)), dim3(256), 0, s, g, phi, E, nx, ny, nz);
  return hipGetLastError();
}

// Direct field: forward x and y passes of rho into W, then per component the z pass with the
// product by i Ghat_a into W2 and the inverse y and x passes into E_a (nodes 0..n-1).
template <typename T>
hipError_t launch_solve_field(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                              const T* rho, void* Wv, void* W2v, const T* gh3, T* E,
                              hipStream_t s) {
  const int64_t ng = (int64_t)nx * ny * nz, gtot = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
  FftArgs a = fft_args<T>(g, p, nx, ny, nz, 2, Wv, W2v);
  a.src = rho;
  PIC_TRY(pass_r2c<T>(a, p, s));
  PIC_TRY((pass_y<T, -1>(a, p, s)));
  for (int q = 0; q < 3; ++q)
    PIC_TRY(field_component<T>(a, p, q, gh3 + q * gtot, E + q * ng, s));
  return hipSuccess;
}

namespace {
// chi = -(t_0 + t_1 + t_2) over the nodes
template <typename T>
__global__ __launch_bounds__(256) void k_neg_sum3(const Geom* __restrict__ g,
                                                  const T* __restrict__ t, int64_t ng,
                                                  T* __restrict__ chi) {
  if (g->status) return;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < ng; i += (int64_t)gridDim.x * 256)
    chi[i] = -(t[i] + t[ng + i] + t[2 * ng + i]);
}
}  // namespace

// Transpose of launch_solve_field: chi = -sum_a (Kbar_a * e_a) / (4 pi eps0), each a full
// zero-padded convolution (forward x and y passes of e_a, the z pass with i Khat_a, the inverse
// y and x passes onto nodes 0..n-1) into tmp (3 nx ny nz), then the signed sum.
template <typename T>
hipError_t launch_solve_field_T(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                const T* e, void* Wv, void* W2v, const T* gh3, T* tmp, T* chi,
                                hipStream_t s) {
  const int64_t ng = (int64_t)nx * ny * nz, gtot = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
  FftArgs a = fft_args<T>(g, p, nx, ny, nz, 2, Wv, W2v);
  for (int q = 0; q < 3; ++q) {
    a.src = e + q * ng;
    PIC_TRY(pass_r2c<T>(a, p, s));
    PIC_TRY((pass_y<T, -1>(a, p, s)));
    PIC_TRY(field_component<T>(a, p, q, gh3 + q * gtot, tmp + q * ng, s));
  }
  int64_t nbk = (ng + 255) / 256;
  if (nbk > 16384) nbk = 16384;
  hipLaunchKernelGGL((k_neg_sum3<T>), dim3((unsigned)nbk), dim3(256), 0, s, g, tmp, ng, chi);
  return hipGetLastError();
}

template hipError_t launch_solve_field_T<double>(const Geom*, const FftPlan&, int, int, int,
                                                 const double*, void*, void*, const double*,
                                                 double*, double*, hipStream_t);
template hipError_t launch_solve_field_T<float>(const Geom*, const FftPlan&, int, int, int,
                                                const float*, void*, void*, const float*,
                                                float*, float*, hipStream_t);

template hipError_t launch_solve_field<double>(const Geom*, const FftPlan&, int, int, int,
                                               const double*, void*, void*, const double*,
                                               double*, hipStream_t);
template hipError_t launch_solve_field<float>(const Geom*, const FftPlan&, int, int, int,
                                              const float*, void*, void*, const float*, float*,
                                              hipStream_t);
template hipError_t launch_green_field_spectrum<double>(const Geom*, const FftPlan&, int, int,
                                                        int, double2*, double*, double*,
                                                        hipStream_t);
template hipError_t launch_green_field_spectrum<float>(const Geom*, const FftPlan&, int, int, int,
                                                       double2*, double*, float*, hipStream_t);

template <typename T>
hipError_t launch_solve_ghost_source(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                     const T* psi, void* Wv, const T* gh, T* chi, hipStream_t s) {
  return run_passes<T>(g, p, nx, ny, nz, 1, psi, Wv, gh, chi, s);
}

// The x and y passes of the charge grid Q into WQ, for launch_solve_ghost_dots.  *done = false and
// nothing run: no register transforms for this length along z.
template <typename T>
hipError_t launch_charge_spectrum(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                  const T* Q, void* WQ, bool* done, hipStream_t s) {
  int LB;
  size_t lds;
  *done = reg_shape<T>(2 * nz, true, &LB, &lds);
  if (!*done) return hipSuccess;
  FftArgs q = fft_args<T>(g, p, nx, ny, nz, 0, WQ, WQ);
  q.src = Q;
  PIC_TRY(pass_r2c<T>(q, p, s));
  return pass_y<T, -1>(q, p, s);
}

// launch_solve_ghost_source, and the geometry sums' partials: partial[b 3 + c] (b < *nparts) adds
// up to sum_n Q_n (dG_c * psi)_n over nodes 0..n-1 for the three spectra dgh (as gh, consecutive)
// and Q's x and y transform WQ.  psi's transform is shared, and no convolution with dgh is formed:
// the sums are taken over the spectra (zdot_reg).  At 64^3 in float64 three convolutions and grid
// dots took 146 us, Q's transforms and the sums take 38 (the sums 24, bound by their registers: two
// lines are live, one wave per SIMD).  WQ == nullptr: *nparts = 0, no sums.
template <typename T>
hipError_t launch_solve_ghost_dots(const Geom* g, const FftPlan& p, int nx, int ny, int nz,
                                   const T* psi, void* Wv, const T* gh, T* chi, const void* WQ,
                                   const T* dgh, double* partial, int max_parts, int* nparts,
                                   hipStream_t s) {
  *nparts = 0;
  int LB;
  size_t lds;
  if (!WQ || !reg_shape<T>(2 * nz, true, &LB, &lds))
    return launch_solve_ghost_source<T>(g, p, nx, ny, nz, psi, Wv, gh, chi, s);
  FftArgs a = fft_args<T>(g, p, nx, ny, nz, 1, Wv, Wv);
  a.src = psi;
  a.gh = gh;
  a.dst = chi;
  PIC_TRY(pass_r2c<T>(a, p, s));
  PIC_TRY((pass_y<T, -1>(a, p, s)));
  FftArgs d = a;
  d.W2 = const_cast<void*>(WQ);  // read only
  d.gh = dgh;
  const int nb = std::min(ceil_div((nx + 1) * 2 * ny, LB), max_parts);
  hipLaunchKernelGGL((k_reg_zdot<T>), dim3(nb), dim3(kFftThreads), lds, s, d,
                     (int64_t)(nx + 1) * (ny + 1) * (nz + 1), partial);
  PIC_TRY(hipGetLastError());
  *nparts = nb;
  PIC_TRY(pass_z<T>(a, p, s));
  PIC_TRY((pass_y<T, +1>(a, p, s)));
  return pass_c2r<T>(a, p, s);
}

template hipError_t launch_solve_ghost_dots<double>(const Geom*, const FftPlan&, int, int, int,
                                                    const double*, void*, const double*, double*,
                                                    const void*, const double*, double*, int,
                                                    int*, hipStream_t);
template hipError_t launch_solve_ghost_dots<float>(const Geom*, const FftPlan&, int, int, int,
                                                   const float*, void*, const float*, float*,
                                                   const void*, const float*, double*, int, int*,
                                                   hipStream_t);
template hipError_t launch_charge_spectrum<double>(const Geom*, const FftPlan&, int, int, int,
                                                   const double*, void*, bool*, hipStream_t);
template hipError_t launch_charge_spectrum<float>(const Geom*, const FftPlan&, int, int, int,
                                                  const float*, void*, bool*, hipStream_t);
template hipError_t launch_solve_ghost_source<double>(const Geom*, const FftPlan&, int, int, int,
                                                      const double*, void*, const double*,
                                                      double*, hipStream_t);
template hipError_t launch_solve_ghost_source<float>(const Geom*, const FftPlan&, int, int, int,
                                                     const float*, void*, const float*, float*,
                                                     hipStream_t);
// ------------------------------------------------------------------------ batched launches

namespace {
int lpb(int L, int lines) {
  int lb = kLdsElems / (L + 1);
  if (lb < 1) lb = 1;
  return lb > lines ? lines : lb;
}
// what one beam's lines of length M need of a pass: workgroups and LDS of the register
// transforms, or the runtime-length engine
template <typename T>
void add_pass(BatchPass* bp, int M, bool lfast, int lines) {
  int lb;
  size_t lds;
  if (!reg_shape<T>(M, lfast, &lb, &lds)) {
    bp->generic = true;
    return;
  }
  bp->blocks = std::max(bp->blocks, ceil_div(lines, lb));
  bp->lds = std::max(bp->lds, lds);
}
template <typename T>
void add_beam(BatchDims* bd, int nx, int ny, int nz) {
  const int Kx = nx + 1;
  add_pass<T>(&bd->r2c, nx, false, ny * nz);
  add_pass<T>(&bd->yf, 2 * ny, true, Kx * nz);
  add_pass<T>(&bd->z, 2 * nz, true, Kx * 2 * ny);
  add_pass<T>(&bd->yi, 2 * ny, true, Kx * (nz + 2));
  add_pass<T>(&bd->c2r, nx, false, (ny + 2) * (nz + 2));
  const int M[3] = {2 * nx, 2 * ny, 2 * nz};
  for (int a = 0; a < 3; ++a) {
    int na, planes;
    green_lines(a, nx, ny, nz, &na, &planes);
    add_pass<double>(&bd->green[a], M[a], a != 0, (na + 1) / 2 * planes);
  }
}
}  // namespace

void batch_fft_dims(BatchDims* bd, int nx, int ny, int nz, bool fp32) {
  if (fp32)
    add_beam<float>(bd, nx, ny, nz);
  else
    add_beam<double>(bd, nx, ny, nz);
}

// Every pass: the register transforms for the beams whose line length has them (the others'
// workgroups exit), and the runtime-length engine if the batch has other beams.
template <typename T>
hipError_t launch_batch_green(const BeamDev* beams, int nb, const BatchDims& bd, hipStream_t s) {
  PIC_TRY(launch_batch_igf(beams, nb, bd.max_nx, bd.max_ny, bd.max_nz, s));
  const int ex = bd.max_nx + 1, ey = bd.max_ny + 1, ez = bd.max_nz + 1;
  // grid extents over the beams: the largest grid needs the most blocks along every axis
  const int M[3] = {2 * bd.max_nx, 2 * bd.max_ny, 2 * bd.max_nz};
  for (int a = 0; a < 3; ++a) {
    if (bd.green[a].blocks) {
      launch_reg_green<T>(a, dim3(bd.green[a].blocks, nb), bd.green[a].lds, GreenArgs{}, beams, s);
      PIC_TRY(hipGetLastError());
    }
    if (!bd.green[a].generic) continue;
    // smaller beams have shorter lines and so at least as many lines per block: the largest
    // beam bounds the block count
    int na, planes;
    green_lines(a, bd.max_nx, bd.max_ny, bd.max_nz, &na, &planes);
    const int ncx = (na + 1) / 2;
    const int gx = ceil_div(ncx, lpb(M[a], ncx));
    hipLaunchKernelGGL(k_green_even_dft_batch, dim3(gx, planes, nb), dim3(1024),
                       (size_t)kLdsElems * sizeof(Cx<double>) + 512 * sizeof(double2), s, beams,
                       a);
    PIC_TRY(hipGetLastError());
  }
  if (!bd.green[2].generic) return hipSuccess;
  const int64_t total = (int64_t)ex * ey * ez;
  hipLaunchKernelGGL((k_green_finish_batch<T>), dim3(grid_for(total), nb), dim3(256), 0, s, beams);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_solve(const BeamDev* beams, int nb, const BatchDims& bd, hipStream_t s) {
  const int nx = bd.max_nx, ny = bd.max_ny, nz = bd.max_nz;
  const int Kx = nx + 1, My = 2 * ny;
  // lines plus a twiddle table of at most 512 entries (2 n <= 512)
  const size_t lds = (size_t)kLdsElems * sizeof(Cx<T>) + 512 * sizeof(typename TwT<T>::type);
  const FftArgs none{};
  const dim3 nt(kFftThreads);
  if (bd.r2c.blocks)
    hipLaunchKernelGGL((k_reg_r2c<T>), dim3(bd.r2c.blocks, nb), nt, bd.r2c.lds, s, none, beams);
  if (bd.r2c.generic)
    hipLaunchKernelGGL((k_r2c_x_batch<T>), dim3(ceil_div(ny, lpb(nx, ny)), nz, nb), dim3(1024),
                       lds, s, beams);
  PIC_TRY(hipGetLastError());
  if (bd.yf.blocks)
    hipLaunchKernelGGL((k_reg_y<T, -1>), dim3(bd.yf.blocks, nb), nt, bd.yf.lds, s, none, beams);
  if (bd.yf.generic)
    hipLaunchKernelGGL((k_c2c_y_batch<T, -1, 0>), dim3(ceil_div(Kx, lpb(My, Kx)), nz, nb),
                       dim3(1024), lds, s, beams);
  PIC_TRY(hipGetLastError());
  if (bd.z.blocks)
    hipLaunchKernelGGL((k_reg_z<T, false>), dim3(bd.z.blocks, nb), nt, bd.z.lds, s, none, beams);
  if (bd.z.generic)
    hipLaunchKernelGGL((k_zconv_batch<T>), dim3(ceil_div(Kx, lpb(2 * nz, Kx)), My, nb),
                       dim3(1024), lds, s, beams);
  PIC_TRY(hipGetLastError());
  if (bd.yi.blocks)
    hipLaunchKernelGGL((k_reg_y<T, +1>), dim3(bd.yi.blocks, nb), nt, bd.yi.lds, s, none, beams);
  if (bd.yi.generic)
    hipLaunchKernelGGL((k_c2c_y_batch<T, +1, 1>), dim3(ceil_div(Kx, lpb(My, Kx)), nz + 2, nb),
                       dim3(1024), lds, s, beams);
  PIC_TRY(hipGetLastError());
  if (bd.c2r.blocks)
    hipLaunchKernelGGL((k_reg_c2r<T>), dim3(bd.c2r.blocks, nb), nt, bd.c2r.lds, s, none, beams);
  if (bd.c2r.generic)
    hipLaunchKernelGGL((k_c2r_x_batch<T>), dim3(ceil_div(ny + 2, lpb(nx, ny + 2)), nz + 2, nb),
                       dim3(1024), lds, s, beams);
  return hipGetLastError();
}

template hipError_t launch_batch_green<double>(const BeamDev*, int, const BatchDims&, hipStream_t);
template hipError_t launch_batch_green<float>(const BeamDev*, int, const BatchDims&, hipStream_t);
template hipError_t launch_batch_solve<double>(const BeamDev*, int, const BatchDims&, hipStream_t);
template hipError_t launch_batch_solve<float>(const BeamDev*, int, const BatchDims&, hipStream_t);

template hipError_t launch_green_spectrum<double>(const Geom*, const FftPlan&, int, int, int,
                                                  double2*, double*, double*, hipStream_t);
template hipError_t launch_green_dh_spectra<double>(const Geom*, const FftPlan&, int, int, int,
                                                    bool, double2*, double*, double*, hipStream_t);
template hipError_t launch_green_dh_spectra<float>(const Geom*, const FftPlan&, int, int, int,
                                                   bool, double2*, double*, float*, hipStream_t);
template hipError_t launch_green_spectrum<float>(const Geom*, const FftPlan&, int, int, int,
                                                 double2*, double*, float*, hipStream_t);
template hipError_t launch_solve<double>(const Geom*, const FftPlan&, int, int, int,
                                         const double*, void*, const double*, double*, double*,
                                         hipStream_t);
template hipError_t launch_solve<float>(const Geom*, const FftPlan&, int, int, int, const float*,
                                        void*, const float*, float*, float*, hipStream_t);

}  // namespace pic
