// 3-D solid harmonic scattering (paper section 2: wavelets psi_{j,l,m}, non-linearity
// rho = sqrt(sum_m |x conv psi_{j,l,m}|^2)), evaluated as the definition states it: every
// convolution on the full periodic grid through 3-D FFTs, the lowpassed result read at
// the samples 2^J n.  A 3-D transform is three passes of the plain in-place transforms of
// the backward pass (last axis as rows, the other two as columns); the pointwise steps
// are the small kernels below.
#include <hip/hip_runtime.h>

#include <string>

#include "fft_regs.hpp"
#include "pad.hpp"
#include "slab_fft.hpp"
#include "scat_kernels.hpp"

namespace scat {

namespace {

int ilog2h(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

unsigned blocks_for(long total) {
  long b = (total + 255) / 256;
  if (b > 65536 * 16) b = 65536 * 16;
  return static_cast<unsigned>(b < 1 ? 1 : b);
}

__global__ __launch_bounds__(256) void k3_real_to_complex(const float *__restrict__ x,
                                                          float2 *__restrict__ out, long total) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride)
    out[i] = make_float2(x[i], 0.f);
}

// dst[v][e] (+)= src[v][e] * filt[e]: one real table applied to every volume of the batch
__global__ __launch_bounds__(256) void k3_mul_table(const float2 *__restrict__ src,
                                                    const float *__restrict__ filt,
                                                    float2 *__restrict__ dst, long total, long n,
                                                    int accumulate) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const float f = filt[i % n];
    const float2 v = src[i];
    float2 o = make_float2(v.x * f, v.y * f);
    if (accumulate) {
      const float2 d = dst[i];
      o.x += d.x;
      o.y += d.y;
    }
    dst[i] = o;
  }
}

// dst[v][k] (+)= phi[k] * Gs[v][chan][k mod m]: the spectrum of the zero-inserted output
// gradient is the small spectrum Gs tiled over the grid (adjoint of lowpass + subsampling)
__global__ __launch_bounds__(256) void k3_tile_phi(const float2 *__restrict__ Gs,
                                                   const float *__restrict__ phi,
                                                   float2 *__restrict__ dst, long volumes, int K,
                                                   int chan, int n0, int n1, int n2, int J,
                                                   int accumulate) {
  const long per = static_cast<long>(n0) * n1 * n2;
  const long total = volumes * per;
  const int m0 = n0 >> J, m1 = n1 >> J, m2 = n2 >> J;
  const long mper = static_cast<long>(m0) * m1 * m2;
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const long v = i / per;
    long e = i - v * per;
    const int c = static_cast<int>(e % n2);
    const long e1 = e / n2;
    const int b = static_cast<int>(e1 % n1);
    const int a = static_cast<int>(e1 / n1);
    const float2 gs = Gs[(static_cast<size_t>(v) * K + chan) * mper +
                         (static_cast<size_t>(a & (m0 - 1)) * m1 + (b & (m1 - 1))) * m2 + (c & (m2 - 1))];
    const float f = phi[e];
    float2 o = make_float2(gs.x * f, gs.y * f);
    if (accumulate) {
      const float2 d = dst[i];
      o.x += d.x;
      o.y += d.y;
    }
    dst[i] = o;
  }
}

// y[i] <- Re(gu[i]) * y[i] / sqrt(acc[i])  (0 where acc = sum_m |y_m|^2 vanishes): the
// gradient of rho = sqrt(sum_m |y_m|^2) with respect to y_m, given the gradient of rho
__global__ __launch_bounds__(256) void k3_rho_back(const float2 *__restrict__ gu,
                                                   const float *__restrict__ acc,
                                                   float2 *__restrict__ y, long total) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const float a = acc[i];
    const float s = over_sqrt(gu[i].x, a);
    const float2 v = y[i];
    y[i] = make_float2(v.x * s, v.y * s);
  }
}

// acc[i] (+)= |y[i]|^2
__global__ __launch_bounds__(256) void k3_accum_abs2(const float2 *__restrict__ y,
                                                     float *__restrict__ acc, long total,
                                                     int first) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const float2 v = y[i];
    const float p = v.x * v.x + v.y * v.y;
    acc[i] = first ? p : acc[i] + p;
  }
}

// out[i] = (sqrt(acc[i]), 0)
__global__ __launch_bounds__(256) void k3_sqrt(const float *__restrict__ acc,
                                               float2 *__restrict__ out, long total) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride)
    out[i] = make_float2(__builtin_amdgcn_sqrtf(acc[i]), 0.f);
}

// out[v][chan][a][b][c] = Re src[v][a s][b s][c s], s = 2^J
__global__ __launch_bounds__(256) void k3_sample(const float2 *__restrict__ src,
                                                 float *__restrict__ out, long volumes, int K,
                                                 int chan, int n0, int n1, int n2, int J) {
  const int m0 = n0 >> J, m1 = n1 >> J, m2 = n2 >> J;
  const long per = static_cast<long>(m0) * m1 * m2;
  const long total = volumes * per;
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const long v = i / per;
    long e = i - v * per;
    const int c = static_cast<int>(e % m2);
    e /= m2;
    const int b = static_cast<int>(e % m1);
    const int a = static_cast<int>(e / m1);
    const size_t s = ((static_cast<size_t>(v) * n0 + (static_cast<size_t>(a) << J)) * n1 +
                      (static_cast<size_t>(b) << J)) * n2 + (static_cast<size_t>(c) << J);
    out[(static_cast<size_t>(v) * K + chan) * per + (static_cast<size_t>(a) * m1 + b) * m2 + c] = src[s].x;
  }
}


// ---- fused passes for volumes whose (axis 1, axis 2) slabs fit a workgroup's LDS --------
// (slabs of up to 4096 points: 256 threads and 1 to 16 slabs per workgroup; 8192 and 16384
// points: one slab per workgroup of 512 or 1024 threads and up to 152 KB of LDS)
//
// A 3-D transform is split into the two slab axes (one workgroup holds whole N1 x N2
// slabs: rows through registers, a transposition through LDS, columns through registers)
// and axis 0 (columns of stride N1*N2).  Every launch takes a LIST of nodes (j, l)
// (blockIdx.y): a 32^3 volume has 32 slabs of 64 threads, so one node of a small batch fills
// a quarter of the chip and runs at the latency of its load - transform - store chain; with
// the nodes of a whole order side by side the launches are both larger and fewer.
//   k3_slab_mul_inv   W_p = inverse transform over the slab axes of F^ (g_2p + i g_2p+1), all
//                     pairs of a (j, l) (the slab of F^ is read once).  The
//                     signal F is real and the tables g_m are real with the parity of l, so
//                     F conv g_m is real (l even) or imaginary (l odd) and one complex
//                     transform carries two of them: |W_p|^2 = |F conv g_2p|^2 +
//                     |F conv g_2p+1|^2, which is all the non-linearity needs
//   k3_axis0_rho      inverse transform along axis 0 of every W_m, sum of squared moduli in
//                     registers, square root, forward transform along axis 0; the result T
//                     is the axis-0 spectrum of a real signal: rows 0 .. n0/2 are stored
//   k3_slab_fwd_low   forward transform over the slab axes of those rows (giving U^ for
//                     k0 <= n0/2 and, by conjugate symmetry, for n0 - k0), product with the
//                     lowpass and the sum over the aliases of the slab axes (periodic
//                     subsampling by 2^J seen from the Fourier side)
//   k3_out            the aliases of axis 0, the small inverse transform, real part and crop

template <int N1, int N2, bool SPLIT>
__global__ __launch_bounds__((Slab<N1, N2>::NT)) void k3_slab_mul_inv(Nodes3 nodes, long slabs, int n0,
                                                       size_t mstride,
                                                       const float2 *__restrict__ tw, int tw_n) {
  using S = Slab<N1, N2>;
  constexpr bool WAVE = S::TS <= 64;  // a slab's threads are lanes of one wavefront
  extern __shared__ float2 lds[];
  const Node3 &nd = nodes.v[blockIdx.y];
  const int M = nd.M;
  // SPLIT: one filter per workgroup (blockIdx.z), no loop state to carry
  if (SPLIT && static_cast<int>(blockIdx.z) >= M) return;
  const int s = threadIdx.x / S::TS, q = threadIdx.x % S::TS;
  const long slab = static_cast<long>(blockIdx.x) * S::SPW + s;
  const bool live = slab < slabs;
  const long sl = live ? slab : slabs - 1;  // idle threads shadow the last slab, store nothing
  float2 *area = lds + s * N1 * S::RS;
  // one filter: the transforms' twiddles from LDS tables, fetched while the operands are (16.6 -> 15.3 us for 12
  // signals of 8 x 32^3); several filters keep them in registers (145 us against 147 for 20 signals of 16 x 64^3)
  float2 *wtab = lds + S::SPW * N1 * S::RS;
  if (SPLIT) S::fill_twiddles(wtab, tw, tw_n, false);
  const int r = q / S::T2, t = q % S::T2;
  const int c = q % N2, t1 = q / N2;
  const int k0 = static_cast<int>(sl % n0);
  const size_t base = static_cast<size_t>(sl) * N1 * N2;
  const float2 *__restrict__ src = nd.src + base + r * N2 + t;
  const float2 *__restrict__ tab = nd.tab;
  float2 *__restrict__ W = nd.W;
  // the slab of F^ stays in registers across the filters, except in the SPLIT variants
  constexpr bool KEEP = !SPLIT;
  float2 f[KEEP ? 16 : 1];
  if (KEEP) {
#pragma unroll
    for (int i = 0; i < 16; ++i) f[KEEP ? i : 0] = src[S::T2 * i];
  }
  const int m_first = SPLIT ? static_cast<int>(blockIdx.z) : 0, m_last = SPLIT ? m_first + 1 : M;
  for (int m = m_first; m < m_last; ++m) {
    const float2 *tb = tab + (static_cast<size_t>(m) * n0 + k0) * N1 * N2 + r * N2 + t;
    float2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      v[i] = c_mul(KEEP ? f[KEEP ? i : 0] : src[S::T2 * i], tb[S::T2 * i]);
      // (1024 threads, 128 registers each) two batches of loads, so that the operands in flight fit
      if (!KEEP && S::NT == 1024 && i == 7) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (SPLIT) {
      __syncthreads();
      S::template transform_tab<true, WAVE>(v, area, r, t, c, t1, wtab);
    } else {
      S::template transform<true, WAVE>(v, area, r, t, c, t1, tw, tw_n);
    }
    if (live) {
      float2 *dst = W + static_cast<size_t>(m) * mstride + base + c;
#pragma unroll
      for (int i = 0; i < 16; ++i) dst[(t1 + S::T1 * i) * N2] = v[i];
    }
    if (!SPLIT) group_sync<WAVE>();  // the slab area is reused by the next filter
  }
}

// A node's T holds slabs k0 = 0 .. n0/2 only (the axis-0 spectrum of a real signal); the slab
// n0 - k0 of U^ and of the folded lowpass product is the conjugate of slab k0 with both
// slab indices negated, and is written from the same registers.  phi == nullptr: U^ only.
template <int N1, int N2>
__global__ __launch_bounds__((Slab<N1, N2>::NT)) void k3_slab_fwd_low(Nodes3 nodes,
                                                       const float *__restrict__ phi,
                                                       float2 *__restrict__ P, long slabs, int n0,
                                                       int J, size_t p_vol_stride, size_t p_chan_stride,
                                                       const float2 *__restrict__ tw, int tw_n) {
  using S = Slab<N1, N2>;
  constexpr bool WAVE = S::TS <= 64;
  extern __shared__ float2 lds[];
  const Node3 &nd = nodes.v[blockIdx.y];
  const int s = threadIdx.x / S::TS, q = threadIdx.x % S::TS;
  const long slab = static_cast<long>(blockIdx.x) * S::SPW + s;
  const bool live = slab < slabs;
  const long sl = live ? slab : slabs - 1;
  float2 *area = lds + s * N1 * S::RS;
  // (twiddles from LDS tables, fetched while the slab is: 39.7 -> 36.2 us a launch of 16 x 64^3; with them slabs of
  // 16 x 256 fit a compute unit three instead of four times, which costs nothing: J = 2, L = 2, 24 volumes of
  // 16 x 16 x 256 169.4 -> 168.7 us, gradient 360.9 -> 357.3; of 64 x 16 x 256 648.8 -> 645.5, 1478 -> 1476)
  float2 *wtab = lds + S::SPW * N1 * S::RS;
  S::fill_twiddles(wtab, tw, tw_n, false);
  const int r = q / S::T2, t = q % S::T2;
  const int c = q % N2, t1 = q / N2;
  const int H = n0 / 2 + 1;
  const int k0 = static_cast<int>(sl % H);
  const long vol = sl / H;
  const bool twin = k0 > 0 && k0 < n0 - k0;  // slab n0 - k0 is a different slab
  const float2 *__restrict__ src = nd.T + static_cast<size_t>(sl) * N1 * N2 + r * N2 + t;
  float2 *__restrict__ Uout = nd.U;
  float2 v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = src[S::T2 * i];
  __syncthreads();
  S::template transform_tab<false, WAVE>(v, area, r, t, c, t1, wtab);
  if (Uout != nullptr && live) {
    float2 *dst = Uout + (static_cast<size_t>(vol) * n0 + k0) * N1 * N2 + c;
#pragma unroll
    for (int i = 0; i < 16; ++i) dst[(t1 + S::T1 * i) * N2] = v[i];
    if (twin) {
      float2 *dm = Uout + (static_cast<size_t>(vol) * n0 + (n0 - k0)) * N1 * N2 + ((N2 - c) & (N2 - 1));
#pragma unroll
      for (int i = 0; i < 16; ++i)
        dm[((N1 - (t1 + S::T1 * i)) & (N1 - 1)) * N2] = make_float2(v[i].x, -v[i].y);
    }
  }
  if (phi == nullptr) return;
  // lowpass product, then the sum over the 4^J aliases of the slab axes
  const float *ph = phi + static_cast<size_t>(k0) * N1 * N2 + c;
  group_sync<WAVE>();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float g = ph[(t1 + S::T1 * i) * N2];
    area[(t1 + S::T1 * i) * S::RS + c] = make_float2(v[i].x * g, v[i].y * g);
  }
  group_sync<WAVE>();
  const int m1 = N1 >> J, m2 = N2 >> J, al = 1 << J;
  if (!live) return;
  float2 *pv = P + static_cast<size_t>(vol) * p_vol_stride + nd.chan * p_chan_stride;
  float2 *dst = pv + static_cast<size_t>(k0) * m1 * m2;
  float2 *dm = pv + static_cast<size_t>(n0 - k0) * m1 * m2;
  for (int o = q; o < m1 * m2; o += S::TS) {
    const int a = o / m2, b = o - a * m2;
    float2 acc = make_float2(0.f, 0.f);
    for (int p1 = 0; p1 < al; ++p1)
      for (int p2 = 0; p2 < al; ++p2) {
        const float2 e = area[(a + m1 * p1) * S::RS + b + m2 * p2];
        acc.x += e.x;
        acc.y += e.y;
      }
    dst[o] = acc;
    if (twin) dm[((m1 - a) & (m1 - 1)) * m2 + ((m2 - b) & (m2 - 1))] = make_float2(acc.x, -acc.y);
  }
}

// Axis 0 of [volumes][E*T][Mc]: a workgroup takes TC columns of one volume, thread (t, c)
// holds rows t + T i.  xreal != nullptr: forward transform of the real input (of u0 x u1 x u2
// samples, extended symmetrically to the grid with u0 > 0, else of the grid's own size).
// Else: inverse transform of the node's M signals W_m, root of the sum of their squared
// moduli, forward transform.  The transformed signal is real, so only rows 0 .. N0/2 of its
// spectrum are stored: T [volumes][N0/2 + 1][Mc].
template <int E, int T>
__global__ __launch_bounds__(256) void k3_axis0_rho(Nodes3 nodes, const float *__restrict__ xreal,
                                                    int u0, int u1, int u2, int n2, int Mc, int TC,
                                                    size_t mstride, const float2 *__restrict__ tw,
                                                    int tw_n) {
  constexpr int N0 = E * T;
  extern __shared__ float2 lds[];
  const Node3 &nd = nodes.v[blockIdx.y];
  const int KS = T * TC + (E == 32 ? 0 : 1);
  const int c = threadIdx.x % TC, t = threadIdx.x / TC;
  const int tiles = Mc / TC;
  const long vol = blockIdx.x / tiles;
  const int c0 = static_cast<int>(blockIdx.x % tiles) * TC;
  const size_t off = static_cast<size_t>(vol) * N0 * Mc + static_cast<size_t>(t) * Mc + c0 + c;
  const size_t step = static_cast<size_t>(T) * Mc;
  float2 wt[E];
  load_twiddles<E, T>(wt, t, tw, tw_n);
  float2 v[E];
  if (xreal != nullptr) {
    if (u0 > 0) {
      const int b = (c0 + c) / n2, e = (c0 + c) % n2;
      const float *x = xreal + (static_cast<size_t>(vol) * u0 * u1 + pad_source(b, u1, Mc / n2)) * u2 +
                       pad_source(e, u2, n2);
#pragma unroll
      for (int i = 0; i < E; ++i)
        v[i] = make_float2(x[static_cast<size_t>(pad_source(t + T * i, u0, N0)) * u1 * u2], 0.f);
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = make_float2(xreal[off + i * step], 0.f);
    }
  } else {
    const float2 *__restrict__ W = nd.W;
    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.f;
    for (int m = 0; m < nd.M; ++m) {
      const float2 *p = W + static_cast<size_t>(m) * mstride + off;
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = p[i * step];
      fft_core<E, T, true, false>(v, t, lds + c, KS, TC, wt);
#pragma unroll
      for (int i = 0; i < E; ++i) acc[i] += v[i].x * v[i].x + v[i].y * v[i].y;
    }
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = make_float2(__builtin_amdgcn_sqrtf(acc[i]), 0.f);
  }
  fft_core<E, T, false, false>(v, t, lds + c, KS, TC, wt);
  float2 *o = nd.T + static_cast<size_t>(vol) * (N0 / 2 + 1) * Mc + static_cast<size_t>(t) * Mc + c0 + c;
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (t + T * i <= N0 / 2) o[i * step] = v[i];
}

// ---- backward pass of the fused plans.  For a node with signals y_p = IFFT(F^ c_p), given
// the gradient g of rho = sqrt(sum_p |y_p|^2) along the slab axes' inverse transform (T):
//   k3_slab_sum_inv   T = inverse slab transform of phi^ * tile(g_S^) (+ the spectra its
//                     children contributed)
//   k3_axis0_back     inverse transform along axis 0 of T and of every W_p, y_p g / rho,
//                     forward transform along axis 0, in place
//   k3_slab_fwd_mulacc  forward slab transform, product with conj(c_p), sum over the pairs:
//                     the node's contribution to its source's gradient spectrum

// W_p <- forward transform along axis 0 of g y_p / rho (0 where rho = 0), y_p = inverse
// transform of W_p (the slab axes' inverse transforms are done).  The signals are read and
// inverse-transformed twice, once for rho and once for the product: keeping them would take a
// write and a read of every signal instead of the second read.  T holds rows 0 .. N0/2 where
// the gradient is real by symmetry (nd.half) and all rows otherwise (its real part counts).
template <int E, int T>
__global__ __launch_bounds__(256) void k3_axis0_back(Nodes3 nodes, int Mc, int TC, size_t mstride,
                                                     const float2 *__restrict__ tw, int tw_n) {
  constexpr int N0 = E * T;
  extern __shared__ float2 lds[];
  const Node3 &nd = nodes.v[blockIdx.y];
  const int P = nd.M;
  const int KS = T * TC + (E == 32 ? 0 : 1);
  const int c = threadIdx.x % TC, t = threadIdx.x / TC;
  const int tiles = Mc / TC;
  const long vol = blockIdx.x / tiles;
  const int c0 = static_cast<int>(blockIdx.x % tiles) * TC;
  const size_t off = static_cast<size_t>(vol) * N0 * Mc + static_cast<size_t>(t) * Mc + c0 + c;
  const size_t step = static_cast<size_t>(T) * Mc;
  // The transforms' twiddles in an LDS table behind the exchange area (wtab[k T + t]); the
  // registers they would take hold the next signal's values, requested before the current
  // signal is transformed (otherwise they would queue behind its stores).
  constexpr bool TAB = T > 1;
  float2 *wtab = lds + E * KS;
  if (TAB) {
    for (int idx = threadIdx.x; idx < N0; idx += blockDim.x)
      wtab[idx] = tw[(idx / T) * (idx % T) * (tw_n / N0)];
    __syncthreads();
  }
  float2 vn[E];
  auto fetch = [&](int p) {
    const float2 *w = nd.W + static_cast<size_t>(p) * mstride + off;
#pragma unroll
    for (int i = 0; i < E; ++i) vn[i] = w[i * step];
  };
  float a[E];
#pragma unroll
  for (int i = 0; i < E; ++i) a[i] = 0.f;
  fetch(0);
  float2 v[E];
  for (int p = 0; p < P; ++p) {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = vn[i];
    if (p + 1 < P) fetch(p + 1);
    fft_core_tab<E, T, true, false>(v, t, lds + c, KS, TC, wtab + t, T);
#pragma unroll
    for (int i = 0; i < E; ++i) a[i] += v[i].x * v[i].x + v[i].y * v[i].y;
  }
  // one pair: its signal is still in v; else the first one is requested again
  float2 g[E];
  {
    const float2 *src = nd.T + static_cast<size_t>(vol) * (nd.half ? N0 / 2 + 1 : N0) * Mc + c0 + c;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int row = t + T * i;
      const bool mir = nd.half && row > N0 / 2;
      g[i] = src[static_cast<size_t>(mir ? N0 - row : row) * Mc];
      if (mir) g[i].y = -g[i].y;
    }
  }
  fft_core_tab<E, T, true, false>(g, t, lds + c, KS, TC, wtab + t, T);
#pragma unroll
  for (int i = 0; i < E; ++i) a[i] = over_sqrt(g[i].x, a[i]);
  if (P > 1) fetch(0);
  for (int p = 0; p < P; ++p) {
    float2 *w = nd.W + static_cast<size_t>(p) * mstride + off;
    if (P > 1) {
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = vn[i];
      if (p + 1 < P) fetch(p + 1);
      fft_core_tab<E, T, true, false>(v, t, lds + c, KS, TC, wtab + t, T);
    }
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = make_float2(v[i].x * a[i], v[i].y * a[i]);
    fft_core_tab<E, T, false, false>(v, t, lds + c, KS, TC, wtab + t, T);
#pragma unroll
    for (int i = 0; i < E; ++i) w[i * step] = v[i];
  }
}

// Slab axes: A[slab] = sum_p conj(c_p) * (forward slab transform of W_p), the adjoint of
// k3_slab_mul_inv (c_p = the pair tables of the node), written over W_0 (a slab is read and
// written by the same workgroup only).
template <int N1, int N2>
__global__ __launch_bounds__((Slab<N1, N2>::NT)) void k3_slab_fwd_mulacc(Nodes3 nodes, long slabs, int n0,
                                                                         size_t mstride,
                                                                         const float2 *__restrict__ tw,
                                                                         int tw_n) {
  using S = Slab<N1, N2>;
  constexpr bool WAVE = S::TS <= 64;
  extern __shared__ float2 lds[];
  const Node3 &nd = nodes.v[blockIdx.y];
  const int P = nd.M;
  const int s = threadIdx.x / S::TS, q = threadIdx.x % S::TS;
  const long slab = static_cast<long>(blockIdx.x) * S::SPW + s;
  const bool live = slab < slabs;
  const long sl = live ? slab : slabs - 1;
  float2 *area = lds + s * N1 * S::RS;
  const int r = q / S::T2, t = q % S::T2;
  const int c = q % N2, t1 = q / N2;
  const int k0 = static_cast<int>(sl % n0);
  const size_t base = static_cast<size_t>(sl) * N1 * N2;
  // the transforms' twiddles in LDS tables: their registers go to the table values, which
  // are requested before the transform they are used after
  float2 *wtab = lds + S::SPW * N1 * S::RS;
  S::fill_twiddles(wtab, tw, tw_n);
  float2 sum[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) sum[i] = make_float2(0.f, 0.f);
  for (int p = 0; p < P; ++p) {
    const float2 *src = nd.W + static_cast<size_t>(p) * mstride + base + r * N2 + t;
    float2 v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = src[S::T2 * i];
    const float2 *tb = nd.tab + (static_cast<size_t>(p) * n0 + k0) * N1 * N2 + c;
    float2 gt[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) gt[i] = tb[(t1 + S::T1 * i) * N2];
    S::template transform_tab<false, WAVE>(v, area, r, t, c, t1, wtab);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float2 g = gt[i];
      g.y = -g.y;
      const float2 o = c_mul(v[i], g);
      sum[i].x += o.x;
      sum[i].y += o.y;
    }
    group_sync<WAVE>();  // the slab area is reused by the next signal
  }
  if (!live) return;
  float2 *dst = nd.W + base + c;
#pragma unroll
  for (int i = 0; i < 16; ++i) dst[(t1 + S::T1 * i) * N2] = sum[i];
}

// T = inverse slab transform of phi^ * tile(g_S^) + sum of the item's spectra A: slabs 0 .. n0/2
// where there are none (the gradient of the lowpass alone is real), else all of them.
template <int N1, int N2>
__global__ __launch_bounds__((Slab<N1, N2>::NT)) void k3_slab_sum_inv(Sums3 sums, const float *__restrict__ phi,
                                                       const float2 *__restrict__ Gs, long volumes, int n0,
                                                       int J, int K, const float2 *__restrict__ tw, int tw_n) {
  using S = Slab<N1, N2>;
  constexpr bool WAVE = S::TS <= 64;
  extern __shared__ float2 lds[];
  const Sum3 &it = sums.v[blockIdx.y];
  const int H = it.count == 0 ? n0 / 2 + 1 : n0;
  const long slabs = volumes * H;
  if (static_cast<long>(blockIdx.x) * S::SPW >= slabs) return;
  const int s = threadIdx.x / S::TS, q = threadIdx.x % S::TS;
  const long slab = static_cast<long>(blockIdx.x) * S::SPW + s;
  const bool live = slab < slabs;
  const long sl = live ? slab : slabs - 1;
  float2 *area = lds + s * N1 * S::RS;
  const int r = q / S::T2, t = q % S::T2;
  const int c = q % N2, t1 = q / N2;
  const int k0 = static_cast<int>(sl % H);
  const long vol = sl / H;
  const int m0 = n0 >> J, m1 = N1 >> J, m2 = N2 >> J;
  const float2 *gs = Gs + ((static_cast<size_t>(vol) * K + it.chan) * m0 + (k0 & (m0 - 1))) * m1 * m2 +
                     (c & (m2 - 1));
  const float *ph = phi + static_cast<size_t>(k0) * N1 * N2 + c;
  const size_t base = (static_cast<size_t>(vol) * n0 + k0) * N1 * N2 + c;
  float2 v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = t1 + S::T1 * i;
    const float f = ph[row * N2];
    const float2 g = gs[(row & (m1 - 1)) * m2];
    v[i] = make_float2(g.x * f, g.y * f);
  }
  for (int a = 0; a < it.count; ++a) {
    const float2 *p = sums.A[it.first + a] + base;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float2 u = p[(t1 + S::T1 * i) * N2];
      v[i].x += u.x;
      v[i].y += u.y;
    }
  }
  S::template transform_back<true, WAVE>(v, area, r, t, c, t1, tw, tw_n);
  if (!live) return;
  float2 *dst = it.T + static_cast<size_t>(sl) * N1 * N2 + r * N2 + t;
#pragma unroll
  for (int i = 0; i < 16; ++i) dst[S::T2 * i] = v[i];
}

// dst[i] = sum of the first item's spectra (which may include dst itself)
__global__ __launch_bounds__(256) void k3_sum_spectra(Sums3 sums, float2 *dst, long total) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  const Sum3 &it = sums.v[0];
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    float2 acc = make_float2(0.f, 0.f);
    for (int a = 0; a < it.count; ++a) {
      const float2 u = sums.A[it.first + a][i];
      acc.x += u.x;
      acc.y += u.y;
    }
    dst[i] = acc;
  }
}

// out [volumes][E*T][Mc] = real part of the inverse transform along axis 0 of T
template <int E, int T>
__global__ __launch_bounds__(256) void k3_axis0_real(const float2 *__restrict__ src, float *__restrict__ out,
                                                     int Mc, int TC, const float2 *__restrict__ tw, int tw_n) {
  constexpr int N0 = E * T;
  extern __shared__ float2 lds[];
  const int KS = T * TC + (E == 32 ? 0 : 1);
  const int c = threadIdx.x % TC, t = threadIdx.x / TC;
  const int tiles = Mc / TC;
  const long vol = blockIdx.x / tiles;
  const int c0 = static_cast<int>(blockIdx.x % tiles) * TC;
  const size_t off = static_cast<size_t>(vol) * N0 * Mc + static_cast<size_t>(t) * Mc + c0 + c;
  const size_t step = static_cast<size_t>(T) * Mc;
  float2 wt[E];
  load_twiddles<E, T>(wt, t, tw, tw_n);
  float2 v[E];
#pragma unroll
  for (int i = 0; i < E; ++i) v[i] = src[off + i * step];
  fft_core<E, T, true, false>(v, t, lds + c, KS, TC, wt);
#pragma unroll
  for (int i = 0; i < E; ++i) out[off + i * step] = v[i].x;
}

// ---- output grids held whole by a workgroup: at most 4096 points, at most 32 a side, lines
// transformed by one thread each
constexpr int kOutPoints = 4096;

template <int M, bool INV>
__device__ __forceinline__ void line_fft(float2 *p, int stride) {
  float2 v[M];
#pragma unroll
  for (int i = 0; i < M; ++i) v[i] = p[i * stride];
  DftRegs<M, INV>::run(v);
#pragma unroll
  for (int i = 0; i < M; ++i) p[i * stride] = v[i];
}
template <bool INV>
__device__ __forceinline__ void line_fft_any(float2 *p, int stride, int m) {
  switch (m) {
    case 2: line_fft<2, INV>(p, stride); break;
    case 4: line_fft<4, INV>(p, stride); break;
    case 8: line_fft<8, INV>(p, stride); break;
    case 16: line_fft<16, INV>(p, stride); break;
    case 32: line_fft<32, INV>(p, stride); break;
    default: break;
  }
}
// transform along the three axes of buf [m0][m1][m2 + 1]
template <bool INV>
__device__ __forceinline__ void cube_fft(float2 *buf, int m0, int m1, int m2) {
  const int rs = m2 + 1;
  for (int l = threadIdx.x; l < m0 * m1; l += blockDim.x) line_fft_any<INV>(buf + l * rs, 1, m2);
  __syncthreads();
  for (int l = threadIdx.x; l < m0 * m2; l += blockDim.x)
    line_fft_any<INV>(buf + (l / m2) * m1 * rs + l % m2, rs, m1);
  __syncthreads();
  for (int l = threadIdx.x; l < m1 * m2; l += blockDim.x)
    line_fft_any<INV>(buf + (l / m2) * rs + l % m2, m1 * rs, m0);
  __syncthreads();
}

// One workgroup per (volume, channel): the sum over the aliases of axis 0 of P [n0][m1 m2], the
// inverse transform on the output grid and its real part, restricted to o0 x o1 x o2 samples.
// One launch for what took a fold, three passes of plain transforms, a real part and a crop
// (six launches of 2 to 8 us each on grids of 512 to 4096 points).
__global__ __launch_bounds__(256) void k3_out(const float2 *__restrict__ P, float *__restrict__ out, int n0,
                                              int m0, int m1, int m2, int o0, int o1, int o2) {
  extern __shared__ float2 lds[];
  const int slab = m1 * m2, pts = m0 * slab, rs = m2 + 1;
  const float2 *src = P + static_cast<size_t>(blockIdx.x) * n0 * slab;
  // four points per thread at a time: their loads are in flight together
  for (int e0 = threadIdx.x; e0 < pts; e0 += 4 * blockDim.x) {
    float2 acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = make_float2(0.f, 0.f);
#pragma unroll 2
    for (int a = 0; a < n0 / m0; ++a) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + u * blockDim.x;
        const float2 w = src[static_cast<size_t>(a) * pts + (e < pts ? e : 0)];
        acc[u].x += w.x;
        acc[u].y += w.y;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * blockDim.x;
      if (e < pts) lds[(e / m2) * rs + e % m2] = acc[u];
    }
  }
  __syncthreads();
  cube_fft<true>(lds, m0, m1, m2);
  float *dst = out + static_cast<size_t>(blockIdx.x) * o0 * o1 * o2;
  for (int e = threadIdx.x; e < o0 * o1 * o2; e += blockDim.x) {
    const int c = e % o2, ab = e / o2;
    dst[e] = lds[((ab / o1) * m1 + ab % o1) * rs + c].x;
  }
}

// The adjoint's first step: Gs [m0][m1][m2] = forward transform of the output gradient of one
// (volume, channel), given on o0 x o1 x o2 samples and zero elsewhere.
__global__ __launch_bounds__(256) void k3_out_adj(const float *__restrict__ gout, float2 *__restrict__ Gs, int m0,
                                                  int m1, int m2, int o0, int o1, int o2) {
  extern __shared__ float2 lds[];
  const int pts = m0 * m1 * m2, rs = m2 + 1;
  const float *src = gout + static_cast<size_t>(blockIdx.x) * o0 * o1 * o2;
  for (int e = threadIdx.x; e < pts; e += blockDim.x) {
    const int c = e % m2, ab = e / m2, a = ab / m1, b = ab % m1;
    const bool in = a < o0 && b < o1 && c < o2;
    lds[ab * rs + c] = make_float2(in ? src[(a * o1 + b) * o2 + c] : 0.f, 0.f);
  }
  __syncthreads();
  cube_fft<false>(lds, m0, m1, m2);
  float2 *dst = Gs + static_cast<size_t>(blockIdx.x) * pts;
  for (int e = threadIdx.x; e < pts; e += blockDim.x) dst[e] = lds[(e / m2) * rs + e % m2];
}

// Q[g][a0][e] = sum_p P[g][a0 + m0 p][e]: g over volumes x channels, e over the m1*m2
// folded slab points
__global__ __launch_bounds__(256) void k3_fold0(const float2 *__restrict__ P,
                                                float2 *__restrict__ Q, long groups, int n0, int m0,
                                                int slab) {
  const long per = static_cast<long>(m0) * slab;
  const long total = groups * per;
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const long g = i / per;
    const long e = i - g * per;  // a0 * slab + point
    const float2 *src = P + static_cast<size_t>(g) * n0 * slab + e;
    float2 acc = make_float2(0.f, 0.f);
    for (int a = 0; a < n0; a += m0) {
      const float2 u = src[static_cast<size_t>(a) * slab];
      acc.x += u.x;
      acc.y += u.y;
    }
    Q[i] = acc;
  }
}

__global__ __launch_bounds__(256) void k3_real_part(const float2 *__restrict__ src,
                                                    float *__restrict__ out, long total) {
  const long stride = static_cast<long>(gridDim.x) * blockDim.x;
  for (long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride)
    out[i] = src[i].x;
}

// Slab transforms of every node of the list.  SPLIT (one filter per workgroup instead of a loop
// over the node's filters) always for the 1024-thread slabs (no registers for the loop state),
// else below 700 workgroups, where the loop's serial chain of transforms is the launch's time: a
// whole forward call with the loop / split takes 104 / 98 us for one volume of 64^3 (512
// workgroups), 131 / 132 us for two (1024), 200 / 220 us for four and 690 / 777 us for sixteen.
template <int N1, int N2>
hipError_t slab_mul_inv_t(const Nodes3 &nodes, long volumes, int n0, const float2 *tw, int tw_n,
                          hipStream_t st) {
  using S = Slab<N1, N2>;
  const long slabs = volumes * n0;
  const long blocks = (slabs + S::SPW - 1) / S::SPW;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  int most = 0, all = 0;
  for (int i = 0; i < nodes.n; ++i) {
    most = nodes.v[i].M > most ? nodes.v[i].M : most;
    all += nodes.v[i].M;
  }
  const bool split = S::NT == 1024 || blocks * nodes.n < 700;
  const std::string name = "k3_slab_mul_inv<" + std::to_string(N1) + ", " + std::to_string(N2) +
                           (split ? ", true>" : ", false>");
  const double pts = static_cast<double>(slabs) * N1 * N2;
  LaunchScope obs(name.c_str(), pts * 8.0 * (nodes.n + all) + 8.0 * all * n0 * N1 * N2,
                  pts * all * (5.0 * (ilog2h(N1) + ilog2h(N2)) + 6.0), st);
  const size_t mstride = static_cast<size_t>(slabs) * N1 * N2;
  if (split) {
    if (most > 65535) return hipErrorInvalidValue;
    constexpr size_t lds = S::lds_bytes + S::tab_elems * sizeof(float2);
    if (lds > 65536) {
      static unsigned long long lds_ok = 0;
      hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k3_slab_mul_inv<N1, N2, true>), lds_ok);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k3_slab_mul_inv<N1, N2, true>), dim3(static_cast<unsigned>(blocks), nodes.n, most),
                       dim3(S::NT), lds, st, nodes, slabs, n0, mstride, tw, tw_n);
    return hipGetLastError();
  }
  if constexpr (S::NT != 1024) {
    if (S::lds_bytes > 65536) {
      static unsigned long long lds_ok = 0;
      hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k3_slab_mul_inv<N1, N2, false>), lds_ok);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k3_slab_mul_inv<N1, N2, false>), dim3(static_cast<unsigned>(blocks), nodes.n),
                       dim3(S::NT), S::lds_bytes, st, nodes, slabs, n0, mstride, tw, tw_n);
  }
  return hipGetLastError();
}

template <int N1, int N2>
hipError_t slab_fwd_low_t(const Nodes3 &nodes, const float *phi, float2 *P, long volumes, int n0, int J,
                          int K, const float2 *tw, int tw_n, hipStream_t st) {
  using S = Slab<N1, N2>;
  const long slabs = volumes * (n0 / 2 + 1);
  const long blocks = (slabs + S::SPW - 1) / S::SPW;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const size_t folded = static_cast<size_t>(n0) * (N1 >> J) * (N2 >> J);
  const std::string name =
      "k3_slab_fwd_low<" + std::to_string(N1) + ", " + std::to_string(N2) + ">";
  const double pts = static_cast<double>(slabs) * N1 * N2;
  const double full = static_cast<double>(volumes) * n0 * N1 * N2;
  int stored = 0;
  for (int i = 0; i < nodes.n; ++i) stored += nodes.v[i].U != nullptr;
  LaunchScope obs(name.c_str(),
                  nodes.n * pts * 8.0 + stored * full * 8.0 +
                      (phi ? 4.0 * (n0 / 2 + 1) * N1 * N2 + nodes.n * 8.0 * volumes * folded : 0.0),
                  nodes.n * pts * (5.0 * (ilog2h(N1) + ilog2h(N2)) + (phi ? 4.0 : 0.0)), st);
  constexpr size_t lds = S::lds_bytes + S::tab_elems * sizeof(float2);
  if (lds > 65536) {
    static unsigned long long lds_ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k3_slab_fwd_low<N1, N2>), lds_ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k3_slab_fwd_low<N1, N2>), dim3(static_cast<unsigned>(blocks), nodes.n), dim3(S::NT),
                     lds, st, nodes, phi, P, slabs, n0, J, folded * K, folded, tw, tw_n);
  return hipGetLastError();
}

template <int E, int T>
hipError_t axis0_t(const Nodes3 &nodes, const float *xreal, const int *user, long volumes, int n2, int Mc,
                   const float2 *tw, int tw_n, hipStream_t st) {
  int TC = 256 / T;
  if (TC > Mc) TC = Mc;
  const long blocks = volumes * (Mc / TC);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const size_t lds =
      T == 1 ? 0 : static_cast<size_t>(E) * (T * TC + (E == 32 ? 0 : 1)) * sizeof(float2);
  const std::string name = "k3_axis0_rho<" + std::to_string(E) + ", " + std::to_string(T) + ">";
  const double pts = static_cast<double>(volumes) * E * T * Mc;
  int all = 0;
  for (int i = 0; i < nodes.n; ++i) all += nodes.v[i].M;
  LaunchScope obs(name.c_str(),
                  pts * (xreal ? 4.0 : 8.0 * all) + nodes.n * pts * 8.0 * (E * T / 2 + 1) / (E * T),
                  pts * ((xreal ? 1 : all + nodes.n) * 5.0 * ilog2h(E * T) + (xreal ? 0.0 : 4.0 * all)), st);
  hipLaunchKernelGGL((k3_axis0_rho<E, T>), dim3(static_cast<unsigned>(blocks), nodes.n), dim3(T * TC), lds, st,
                     nodes, xreal, user ? user[0] : 0, user ? user[1] : 0, user ? user[2] : 0, n2, Mc, TC,
                     static_cast<size_t>(volumes) * E * T * Mc, tw, tw_n);
  return hipGetLastError();
}

template <int E, int T>
hipError_t axis0_back_t(const Nodes3 &nodes, long volumes, int Mc, const float2 *tw, int tw_n, hipStream_t st) {
  int TC = 256 / T;
  if (TC > Mc) TC = Mc;
  const long blocks = volumes * (Mc / TC);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  // exchange area of the transforms, then their twiddle table
  const size_t lds =
      T == 1 ? 0 : (static_cast<size_t>(E) * (T * TC + (E == 32 ? 0 : 1)) + E * T) * sizeof(float2);
  const std::string name = "k3_axis0_back<" + std::to_string(E) + ", " + std::to_string(T) + ">";
  const double pts = static_cast<double>(volumes) * E * T * Mc;
  int all = 0;
  for (int i = 0; i < nodes.n; ++i) all += nodes.v[i].M;
  LaunchScope obs(name.c_str(), pts * (16.0 * all + 8.0 * nodes.n),
                  pts * ((2 * all + nodes.n) * 5.0 * ilog2h(E * T) + 6.0 * all), st);
  hipLaunchKernelGGL((k3_axis0_back<E, T>), dim3(static_cast<unsigned>(blocks), nodes.n), dim3(T * TC), lds, st,
                     nodes, Mc, TC, static_cast<size_t>(volumes) * E * T * Mc, tw, tw_n);
  return hipGetLastError();
}

template <int E, int T>
hipError_t axis0_real_t(const float2 *src, float *out, long volumes, int Mc, const float2 *tw, int tw_n,
                        hipStream_t st) {
  int TC = 256 / T;
  if (TC > Mc) TC = Mc;
  const long blocks = volumes * (Mc / TC);
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const size_t lds =
      T == 1 ? 0 : static_cast<size_t>(E) * (T * TC + (E == 32 ? 0 : 1)) * sizeof(float2);
  const std::string name = "k3_axis0_real<" + std::to_string(E) + ", " + std::to_string(T) + ">";
  const double pts = static_cast<double>(volumes) * E * T * Mc;
  LaunchScope obs(name.c_str(), pts * 12.0, pts * 5.0 * ilog2h(E * T), st);
  hipLaunchKernelGGL((k3_axis0_real<E, T>), dim3(static_cast<unsigned>(blocks)), dim3(T * TC), lds, st, src, out,
                     Mc, TC, tw, tw_n);
  return hipGetLastError();
}

template <int N1, int N2>
hipError_t slab_fwd_mulacc_t(const Nodes3 &nodes, long volumes, int n0, const float2 *tw, int tw_n,
                             hipStream_t st) {
  using S = Slab<N1, N2>;
  const long slabs = volumes * n0;
  const long blocks = (slabs + S::SPW - 1) / S::SPW;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const std::string name =
      "k3_slab_fwd_mulacc<" + std::to_string(N1) + ", " + std::to_string(N2) + ">";
  const double pts = static_cast<double>(slabs) * N1 * N2;
  int all = 0;
  for (int i = 0; i < nodes.n; ++i) all += nodes.v[i].M;
  LaunchScope obs(name.c_str(), pts * 8.0 * (all + nodes.n) + 8.0 * all * n0 * N1 * N2,
                  pts * all * (5.0 * (ilog2h(N1) + ilog2h(N2)) + 8.0), st);
  const size_t lds = S::lds_bytes + S::tab_elems * sizeof(float2);
  if (lds > 65536) {
    static unsigned long long lds_ok = 0;
    hipError_t e =
        allow_large_lds(reinterpret_cast<const void *>(k3_slab_fwd_mulacc<N1, N2>), lds_ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k3_slab_fwd_mulacc<N1, N2>), dim3(static_cast<unsigned>(blocks), nodes.n), dim3(S::NT),
                     lds, st, nodes, slabs, n0, static_cast<size_t>(slabs) * N1 * N2, tw, tw_n);
  return hipGetLastError();
}

template <int N1, int N2>
hipError_t slab_sum_inv_t(const Sums3 &sums, const float *phi, const float2 *Gs, long volumes, int n0, int J,
                          int K, const float2 *tw, int tw_n, hipStream_t st) {
  using S = Slab<N1, N2>;
  const long blocks = (volumes * n0 + S::SPW - 1) / S::SPW;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const std::string name = "k3_slab_sum_inv<" + std::to_string(N1) + ", " + std::to_string(N2) + ">";
  const double pts = static_cast<double>(volumes) * n0 * N1 * N2;
  double moved = 0, done = 0;
  for (int i = 0; i < sums.n; ++i) {
    moved += sums.v[i].count == 0 ? 0.5 : 1.0 + sums.v[i].count;
    done += sums.v[i].count == 0 ? 0.5 : 1.0;
  }
  LaunchScope obs(name.c_str(), pts * 8.0 * moved + 4.0 * n0 * N1 * N2,
                  pts * done * (5.0 * (ilog2h(N1) + ilog2h(N2)) + 4.0), st);
  if (S::lds_bytes > 65536) {
    static unsigned long long lds_ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k3_slab_sum_inv<N1, N2>), lds_ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k3_slab_sum_inv<N1, N2>), dim3(static_cast<unsigned>(blocks), sums.n), dim3(S::NT),
                     S::lds_bytes, st, sums, phi, Gs, volumes, n0, J, K, tw, tw_n);
  return hipGetLastError();
}

}  // namespace

bool fused3_supported(int n0, int n1, int n2, int J) {
  auto p2 = [](int v) { return v > 0 && (v & (v - 1)) == 0; };
  // slabs of up to 16384 points, except 256 x 64 whose padded rows exceed the LDS of a CU
  return p2(n0) && p2(n1) && p2(n2) && n0 >= 4 && n0 <= 256 && n1 >= 16 && n2 >= 16 &&
         n1 * n2 <= 16384 && !(n1 == 256 && n2 == 64) && J >= 0 && J <= 4 && (n1 >> J) >= 1 &&
         (n2 >> J) >= 1;
}

#define SCAT3_SLAB_DISPATCH(CALL)                  \
  switch ((n1 << 12) | n2) {                       \
    case (16 << 12) | 16: CALL(16, 16);            \
    case (16 << 12) | 32: CALL(16, 32);            \
    case (16 << 12) | 64: CALL(16, 64);            \
    case (16 << 12) | 128: CALL(16, 128);          \
    case (16 << 12) | 256: CALL(16, 256);          \
    case (32 << 12) | 16: CALL(32, 16);            \
    case (32 << 12) | 32: CALL(32, 32);            \
    case (32 << 12) | 64: CALL(32, 64);            \
    case (32 << 12) | 128: CALL(32, 128);          \
    case (64 << 12) | 16: CALL(64, 16);            \
    case (64 << 12) | 32: CALL(64, 32);            \
    case (64 << 12) | 64: CALL(64, 64);            \
    case (128 << 12) | 16: CALL(128, 16);          \
    case (128 << 12) | 32: CALL(128, 32);          \
    case (256 << 12) | 16: CALL(256, 16);          \
    case (32 << 12) | 256: CALL(32, 256);          \
    case (64 << 12) | 128: CALL(64, 128);          \
    case (128 << 12) | 64: CALL(128, 64);          \
    case (256 << 12) | 32: CALL(256, 32);          \
    case (64 << 12) | 256: CALL(64, 256);          \
    case (128 << 12) | 128: CALL(128, 128);        \
    default: return hipErrorInvalidValue;          \
  }

hipError_t launch3_slab_mul_inv(const Nodes3 &nodes, long volumes, int n0, int n1, int n2, const float2 *tw,
                                int tw_n, hipStream_t st) {
  if (volumes <= 0 || nodes.n <= 0) return hipSuccess;
  if (tw_n % n1 != 0 || tw_n % n2 != 0 || nodes.n > kMaxNodes3) return hipErrorInvalidValue;
#define SCAT3_A(A_, B_) return slab_mul_inv_t<A_, B_>(nodes, volumes, n0, tw, tw_n, st)
  SCAT3_SLAB_DISPATCH(SCAT3_A)
#undef SCAT3_A
}

hipError_t launch3_slab_fwd_low(const Nodes3 &nodes, const float *phi, float2 *P, long volumes, int n0, int n1,
                                int n2, int J, int K, const float2 *tw, int tw_n, hipStream_t st) {
  if (volumes <= 0 || nodes.n <= 0) return hipSuccess;
  if (tw_n % n1 != 0 || tw_n % n2 != 0 || J < 0 || J > 4 || (n1 >> J) < 1 || (n2 >> J) < 1 ||
      nodes.n > kMaxNodes3)
    return hipErrorInvalidValue;
#define SCAT3_C(A_, B_) return slab_fwd_low_t<A_, B_>(nodes, phi, P, volumes, n0, J, K, tw, tw_n, st)
  SCAT3_SLAB_DISPATCH(SCAT3_C)
#undef SCAT3_C
}

#define SCAT3_AXIS0_DISPATCH(CALL)        \
  switch (n0) {                           \
    case 4: CALL(4, 1);                   \
    case 8: CALL(8, 1);                   \
    case 16: CALL(16, 1);                 \
    case 32: CALL(16, 2);                 \
    case 64: CALL(16, 4);                 \
    case 128: CALL(16, 8);                \
    case 256: CALL(16, 16);               \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch3_axis0_rho(const Nodes3 &nodes, const float *xreal, const int *user, long volumes, int n0,
                             int n2, int Mc, const float2 *tw, int tw_n, hipStream_t st) {
  if (volumes <= 0 || nodes.n <= 0) return hipSuccess;
  if (tw_n % n0 != 0 || Mc < 256 || (Mc & (Mc - 1)) != 0 || nodes.n > kMaxNodes3 ||
      (xreal != nullptr && nodes.n != 1))
    return hipErrorInvalidValue;
  for (int i = 0; xreal == nullptr && i < nodes.n; ++i)
    if (nodes.v[i].M <= 0) return hipErrorInvalidValue;
#define SCAT3_B(E_, T_) return axis0_t<E_, T_>(nodes, xreal, user, volumes, n2, Mc, tw, tw_n, st)
  SCAT3_AXIS0_DISPATCH(SCAT3_B)
#undef SCAT3_B
}

hipError_t launch3_axis0_back(const Nodes3 &nodes, long volumes, int n0, int Mc, const float2 *tw, int tw_n,
                              hipStream_t st) {
  if (volumes <= 0 || nodes.n <= 0) return hipSuccess;
  if (tw_n % n0 != 0 || Mc < 256 || (Mc & (Mc - 1)) != 0 || nodes.n > kMaxNodes3) return hipErrorInvalidValue;
  for (int i = 0; i < nodes.n; ++i)
    if (nodes.v[i].M <= 0 || nodes.v[i].T == nullptr) return hipErrorInvalidValue;
#define SCAT3_AB(E_, T_) return axis0_back_t<E_, T_>(nodes, volumes, Mc, tw, tw_n, st)
  SCAT3_AXIS0_DISPATCH(SCAT3_AB)
#undef SCAT3_AB
}

hipError_t launch3_axis0_real(const float2 *src, float *out, long volumes, int n0, int Mc, const float2 *tw,
                              int tw_n, hipStream_t st) {
  if (volumes <= 0) return hipSuccess;
  if (tw_n % n0 != 0 || Mc < 256 || (Mc & (Mc - 1)) != 0) return hipErrorInvalidValue;
#define SCAT3_AR(E_, T_) return axis0_real_t<E_, T_>(src, out, volumes, Mc, tw, tw_n, st)
  SCAT3_AXIS0_DISPATCH(SCAT3_AR)
#undef SCAT3_AR
}

hipError_t launch3_slab_fwd_mulacc(const Nodes3 &nodes, long volumes, int n0, int n1, int n2, const float2 *tw,
                                   int tw_n, hipStream_t st) {
  if (volumes <= 0 || nodes.n <= 0) return hipSuccess;
  if (tw_n % n1 != 0 || tw_n % n2 != 0 || nodes.n > kMaxNodes3) return hipErrorInvalidValue;
#define SCAT3_D(A_, B_) return slab_fwd_mulacc_t<A_, B_>(nodes, volumes, n0, tw, tw_n, st)
  SCAT3_SLAB_DISPATCH(SCAT3_D)
#undef SCAT3_D
}

hipError_t launch3_slab_sum_inv(const Sums3 &sums, const float *phi, const float2 *Gs, long volumes, int n0,
                                int n1, int n2, int J, int K, const float2 *tw, int tw_n, hipStream_t st) {
  if (volumes <= 0 || sums.n <= 0) return hipSuccess;
  if (tw_n % n1 != 0 || tw_n % n2 != 0 || J < 0 || (n0 >> J) < 1 || (n1 >> J) < 1 || (n2 >> J) < 1 ||
      sums.n > kMaxNodes3)
    return hipErrorInvalidValue;
  for (int i = 0; i < sums.n; ++i)
    if (sums.v[i].first < 0 || sums.v[i].count < 0 || sums.v[i].first + sums.v[i].count > kMaxSpectra3)
      return hipErrorInvalidValue;
#define SCAT3_S(A_, B_) return slab_sum_inv_t<A_, B_>(sums, phi, Gs, volumes, n0, J, K, tw, tw_n, st)
  SCAT3_SLAB_DISPATCH(SCAT3_S)
#undef SCAT3_S
}

hipError_t launch3_sum_spectra(const Sums3 &sums, float2 *dst, long total, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  if (sums.n != 1 || sums.v[0].first < 0 || sums.v[0].count < 1 ||
      sums.v[0].first + sums.v[0].count > kMaxSpectra3)
    return hipErrorInvalidValue;
  LaunchScope obs("k3_sum_spectra", total * 8.0 * (1 + sums.v[0].count), total * 2.0 * sums.v[0].count, st);
  hipLaunchKernelGGL(k3_sum_spectra, dim3(blocks_for(total)), dim3(256), 0, st, sums, dst, total);
  return hipGetLastError();
}

bool out3_supported(int m0, int m1, int m2) {
  return m0 <= 32 && m1 <= 32 && m2 <= 32 && m0 * m1 * m2 <= kOutPoints;
}

hipError_t launch3_out(const float2 *P, float *out, long maps, int n0, int m0, int m1, int m2, const int *o,
                       hipStream_t st) {
  if (maps <= 0) return hipSuccess;
  if (!out3_supported(m0, m1, m2) || n0 % m0 != 0 || o[0] > m0 || o[1] > m1 || o[2] > m2 || maps > 0x7fffffffL)
    return hipErrorInvalidValue;
  const double pts = static_cast<double>(maps) * m0 * m1 * m2;
  LaunchScope obs("k3_out", pts * 8.0 * (n0 / m0) + 4.0 * maps * o[0] * o[1] * o[2],
                  pts * 5.0 * (ilog2h(m0) + ilog2h(m1) + ilog2h(m2)), st);
  hipLaunchKernelGGL(k3_out, dim3(static_cast<unsigned>(maps)), dim3(256),
                     static_cast<size_t>(m0) * m1 * (m2 + 1) * sizeof(float2), st, P, out, n0, m0, m1, m2, o[0],
                     o[1], o[2]);
  return hipGetLastError();
}

hipError_t launch3_out_adj(const float *gout, float2 *Gs, long maps, int m0, int m1, int m2, const int *o,
                           hipStream_t st) {
  if (maps <= 0) return hipSuccess;
  if (!out3_supported(m0, m1, m2) || o[0] > m0 || o[1] > m1 || o[2] > m2 || maps > 0x7fffffffL)
    return hipErrorInvalidValue;
  const double pts = static_cast<double>(maps) * m0 * m1 * m2;
  LaunchScope obs("k3_out_adj", pts * 8.0 + 4.0 * maps * o[0] * o[1] * o[2],
                  pts * 5.0 * (ilog2h(m0) + ilog2h(m1) + ilog2h(m2)), st);
  hipLaunchKernelGGL(k3_out_adj, dim3(static_cast<unsigned>(maps)), dim3(256),
                     static_cast<size_t>(m0) * m1 * (m2 + 1) * sizeof(float2), st, gout, Gs, m0, m1, m2, o[0],
                     o[1], o[2]);
  return hipGetLastError();
}

hipError_t launch3_fold0(const float2 *P, float2 *Q, long groups, int n0, int m0, int slab,
                         hipStream_t st) {
  const long total = groups * m0 * slab;
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_fold0", groups * 8.0 * slab * (n0 + m0), groups * 2.0 * slab * n0, st);
  hipLaunchKernelGGL(k3_fold0, dim3(blocks_for(total)), dim3(256), 0, st, P, Q, groups, n0, m0, slab);
  return hipGetLastError();
}

hipError_t launch3_real_part(const float2 *src, float *out, long total, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_real_part", total * 12.0, 0.0, st);
  hipLaunchKernelGGL(k3_real_part, dim3(blocks_for(total)), dim3(256), 0, st, src, out, total);
  return hipGetLastError();
}

hipError_t launch3_fft(float2 *data, long volumes, int n0, int n1, int n2, bool inverse,
                       const float2 *tw, int tw_n, hipStream_t st) {
  hipError_t e = launch_fft_rows_inplace(data, volumes * n0 * n1, n2, inverse, tw, tw_n, st);
  if (e != hipSuccess) return e;
  e = launch_fft_cols_inplace(data, volumes * n0, n1, n2, inverse, tw, tw_n, st);
  if (e != hipSuccess) return e;
  return launch_fft_cols_inplace(data, volumes, n0, n1 * n2, inverse, tw, tw_n, st);
}

hipError_t launch3_real_to_complex(const float *x, float2 *out, long total, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_real_to_complex", total * 12.0, 0.0, st);
  hipLaunchKernelGGL(k3_real_to_complex, dim3(blocks_for(total)), dim3(256), 0, st, x, out, total);
  return hipGetLastError();
}

hipError_t launch3_mul_table(const float2 *src, const float *filt, float2 *dst, long volumes, long n,
                             hipStream_t st, bool accumulate) {
  const long total = volumes * n;
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_mul_table", total * (accumulate ? 24.0 : 16.0) + n * 4.0, total * 2.0, st);
  hipLaunchKernelGGL(k3_mul_table, dim3(blocks_for(total)), dim3(256), 0, st, src, filt, dst, total, n, accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch3_tile_phi(const float2 *Gs, const float *phi, float2 *dst, long volumes, int K,
                            int chan, int n0, int n1, int n2, int J, bool accumulate, hipStream_t st) {
  const long total = volumes * n0 * n1 * n2;
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_tile_phi", total * (accumulate ? 16.0 : 8.0) + 4.0 * n0 * n1 * n2, total * 2.0,
                  st);
  hipLaunchKernelGGL(k3_tile_phi, dim3(blocks_for(total)), dim3(256), 0, st, Gs, phi, dst, volumes, K,
                     chan, n0, n1, n2, J, accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch3_rho_back(const float2 *gu, const float *acc, float2 *y, long total,
                            hipStream_t st) {
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_rho_back", total * 28.0, total * 4.0, st);
  hipLaunchKernelGGL(k3_rho_back, dim3(blocks_for(total)), dim3(256), 0, st, gu, acc, y, total);
  return hipGetLastError();
}

hipError_t launch3_accum_abs2(const float2 *y, float *acc, long total, bool first, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_accum_abs2", total * (first ? 12.0 : 16.0), total * 4.0, st);
  hipLaunchKernelGGL(k3_accum_abs2, dim3(blocks_for(total)), dim3(256), 0, st, y, acc, total,
                     first ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch3_sqrt(const float *acc, float2 *out, long total, hipStream_t st) {
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_sqrt", total * 12.0, total * 1.0, st);
  hipLaunchKernelGGL(k3_sqrt, dim3(blocks_for(total)), dim3(256), 0, st, acc, out, total);
  return hipGetLastError();
}

hipError_t launch3_sample(const float2 *src, float *out, long volumes, int K, int chan, int n0,
                          int n1, int n2, int J, hipStream_t st) {
  const long total = volumes * (n0 >> J) * (n1 >> J) * (n2 >> J);
  if (total <= 0) return hipSuccess;
  LaunchScope obs("k3_sample", total * 12.0, 0.0, st);
  hipLaunchKernelGGL(k3_sample, dim3(blocks_for(total)), dim3(256), 0, st, src, out, volumes, K, chan,
                     n0, n1, n2, J);
  return hipGetLastError();
}

}  // namespace scat
