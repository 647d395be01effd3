// Backward pass of 2-D plans whose every node is one workgroup: grids of at most 128 x 128 points,
// square or 2 : 1, with no node below 16 a side.
//
// A node's adjoint recomputes its signal from its source's half spectrum (no tape, no taped forward
// pass: only the first-order moduli with children are formed again), sums its lowpass term and its
// children's gradient spectra, and goes through the modulus, all in the registers and the LDS of
// its N1 N2 / 16 threads.  The passes that serve these plans otherwise (taped row and column passes,
// k_rows2d_adj, k_node_modback) write and read a complex value per point four times more, and at a
// small batch are launches of a few dozen workgroups.  Backward pass, passes -> here (L = 8): 128
// planes of 32 x 32, J = 2, 204 -> 84 us, 2048 of them 1160 -> 604 us; 512 of 64 x 64, J = 3, 1457 -> 938 us;
// 100 of 128 x 128, J = 3, 994 -> 881 us, J = 2, 619 -> 614 us (one workgroup a compute unit at octave 0:
// the smallest gain; plane_pays in scat_capi.hip has the line); one of 64 x 64 254 -> 152 us.  Error
// against 64 bits the same (20 shapes, 4 inputs each: 0.99 of the passes' on average).
// What bounds it is the children's spectra and wavelets, read through L2 by every parent.
#include <hip/hip_runtime.h>

#include <string>

#include "fft_regs.hpp"
#include "scat_kernels.hpp"

namespace scat {

namespace {

// N1 x N2 points on N1 N2 / 16 threads, 16 each.  Column layout: column c = q % N2, rows
// t1 + T1 i; row layout: row r = q / T2, columns t + T2 i.  (the LDS strides are those of k_node_rect)
template <int N1, int N2>
struct Plane {
  static constexpr int T1 = N1 / 16, T2 = N2 / 16;
  static constexpr int TS = N1 * N2 / 16;
  static constexpr int NT = TS < 256 ? 256 : TS;
  static constexpr int SPW = NT / TS;
  static constexpr int RS = N2 + N2 / 16;
  static constexpr bool WAVE = TS <= 64;
  static constexpr size_t lds_bytes = (static_cast<size_t>(SPW) * N1 * RS + N1 + N2) * sizeof(float2);
  static_assert(TS >= 16 && TS <= 1024 && lds_bytes <= 160 * 1024, "plane shape");

  // q: this thread in its plane; area: the plane's LDS; tab: see twiddles()
  struct At {
    int r, t, c, t1;
    float2 *area;
    const float2 *tab;
  };
  static __device__ __forceinline__ At at(float2 *lds) {
    const int slab = TS >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / TS) : threadIdx.x / TS;
    const int q = threadIdx.x % TS;
    At a;
    a.r = q / T2;
    a.t = q % T2;
    a.c = q % N2;
    a.t1 = N2 >= 64 ? __builtin_amdgcn_readfirstlane(q / N2) : q / N2;
    a.area = lds + slab * (N1 * RS);
    a.tab = lds + SPW * (N1 * RS);
    return a;
  }
  static __device__ __forceinline__ void twiddles(float2 *lds, const float2 *__restrict__ tw, int tw_n) {
    float2 *tab = lds + SPW * (N1 * RS);
    for (int i = threadIdx.x; i < N2; i += NT) tab[i] = tw[(i / T2) * (i % T2) * (tw_n / N2)];
    for (int i = threadIdx.x; i < N1; i += NT) tab[N2 + i] = tw[(i / T1) * (i % T1) * (tw_n / N1)];
    __syncthreads();
  }
  // spectrum in column layout -> signal in row layout, and back
  static __device__ __forceinline__ void inverse(float2 (&v)[16], const At &a) {
    fft_core_tab<16, T1, true, WAVE>(v, a.t1, a.area + a.c, T1 * RS, RS, a.tab + N2 + a.t1, T1);
#pragma unroll
    for (int i = 0; i < 16; ++i) a.area[(a.t1 + T1 * i) * RS + a.c] = v[i];
    group_sync<WAVE>();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = a.area[a.r * RS + a.t + T2 * i];
    group_sync<WAVE>();
    fft_core_tab<16, T2, true, WAVE>(v, a.t, a.area + a.r * RS, T2, 1, a.tab + a.t, T2);
  }
  static __device__ __forceinline__ void forward(float2 (&v)[16], const At &a) {
    fft_core_tab<16, T2, false, WAVE>(v, a.t, a.area + a.r * RS, T2, 1, a.tab + a.t, T2);
#pragma unroll
    for (int i = 0; i < 16; ++i) a.area[a.r * RS + a.t + T2 * i] = v[i];
    group_sync<WAVE>();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = a.area[(a.t1 + T1 * i) * RS + a.c];
    group_sync<WAVE>();
    fft_core_tab<16, T1, false, WAVE>(v, a.t1, a.area + a.c, T1 * RS, RS, a.tab + N2 + a.t1, T1);
  }
};

struct PlaneKid {
  const float2 *g;                  // [nodes][L][Mr][Mc] gradient spectra
  const float *filt;                // [L][N1][N2]
  const unsigned long long *mask;   // [L][3]: word 2, blocks of N1 / 16 rows in use
  int Mr, Mc;
};

struct PlaneArgs {
  const float2 *src;               // [NS][Sr/2+1][Sc]
  const float *filt;               // [F][Sr][Sc]
  const unsigned long long *mask;  // [F][3]: words 0, 1, alias blocks in use by the node's upper, lower half
  float2 *dst;                     // forward: half spectra; adjoint: spectra
  const float2 *gh;                // spectra of the output gradients [planes][K][m_r][m_c]
  const float *phi_r, *phi_c;
  unsigned nodes, blocks;
  int F, G, Sr, lgA, chan_base, chan_src, K, m_r, m_c, kids, L;
  PlaneKid kid[kPlaneMaxOctaves];
  const float2 *tw;
  int tw_n;
};

// Each XCD (workgroups are dealt to the eight in turn) takes a contiguous run of nodes, filter
// fastest: the filters of a source, and the children of a node, meet in one L2.
template <int N1, int N2, bool BACK>
__global__ __launch_bounds__((Plane<N1, N2>::NT), (Plane<N1, N2>::TS > 512 || !BACK ? 4 : 3)) void k_plane_nodes(
    PlaneArgs a) {
  using P = Plane<N1, N2>;
  constexpr int T1 = P::T1, TS = P::TS;
  extern __shared__ __attribute__((aligned(16))) float2 lds[];
  const unsigned blk = (blockIdx.x & 7) * (a.blocks >> 3) + (blockIdx.x >> 3);
  if (blk * P::SPW >= a.nodes) return;  // (all threads of the workgroup)
  const unsigned slab = TS >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / TS) : threadIdx.x / TS;
  const bool live = blk * P::SPW + slab < a.nodes;
  const unsigned node = live ? blk * P::SPW + slab : a.nodes - 1;  // idle slabs shadow the last node, store nothing
  const unsigned s = node / static_cast<unsigned>(a.F);
  const int f = static_cast<int>(node - s * a.F);
  const typename P::At at = P::at(lds);
  P::twiddles(lds, a.tw, a.tw_n);

  // ---- spectrum of the node, as in k_node_rect
  float2 v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = make_float2(0.f, 0.f);
  {
    const int Sr = a.Sr, Sc = N2 << a.lgA, A = 1 << a.lgA;
    const float2 *src = a.src + static_cast<size_t>(s) * (Sr / 2 + 1) * Sc;
    const float *filt = a.filt + static_cast<size_t>(f) * Sr * Sc;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      unsigned long long rem = a.mask[3 * f + h];
      while (rem != 0ull) {
        const int bit = __ffsll(static_cast<long long>(rem)) - 1;
        rem &= rem - 1ull;
        const int ar = bit >> a.lgA, ac = bit & (A - 1);
        const int kc = at.c + N2 * ac, kcm = (Sc - kc) & (Sc - 1);
        float2 x[8];
        float w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          // rows above Sr / 2 are the conjugates of the stored ones
          const int kr = at.t1 + T1 * (8 * h + i) + N1 * ar;
          const bool mir = kr > Sr / 2;
          x[i] = src[(mir ? Sr - kr : kr) * Sc + (mir ? kcm : kc)];
          w[i] = filt[kr * Sc + kc];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const bool mir = at.t1 + T1 * (8 * h + i) + N1 * ar > Sr / 2;
          float2 &z = v[8 * h + i];
          z.x = fmaf(x[i].x, w[i], z.x);
          z.y = fmaf(x[i].y, mir ? -w[i] : w[i], z.y);
        }
      }
    }
  }
  P::inverse(v, at);

  if constexpr (!BACK) {
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = make_float2(__builtin_amdgcn_sqrtf(v[i].x * v[i].x + v[i].y * v[i].y), 0.f);
    P::forward(v, at);
    if (live) {
      float2 *up = a.dst + static_cast<size_t>(node) * (N1 / 2 + 1) * N2 + at.c;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (at.t1 + T1 * i <= N1 / 2) up[(at.t1 + T1 * i) * N2] = v[i];
    }
  } else {
    float2 y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = v[i];
    // ---- gradient spectrum: own lowpass term, then the children's
    {
      const unsigned plane = s / static_cast<unsigned>(a.G);
      const size_t row = static_cast<size_t>(plane) * a.K + a.chan_base + (s - plane * a.G) * a.chan_src + f;
      const float2 *gh = a.gh + row * (a.m_r * a.m_c) + (at.c & (a.m_c - 1));
      const float pc = a.phi_c[at.c];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kr = at.t1 + T1 * i;
        const float2 z = gh[(kr & (a.m_r - 1)) * a.m_c];
        const float w = a.phi_r[kr] * pc;
        v[i] = make_float2(w * z.x, w * z.y);
      }
    }
    for (int o = 0; o < a.kids; ++o) {
      const PlaneKid &kd = a.kid[o];
      const int Mr = kd.Mr, Mc = kd.Mc;
      const float2 *kg = kd.g + static_cast<size_t>(node) * a.L * (Mr * Mc) + (at.c & (Mc - 1));
      const float *filt = kd.filt + at.c;
      for (int l = 0; l < a.L; ++l, kg += Mr * Mc, filt += N1 * N2) {
        const unsigned use = static_cast<unsigned>(kd.mask[3 * l + 2]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if ((use >> (8 * h) & 255u) == 0u) continue;
          float2 z[8];
          float w[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int kr = at.t1 + T1 * (8 * h + i);
            z[i] = kg[(kr & (Mr - 1)) * Mc];
            w[i] = filt[kr * N2];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            v[8 * h + i].x = fmaf(w[i], z[i].x, v[8 * h + i].x);
            v[8 * h + i].y = fmaf(w[i], z[i].y, v[8 * h + i].y);
          }
        }
      }
    }
    P::inverse(v, at);
    // ---- through the modulus
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float r = over_sqrt(v[i].x, y[i].x * y[i].x + y[i].y * y[i].y);
      v[i] = make_float2(y[i].x * r, y[i].y * r);
    }
    P::forward(v, at);
    if (live) {
      float2 *up = a.dst + static_cast<size_t>(node) * (N1 * N2) + at.c;
#pragma unroll
      for (int i = 0; i < 16; ++i) up[(at.t1 + T1 * i) * N2] = v[i];
    }
  }
}

// IN: planes -> half spectra; else spectra -> real parts
template <int N1, int N2, bool IN>
__global__ __launch_bounds__((Plane<N1, N2>::NT), 4) void k_plane_end(const float *__restrict__ xin, float *__restrict__ xout,
                                                                      const float2 *__restrict__ sin,
                                                                      float2 *__restrict__ sout, unsigned planes,
                                                                      const float2 *__restrict__ tw, int tw_n) {
  using P = Plane<N1, N2>;
  extern __shared__ __attribute__((aligned(16))) float2 lds[];
  const unsigned want = blockIdx.x * P::SPW + threadIdx.x / P::TS;
  const bool live = want < planes;
  const size_t n = live ? want : planes - 1;
  const typename P::At at = P::at(lds);
  P::twiddles(lds, tw, tw_n);
  float2 v[16];
  if constexpr (IN) {
    const float *x = xin + n * (N1 * N2) + at.r * N2 + at.t;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = make_float2(x[P::T2 * i], 0.f);
    P::forward(v, at);
    if (live) {
      float2 *up = sout + n * ((N1 / 2 + 1) * N2) + at.c;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (at.t1 + P::T1 * i <= N1 / 2) up[(at.t1 + P::T1 * i) * N2] = v[i];
    }
  } else {
    const float2 *x = sin + n * (N1 * N2) + at.c;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = x[(at.t1 + P::T1 * i) * N2];
    P::inverse(v, at);
    if (live) {
      float *o = xout + n * (N1 * N2) + at.r * N2 + at.t;
#pragma unroll
      for (int i = 0; i < 16; ++i) o[P::T2 * i] = v[i].x;
    }
  }
}

// Gradient spectrum of the input, one thread a frequency: lowpass term plus, for each first-order
// wavelet that is not negligible on this block of 256 frequencies, its node's gradient spectrum.
struct PlaneSumArgs {
  float2 *dst;
  const float2 *gh;
  const float *phi_r, *phi_c, *filt;
  const int *list;  // per block: where its wavelets start (blocks + 1 entries), then the wavelets
  const float2 *g[kPlaneMaxOctaves];
  signed char res[kPlaneMaxOctaves];
  unsigned long long total;
  int lgR, lgC, m_r, m_c, K, L;
};

__global__ __launch_bounds__(256) void k_plane_sum(PlaneSumArgs a) {
  const unsigned long long at = static_cast<unsigned long long>(blockIdx.x) * 256 + threadIdx.x;  // 256 divides the plane
  if (at >= a.total) return;
  const int lgN = a.lgR + a.lgC;
  const size_t s = at >> lgN;
  const int k = static_cast<int>(at & ((1u << lgN) - 1));
  const int kr = k >> a.lgC, kc = k & ((1 << a.lgC) - 1);
  const int blk = __builtin_amdgcn_readfirstlane(k >> 8);
  const float2 z0 = a.gh[(s * a.K * a.m_r + (kr & (a.m_r - 1))) * a.m_c + (kc & (a.m_c - 1))];
  const float w0 = a.phi_r[kr] * a.phi_c[kc];
  float2 acc = make_float2(w0 * z0.x, w0 * z0.y);
#pragma unroll 4
  for (int e = a.list[blk]; e < a.list[blk + 1]; ++e) {
    const int f = a.list[e], j = f / a.L, res = a.res[j];
    const int Mr = 1 << (a.lgR - res), lgc = a.lgC - res;
    const float2 z = a.g[j][(((s * a.L + (f - j * a.L)) * Mr + (kr & (Mr - 1))) << lgc) + (kc & ((1 << lgc) - 1))];
    const float w = a.filt[(static_cast<size_t>(f) << lgN) + k];
    acc.x = fmaf(w, z.x, acc.x);
    acc.y = fmaf(w, z.y, acc.y);
  }
  a.dst[at] = acc;
}

int lg2i(int n) {
  int r = 0;
  while ((1 << r) < n) ++r;
  return r;
}

template <int N1, int N2, bool BACK>
hipError_t run_nodes(PlaneArgs &a, hipStream_t st) {
  using P = Plane<N1, N2>;
  a.blocks = ((a.nodes + P::SPW - 1) / P::SPW + 7) / 8 * 8;
  const double pts = static_cast<double>(N1) * N2, nd = a.nodes;
  const std::string name = "k_plane_nodes<" + std::to_string(N1) + ", " + std::to_string(N2) + (BACK ? ", true>" : ", false>");
  const double spts = static_cast<double>(a.Sr) * (N2 << a.lgA);
  double bytes = nd / a.F * spts * 4 + a.F * spts * 4 + nd * pts * (BACK ? 8 : 4);
  for (int o = 0; o < a.kids; ++o) bytes += nd * a.L * a.kid[o].Mr * a.kid[o].Mc * 8.0 + a.L * pts * 4;
  if (BACK) bytes += nd * a.m_r * a.m_c * 8.0;
  // transforms, filter product, modulus; adjoint: lowpass and children's products
  LaunchScope obs(name.c_str(), bytes,
                  nd * (5.0 * pts * lg2i(N1 * N2) * (BACK ? 3 : 1.5) + 4.0 * spts + 4.0 * pts +
                        (BACK ? 4.0 * pts * (1 + a.kids * a.L) : 0.0)),
                  st);
  if (P::lds_bytes > 65536) {
    static unsigned long long ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k_plane_nodes<N1, N2, BACK>), ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_plane_nodes<N1, N2, BACK>), dim3(a.blocks), dim3(P::NT), P::lds_bytes, st, a);
  return hipGetLastError();
}

template <int N1, int N2, bool IN>
hipError_t run_end(const float *xin, float *xout, const float2 *sin, float2 *sout, unsigned planes, const float2 *tw,
                   int tw_n, hipStream_t st) {
  using P = Plane<N1, N2>;
  const std::string name = "k_plane_end<" + std::to_string(N1) + ", " + std::to_string(N2) + (IN ? ", true>" : ", false>");
  const double pts = static_cast<double>(N1) * N2 * planes;
  LaunchScope obs(name.c_str(), pts * (IN ? 8 : 12), pts * (IN ? 2.5 : 5.0) * lg2i(N1 * N2), st);
  if (P::lds_bytes > 65536) {
    static unsigned long long ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k_plane_end<N1, N2, IN>), ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_plane_end<N1, N2, IN>), dim3((planes + P::SPW - 1) / P::SPW), dim3(P::NT), P::lds_bytes, st, xin,
                     xout, sin, sout, planes, tw, tw_n);
  return hipGetLastError();
}

bool pow2i(int n) { return n > 0 && (n & (n - 1)) == 0; }

#define SCAT_PLANES(N1_, N2_, CALL)                      \
  switch ((N1_) << 12 | (N2_)) {                         \
    case 16 << 12 | 16: return CALL(16, 16);             \
    case 16 << 12 | 32: return CALL(16, 32);             \
    case 32 << 12 | 16: return CALL(32, 16);             \
    case 32 << 12 | 32: return CALL(32, 32);             \
    case 32 << 12 | 64: return CALL(32, 64);             \
    case 64 << 12 | 32: return CALL(64, 32);             \
    case 64 << 12 | 64: return CALL(64, 64);             \
    case 64 << 12 | 128: return CALL(64, 128);           \
    case 128 << 12 | 64: return CALL(128, 64);           \
    case 128 << 12 | 128: return CALL(128, 128);         \
    default: return hipErrorInvalidValue;                \
  }

}  // namespace

bool plane_supported(int N1, int N2) {
  return pow2i(N1) && pow2i(N2) && N1 >= 16 && N2 >= 16 && N1 <= 128 && N2 <= 128 && N1 <= 2 * N2 && N2 <= 2 * N1;
}

hipError_t launch_plane_nodes(const PlaneNodes &n, bool back, hipStream_t st) {
  if (!plane_supported(n.N1, n.N2) || !pow2i(n.A) || n.A > 8 || n.NS < 1 || n.F < 1 || n.G < 1 || n.kids < 0 ||
      n.kids > kPlaneMaxOctaves || n.NS > 0x7fff0000L / n.F || n.tw_n % n.N1 != 0 || n.tw_n % n.N2 != 0 ||
      (back && (n.gh == nullptr || !pow2i(n.m_r) || !pow2i(n.m_c) || n.m_r > n.N1 || n.m_c > n.N2)))
    return hipErrorInvalidValue;
  PlaneArgs a{};
  a.src = n.src;
  a.filt = n.filt;
  a.mask = n.mask;
  a.dst = n.dst;
  a.gh = n.gh;
  a.phi_r = n.phi_r;
  a.phi_c = n.phi_c;
  a.nodes = static_cast<unsigned>(n.NS * n.F);
  a.F = n.F;
  a.G = n.G;
  a.Sr = n.N1 * n.A;
  a.lgA = lg2i(n.A);
  a.chan_base = n.chan_base;
  a.chan_src = n.chan_src;
  a.K = n.K;
  a.m_r = n.m_r;
  a.m_c = n.m_c;
  a.kids = n.kids;
  a.L = n.L;
  for (int o = 0; o < n.kids; ++o) {
    if (!pow2i(n.kid[o].Mr) || !pow2i(n.kid[o].Mc) || n.kid[o].Mr > n.N1 || n.kid[o].Mc > n.N2) return hipErrorInvalidValue;
    a.kid[o] = PlaneKid{n.kid[o].g, n.kid[o].filt, n.kid[o].mask, n.kid[o].Mr, n.kid[o].Mc};
  }
  a.tw = n.tw;
  a.tw_n = n.tw_n;
#define SCAT_CALL(X, Y) (back ? run_nodes<X, Y, true>(a, st) : run_nodes<X, Y, false>(a, st))
  SCAT_PLANES(n.N1, n.N2, SCAT_CALL)
#undef SCAT_CALL
}

hipError_t launch_plane_in(const float *x, float2 *spec, long planes, int N1, int N2, const float2 *tw, int tw_n,
                           hipStream_t st) {
  if (planes < 1 || planes > 0x7fffffffL || tw_n % N1 != 0 || tw_n % N2 != 0) return hipErrorInvalidValue;
  const unsigned n = static_cast<unsigned>(planes);
#define SCAT_CALL(X, Y) (run_end<X, Y, true>(x, nullptr, nullptr, spec, n, tw, tw_n, st))
  SCAT_PLANES(N1, N2, SCAT_CALL)
#undef SCAT_CALL
}

hipError_t launch_plane_real(const float2 *spec, float *out, long planes, int N1, int N2, const float2 *tw, int tw_n,
                             hipStream_t st) {
  if (planes < 1 || planes > 0x7fffffffL || tw_n % N1 != 0 || tw_n % N2 != 0) return hipErrorInvalidValue;
  const unsigned n = static_cast<unsigned>(planes);
#define SCAT_CALL(X, Y) (run_end<X, Y, false>(nullptr, out, spec, nullptr, n, tw, tw_n, st))
  SCAT_PLANES(N1, N2, SCAT_CALL)
#undef SCAT_CALL
}

hipError_t launch_plane_sum(const PlaneSum &s, hipStream_t st) {
  if (s.planes < 1 || s.J < 1 || s.J > kPlaneMaxOctaves || !plane_supported(s.N1, s.N2)) return hipErrorInvalidValue;
  PlaneSumArgs a{};
  a.dst = s.dst;
  a.gh = s.gh;
  a.phi_r = s.phi_r;
  a.phi_c = s.phi_c;
  a.filt = s.filt;
  a.list = s.list;
  for (int j = 0; j < s.J; ++j) {
    a.g[j] = s.g[j];
    a.res[j] = static_cast<signed char>(s.res[j]);
  }
  a.lgR = lg2i(s.N1);
  a.lgC = lg2i(s.N2);
  a.total = static_cast<unsigned long long>(s.planes) << (a.lgR + a.lgC);
  a.m_r = s.m_r;
  a.m_c = s.m_c;
  a.K = s.K;
  a.L = s.L;
  const unsigned long long blocks = (a.total + 255) / 256;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  const double n = static_cast<double>(s.N1) * s.N2, planes = static_cast<double>(s.planes);
  double bytes = planes * 8.0 * (n + s.m_r * s.m_c) + 4.0 * n * (1 + s.J * s.L);
  for (int j = 0; j < s.J; ++j) bytes += planes * 8.0 * s.L * (s.N1 >> s.res[j]) * (s.N2 >> s.res[j]);
  LaunchScope obs("k_plane_sum", bytes, planes * 4.0 * (n + 256.0 * s.listed), st);
  hipLaunchKernelGGL(k_plane_sum, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
  return hipGetLastError();
}

#undef SCAT_PLANES

}  // namespace scat
