// Whole nodes of the 1-D cascade: plans whose periodic grid has at most 8192 samples.
//
// Spectra are kept in natural order, real signals' as half spectra [M/2+1].  M / 16 threads hold a
// node of M samples, 16 each: filter product with the source's half spectrum +
// periodisation, inverse transform, modulus, forward transform, and from the spectrum in LDS the
// folded product with phi (half spectrum of the output grid) and the half spectrum for the children.
// The adjoint of a node is one workgroup too: it recomputes its signal from the source's spectrum (no
// tape), sums its lowpass term and its children's gradient spectra, and goes through the modulus.
// One launch takes all nodes of an order, whatever their length.
//
// Why: the schedule of four-step passes launches every octave's and every pair of octaves' row
// and column pass by itself; at 32 signals of 8192 a launch has 32 ... 512 workgroups and takes the
// latency of its own load-transform-store chain (5 ... 30 us, 85 launches in a training step), and at
// large batches every pass goes through memory.  Measured, passes -> here: training step of 32
// signals of 5000 samples (J 5, Q 8) 827 -> 195 us; forward / backward of 600 x 8192 (J 5, Q 8) 1609 ->
// 610 / 2874 -> 1724 us, 2048 x 2048 (J 4, Q 8) 1548 -> 408 / 2693 -> 1175 us, one signal of 2048 190 ->
// 27 / 345 -> 56 us: no size, batch or oversampling was found where the passes are the better ones.
// Error against 64 bits (40 shapes, 4 inputs each): 0.93 of the passes' forward (0.83 ... 1.07 by shape),
// 0.97 backward (0.86 ... 1.10; 1.7e-7 ... 4.6e-7).
// What bounds it at large batches is the LDS exchanges (two a transform) and the source and filter reads
// through L2; at small ones the chain of eleven launches.
#include <hip/hip_runtime.h>

#include <string>

#include "fft_regs.hpp"
#include "pad.hpp"
#include "scat_kernels.hpp"

namespace scat {

namespace {

// M = 2^LG samples, 16 per thread: thread q holds x[q + T i] in v[i] before a transform and X[q + T i]
// after it; NT threads a workgroup.  Up to 256 samples one fft_core; above, a radix-16 stage across the
// threads, an exchange, and 16 transforms of T samples (thread q: number q % 16, thread q / 16 of its T / 16);
// at 8192 samples those are 16 x 32, the 32 points by pairs of lanes, after a second exchange.
template <int LG, int NT>
struct Line {
  static constexpr int M = 1 << LG;
  static constexpr int E = 16;
  static constexpr int T = M / E;
  static constexpr bool ONE = M <= 256;
  static constexpr bool PAIR = LG == 13;
  static constexpr bool WAVE = T <= 64;
  static constexpr int SPW = NT / T;
  // row strides of the two exchanges: a half-wavefront's E (or E x 2) rows on distinct banks
  static constexpr int S1 = ONE ? (T >= 8 ? T + 1 : T) : PAIR ? T + 16 : T + 2;
  static constexpr int S2 = PAIR ? 34 : T >= 128 ? T + 16 : T + 2;
  static constexpr int SLOT = PAIR ? 256 * S2 : E * (!ONE && S2 > S1 ? S2 : S1);
  static constexpr size_t lds_bytes = static_cast<size_t>(SPW) * SLOT * sizeof(float2);
  static_assert(LG >= 4 && LG <= 13 && SLOT >= M && SLOT >= E * S1 && SPW >= 1, "line length");

  // Thread number of a slab's thread (PAIR: that of the transform's last stage, lanes 2 u and 2 u + 1)
  static __device__ __forceinline__ int number(int th) { return PAIR ? (th >> 1) + 256 * (th & 1) : th; }

  // tw: the tables of line_twiddles(); every thread of the workgroup calls it
  template <bool INV>
  static __device__ __forceinline__ void fft(float2 (&v)[E], int q, float2 *slot, const float2 *__restrict__ tw) {
    const float2 *main = tw + 2 * M;
    if constexpr (ONE) {
      fft_core_tab<E, T, INV, true>(v, q, slot, S1, 1, main + q, T);
    } else if constexpr (PAIR) {
      DftRegs<E, INV>::run(v);
#pragma unroll
      for (int i = 1; i < E; ++i) {
        float2 w = main[i * T + q];
        if (INV) w.y = -w.y;
        v[i] = c_mul(v[i], w);
      }
      // (the upper half of a row 16 elements further: a pair's lanes on different banks)
#pragma unroll
      for (int i = 0; i < E; ++i) slot[i * S1 + q + 16 * (q >> 8)] = v[i];
      __syncthreads();
      const int th = threadIdx.x, k1 = th >> 5, t = th & 31;
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = slot[k1 * S1 + t + 32 * i + 16 * (i >> 3)];
      __syncthreads();
      DftRegs<E, INV>::run(v);
#pragma unroll
      for (int i = 1; i < E; ++i) {
        float2 w = main[M + i * 32 + t];
        if (INV) w.y = -w.y;
        v[i] = c_mul(v[i], w);
      }
#pragma unroll
      for (int i = 0; i < E; ++i) slot[(16 * i + k1) * S2 + t] = v[i];
      __syncthreads();
      const int tp = th & 1;
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = slot[(th >> 1) * S2 + tp + 2 * i];
      __syncthreads();
      PairTw pw;
      pair_twiddles(pw, tp);
      fft32_pair<INV>(v, tp, pw);
    } else {
      constexpr int TT = T / E;
      const int k1 = q % E, t = q / E;
      DftRegs<E, INV>::run(v);
#pragma unroll
      for (int i = 1; i < E; ++i) {
        float2 w = main[i * T + q];
        if (INV) w.y = -w.y;
        v[i] = c_mul(v[i], w);
      }
#pragma unroll
      for (int i = 0; i < E; ++i) slot[i * S1 + q] = v[i];
      group_sync<WAVE>();
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = slot[k1 * S1 + t + TT * i];
      group_sync<WAVE>();
      fft_core_tab<E, TT, INV, WAVE>(v, t, slot + k1, S2, E, main + M + t, TT);
    }
  }
};

struct NodeSeg {
  const float2 *src;               // [sources][S/2+1]
  const float *filt;               // [F][S]
  const unsigned long long *mask;  // [F][2]: alias blocks in use, lower and upper half of the node's spectrum
  const float *phi;                // [M]
  float2 *dst;                     // forward: half spectra for the children or null; backward: [nodes][M]
  unsigned nodes, first_block, blocks;
  int F, G, base, stride;          // node -> channel base + (node % G) stride of signal node / G
  unsigned phi_mask;
  short kid0, kids;                // backward
  signed char lgM, lgA, reach;
};

struct NodeKid {
  const float2 *g;    // [nodes][Mc]
  const float *filt;  // [M]
  unsigned mask;
  int lgM;
};

struct NodeArgs {
  NodeSeg seg[kLineMaxSegs];
  NodeKid kid[kLineMaxSegs];
  float2 *low;  // forward: written (null: not formed); backward: spectra of the output gradients; [.][m/2+1]
  const float2 *tw;
  int n, lgm, K;
};
static_assert(sizeof(NodeArgs) <= 4000, "kernel arguments");

// phi times the spectrum in `slot`, folded to the output grid
template <int LG, int NT>
__device__ __forceinline__ void fold_low(const float2 *slot, const float *__restrict__ phi, float2 *dst, int q, int lgm,
                                         int reach) {
  constexpr int M = Line<LG, NT>::M, T = Line<LG, NT>::T;
  const int m = 1 << lgm, A = M >> lgm;
  const int a0 = 2 * reach + 1 >= A ? 0 : -reach, cnt = 2 * reach + 1 >= A ? A : 2 * reach + 1;
  for (int k0 = q; k0 <= m / 2; k0 += T) {
    float2 s = make_float2(0.f, 0.f);
    for (int a = 0; a < cnt; ++a) {
      const int k = (k0 + m * (a0 + a)) & (M - 1);
      const float w = phi[k];
      const float2 z = slot[k];
      s.x = fmaf(w, z.x, s.x);
      s.y = fmaf(w, z.y, s.y);
    }
    dst[k0] = s;
  }
}

template <int LG, bool BACK, int NT>
__device__ __forceinline__ void line_node(const NodeArgs &a, const NodeSeg &g, unsigned blk, float2 *lds) {
  using L = Line<LG, NT>;
  constexpr int M = L::M, E = L::E, T = L::T, H = E / 2;
  const int slab = T >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / T) : threadIdx.x / T;
  const int q = L::number(threadIdx.x % T);
  if (blk * L::SPW >= g.nodes) return;  // (all threads of the workgroup)
  const bool live = blk * L::SPW + slab < g.nodes;
  const unsigned node = live ? blk * L::SPW + slab : g.nodes - 1;  // idle slabs shadow the last node, store nothing
  const unsigned s = node / static_cast<unsigned>(g.F);
  const int f = static_cast<int>(node - s * g.F);
  float2 *slot = lds + slab * L::SLOT;
  const unsigned plane = node / static_cast<unsigned>(g.G);
  const size_t row = static_cast<size_t>(plane) * a.K + g.base + (node - plane * g.G) * g.stride;
  const int m = 1 << a.lgm;

  // ---- spectrum of the node: the alias blocks of either half on which the wavelet is not negligible
  float2 v[E];
#pragma unroll
  for (int i = 0; i < E; ++i) v[i] = make_float2(0.f, 0.f);
  {
    const int S = M << g.lgA;
    const float2 *src = g.src + static_cast<size_t>(s) * (S / 2 + 1);
    const float *filt = g.filt + static_cast<size_t>(f) * S;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      unsigned long long rem = g.mask[2 * f + h];
      while (rem != 0ull) {
        const int al = __ffsll(static_cast<long long>(rem)) - 1;
        rem &= rem - 1ull;
        float2 x[H];
        float w[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
          const int k = q + T * (H * h + i) + M * al;
          x[i] = src[k > S / 2 ? S - k : k];
          w[i] = filt[k];
        }
#pragma unroll
        for (int i = 0; i < H; ++i) {
          const int k = q + T * (H * h + i) + M * al;
          float2 &z = v[H * h + i];
          z.x = fmaf(x[i].x, w[i], z.x);
          z.y = fmaf(x[i].y, k > S / 2 ? -w[i] : w[i], z.y);
        }
      }
    }
  }
  L::template fft<true>(v, q, slot, a.tw);

  if constexpr (!BACK) {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = make_float2(__builtin_amdgcn_sqrtf(v[i].x * v[i].x + v[i].y * v[i].y), 0.f);
    L::template fft<false>(v, q, slot, a.tw);
    if (g.dst != nullptr && live) {
      float2 *up = g.dst + static_cast<size_t>(node) * (M / 2 + 1) + q;
#pragma unroll
      for (int i = 0; i < H; ++i) up[T * i] = v[i];
      if (q == 0) up[M / 2] = v[H];
    }
    if (a.low != nullptr) {
#pragma unroll
      for (int i = 0; i < E; ++i) slot[q + T * i] = v[i];
      group_sync<L::WAVE>();
      if (live) fold_low<LG, NT>(slot, g.phi, a.low + row * (m / 2 + 1), q, a.lgm, g.reach);
    }
  } else {
    float2 y[E];
#pragma unroll
    for (int i = 0; i < E; ++i) y[i] = v[i];
    // ---- gradient spectrum: own lowpass term, then the children's
    const float2 *gh = a.low + row * (m / 2 + 1);
#pragma unroll
    for (int i = 0; i < E; ++i) {
      v[i] = make_float2(0.f, 0.f);
      if (g.phi_mask >> i & 1u) {
        const int k = q + T * i, kk = k & (m - 1);
        const bool mir = kk > m / 2;
        const float2 z = gh[mir ? m - kk : kk];
        const float w = g.phi[k];
        v[i] = make_float2(w * z.x, mir ? -w * z.y : w * z.y);
      }
    }
    for (int c = g.kid0; c < g.kid0 + g.kids; ++c) {
      const NodeKid &kd = a.kid[c];
      const float2 *kg = kd.g + (static_cast<size_t>(node) << kd.lgM);
      const int wrap = (1 << kd.lgM) - 1;
#pragma unroll
      for (int b = 0; b < E; b += 4) {
        if ((kd.mask >> b & 15u) == 0u) continue;
#pragma unroll
        for (int i = b; i < b + 4; ++i) {
          const int k = q + T * i;
          const float2 z = kg[k & wrap];
          const float w = kd.filt[k];
          v[i].x = fmaf(w, z.x, v[i].x);
          v[i].y = fmaf(w, z.y, v[i].y);
        }
      }
    }
    L::template fft<true>(v, q, slot, a.tw);
    // ---- through the modulus
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const float r = over_sqrt(v[i].x, y[i].x * y[i].x + y[i].y * y[i].y);
      v[i] = make_float2(y[i].x * r, y[i].y * r);
    }
    L::template fft<false>(v, q, slot, a.tw);
    if (live) {
      float2 *up = g.dst + (static_cast<size_t>(node) << LG) + q;
#pragma unroll
      for (int i = 0; i < E; ++i) up[T * i] = v[i];
    }
  }
}

// All nodes of an order.  Each XCD (workgroups are dealt to the eight in turn) takes a contiguous run
// of a segment's nodes: the filters of a source meet in one L2.  BIG: some nodes have 8192 samples, 512
// threads; two workgroups of eight waves fit a compute unit (70 KB of LDS each).  With 256 threads of 32
// samples it was eight waves: 32 x 8192, J = 5, Q = 8 forward 58.1 -> 56.6 us, backward 138 -> 133; 200 x 7000, first
// order, 123 -> 118, 243 -> 222; 600 x 8192 611 -> 604, 1722 -> 1717.  The adjoint holds a node's signal beside
// its gradient: without BIG four waves a SIMD would spill and be slower than three; BIG has to have them, and
// with them 20 bytes of scratch a lane, in the times above (two waves, no scratch, one workgroup a compute unit: 32 x 8192
// 145 us, 600 x 8192 1913).
constexpr int line_threads(bool big) { return big ? 512 : 256; }
template <bool BACK, bool BIG>
__global__ __launch_bounds__(line_threads(BIG), BACK && !BIG ? 3 : 4) void k_line_nodes(NodeArgs a) {
  constexpr int NT = line_threads(BIG);
  extern __shared__ __attribute__((aligned(16))) float2 lds[];
  int i = 0;
  while (i + 1 < a.n && blockIdx.x >= a.seg[i + 1].first_block) ++i;
  const NodeSeg &g = a.seg[i];
  const unsigned b = blockIdx.x - g.first_block;
  const unsigned blk = (b & 7) * (g.blocks >> 3) + (b >> 3);
  switch (g.lgM) {
    case 5: return line_node<5, BACK, NT>(a, g, blk, lds);
    case 6: return line_node<6, BACK, NT>(a, g, blk, lds);
    case 7: return line_node<7, BACK, NT>(a, g, blk, lds);
    case 8: return line_node<8, BACK, NT>(a, g, blk, lds);
    case 9: return line_node<9, BACK, NT>(a, g, blk, lds);
    case 10: return line_node<10, BACK, NT>(a, g, blk, lds);
    case 11: return line_node<11, BACK, NT>(a, g, blk, lds);
    case 12: return line_node<12, BACK, NT>(a, g, blk, lds);
    case 13:
      if constexpr (BIG) line_node<13, BACK, NT>(a, g, blk, lds);
      return;
  }
}

// ---- transforms at the two ends of the cascade
enum { kIn, kOut, kGradOut, kGradIn };

struct EndArgs {
  const float *xin;  // kIn: signals [.][len]; kGradOut: output gradients [.][len]
  float *xout;       // kOut: outputs [.][len]; kGradIn: input gradients [.][len]
  const float2 *sin;
  float2 *sout;
  float2 *low;  // kIn: row s K of the output grid's half spectra, or null
  const float *phi;
  const float2 *tw;
  unsigned rows;
  int len, lgm, K, reach;
};

// kIn: signal (extended symmetrically to M samples) -> half spectrum (+ lowpass of order 0);
// kOut: half spectrum -> its first len real samples; kGradOut: len real samples and zeros -> half
// spectrum; kGradIn: full spectrum -> real part, folded back to the len samples that were extended.
template <int LG, int MODE>
__global__ __launch_bounds__(line_threads(LG == 13), 4) void k_line_end(EndArgs a) {
  constexpr int NT = line_threads(LG == 13);
  using L = Line<LG, NT>;
  constexpr int M = L::M, E = L::E, T = L::T, H = E / 2;
  extern __shared__ __attribute__((aligned(16))) float2 lds[];
  const int slab = threadIdx.x / T, q = L::number(threadIdx.x % T);
  const unsigned at = blockIdx.x * L::SPW + slab;
  const bool live = at < a.rows;
  const size_t r = live ? at : a.rows - 1;
  float2 *slot = lds + slab * L::SLOT;
  float2 v[E];
  if constexpr (MODE == kIn || MODE == kGradOut) {
    const float *x = a.xin + r * a.len;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int t = q + T * i;
      float u = 0.f;
      if (MODE == kIn)
        u = x[a.len == M ? t : pad_source(t, a.len, M)];
      else if (t < a.len)
        u = x[t];
      v[i] = make_float2(u, 0.f);
    }
    L::template fft<false>(v, q, slot, a.tw);
    if (live) {
      float2 *up = a.sout + r * (M / 2 + 1) + q;
#pragma unroll
      for (int i = 0; i < H; ++i) up[T * i] = v[i];
      if (q == 0) up[M / 2] = v[H];
    }
    if (MODE == kIn && a.low != nullptr) {
#pragma unroll
      for (int i = 0; i < E; ++i) slot[q + T * i] = v[i];
      group_sync<L::WAVE>();
      if (live) fold_low<LG, NT>(slot, a.phi, a.low + r * a.K * ((1 << a.lgm) / 2 + 1), q, a.lgm, a.reach);
    }
  } else {
    const float2 *x = a.sin + r * (MODE == kOut ? M / 2 + 1 : M);
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int k = q + T * i;
      if (MODE == kOut && k > M / 2) {
        v[i] = x[M - k];
        v[i].y = -v[i].y;
      } else {
        v[i] = x[k];
      }
    }
    L::template fft<true>(v, q, slot, a.tw);
    float *o = a.xout + r * a.len;
    if (MODE == kOut || a.len == M) {
      if (live) {
#pragma unroll
        for (int i = 0; i < E; ++i)
          if (q + T * i < a.len) o[q + T * i] = v[i].x;
      }
    } else {
      float *line = reinterpret_cast<float *>(slot);
#pragma unroll
      for (int i = 0; i < E; ++i) line[q + T * i] = v[i].x;
      group_sync<L::WAVE>();
      if (live)
        for (int t = q; t < a.len; t += T) {
          float acc = 0.f;
          for_each_image(t, a.len, M, [&](int p) { acc += line[p]; });
          o[t] = acc;
        }
    }
  }
}

// ---- gradient spectrum of the input: lowpass term plus, for each first-order wavelet that is not
// negligible on this block of 256 frequencies, its node's gradient spectrum.  One thread a frequency:
// a workgroup per signal would leave most of the chip idle at the batches of a training step.
struct SumArgs {
  float2 *dst;              // [signals][N]
  const float2 *gh;         // row s K: the gradient of order 0
  const float *phi, *filt;  // [N], [wavelets][N]
  const int *list;          // per block: where its wavelets start (blocks + 1 entries), then the wavelets
  const float2 *g[kLineMaxOctaves];
  signed char lgM[kLineMaxOctaves];
  unsigned long long total;
  int lgN, lgm, K, Q;
};

__global__ __launch_bounds__(256) void k_line_sum(SumArgs a) {
  const unsigned long long at = static_cast<unsigned long long>(blockIdx.x) * 256 + threadIdx.x;
  if (at >= a.total) return;
  const size_t s = at >> a.lgN;
  const int k = static_cast<int>(at & ((1u << a.lgN) - 1));
  const int blk = __builtin_amdgcn_readfirstlane(k >> 8);
  const int m = 1 << a.lgm, kk = k & (m - 1);
  const bool mir = kk > m / 2;
  const float2 z0 = a.gh[s * a.K * (m / 2 + 1) + (mir ? m - kk : kk)];
  const float w0 = a.phi[k];
  float2 acc = make_float2(w0 * z0.x, mir ? -w0 * z0.y : w0 * z0.y);
#pragma unroll 4
  for (int e = a.list[blk]; e < a.list[blk + 1]; ++e) {
    const int f = a.list[e], j = f / a.Q, lg = a.lgM[j];
    const float2 z = a.g[j][((s * a.Q + (f - j * a.Q)) << lg) + (k & ((1 << lg) - 1))];
    const float w = a.filt[(static_cast<size_t>(f) << a.lgN) + k];
    acc.x = fmaf(w, z.x, acc.x);
    acc.y = fmaf(w, z.y, acc.y);
  }
  a.dst[at] = acc;
}

template <int LG>
hipError_t line_shape(bool big, size_t &lds, unsigned &per) {
  lds = big ? Line<LG, 512>::lds_bytes : Line<LG, LG == 13 ? 512 : 256>::lds_bytes;
  per = big ? Line<LG, 512>::SPW : Line<LG, LG == 13 ? 512 : 256>::SPW;
  return hipSuccess;
}

hipError_t shape_of(int lg, bool big, size_t &lds, unsigned &per) {
  switch (lg) {
    case 5: return line_shape<5>(big, lds, per);
    case 6: return line_shape<6>(big, lds, per);
    case 7: return line_shape<7>(big, lds, per);
    case 8: return line_shape<8>(big, lds, per);
    case 9: return line_shape<9>(big, lds, per);
    case 10: return line_shape<10>(big, lds, per);
    case 11: return line_shape<11>(big, lds, per);
    case 12: return line_shape<12>(big, lds, per);
    case 13: return line_shape<13>(big, lds, per);
    default: return hipErrorInvalidValue;
  }
}

template <bool BACK, bool BIG>
hipError_t run_nodes(const NodeArgs &a, unsigned blocks, size_t lds, hipStream_t st) {
  if (lds > 65536) {
    static unsigned long long ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k_line_nodes<BACK, BIG>), ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_line_nodes<BACK, BIG>), dim3(blocks), dim3(line_threads(BIG)), lds, st, a);
  return hipGetLastError();
}

template <int LG, int MODE>
hipError_t run_end_t(const EndArgs &a, hipStream_t st) {
  using L = Line<LG, line_threads(LG == 13)>;
  constexpr size_t lds = L::lds_bytes;
  if (lds > 65536) {
    static unsigned long long ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k_line_end<LG, MODE>), ok);
    if (e != hipSuccess) return e;
  }
  const unsigned blocks = (a.rows + L::SPW - 1) / L::SPW;
  hipLaunchKernelGGL((k_line_end<LG, MODE>), dim3(blocks), dim3(line_threads(LG == 13)), lds, st, a);
  return hipGetLastError();
}

template <int MODE>
hipError_t run_end(int lg, const EndArgs &a, hipStream_t st) {
  static const char *const what[] = {"in", "out", "grad_out", "grad_in"};
  const std::string name = std::string("k_line_end<") + std::to_string(lg) + ", " + what[MODE] + ">";
  const double M = static_cast<double>(1 << lg), rows = a.rows;
  LaunchScope obs(name.c_str(), rows * 4.0 * (a.len + (MODE == kGradIn ? 2.0 * M : M)),
                  rows * M * (MODE == kGradIn ? 5.0 : 2.5) * lg, st);
  switch (lg) {
    case 4: return run_end_t<4, MODE>(a, st);
    case 5: return run_end_t<5, MODE>(a, st);
    case 6: return run_end_t<6, MODE>(a, st);
    case 7: return run_end_t<7, MODE>(a, st);
    case 8: return run_end_t<8, MODE>(a, st);
    case 9: return run_end_t<9, MODE>(a, st);
    case 10: return run_end_t<10, MODE>(a, st);
    case 11: return run_end_t<11, MODE>(a, st);
    case 12: return run_end_t<12, MODE>(a, st);
    case 13: return run_end_t<13, MODE>(a, st);
    default: return hipErrorInvalidValue;
  }
}

EndArgs end_args(const LineEnd &e) {
  EndArgs a{};
  a.rows = static_cast<unsigned>(e.rows);
  a.len = e.len;
  a.low = e.low;
  a.phi = e.phi;
  a.lgm = e.lgm;
  a.K = e.K;
  a.reach = e.reach;
  a.tw = e.tw;
  return a;
}

bool end_ok(const LineEnd &e) { return e.rows > 0 && e.rows < 0x7fffffffL && e.len >= 1 && e.len <= 1 << e.lg; }

}  // namespace

int line_block(int lgM) { return (1 << lgM) / 16; }

hipError_t launch_line_nodes(const LineNodes *list, int n, float2 *low, int lgm, int K, const float2 *tw, bool back,
                             hipStream_t st) {
  if (n < 1 || n > kLineMaxSegs) return hipErrorInvalidValue;
  NodeArgs a{};
  a.low = low;
  a.tw = tw;
  a.n = n;
  a.lgm = lgm;
  a.K = K;
  size_t lds = 0;
  unsigned long long first = 0;
  int kids = 0;
  bool big = false;
  for (int i = 0; i < n; ++i) big = big || list[i].lgM == 13;
  double bytes = 0, flops = 0;
  for (int i = 0; i < n; ++i) {
    const LineNodes &s = list[i];
    size_t need = 0;
    unsigned per = 0;
    if (s.lgM < 5 || s.lgM > 13 || s.lgM < lgm || s.lgA < 0 || s.lgA > 6 || s.nodes < 1 || s.F < 1 || s.G < 1 ||
        s.nodes > 0x7fff0000L || kids + s.kids > kLineMaxSegs || (back && (low == nullptr || s.dst == nullptr)))
      return hipErrorInvalidValue;
    hipError_t e = shape_of(s.lgM, big, need, per);
    if (e != hipSuccess) return e;
    lds = need > lds ? need : lds;
    NodeSeg &g = a.seg[i];
    g.src = s.src;
    g.filt = s.filt;
    g.mask = s.mask;
    g.phi = s.phi;
    g.dst = s.dst;
    g.nodes = static_cast<unsigned>(s.nodes);
    g.first_block = static_cast<unsigned>(first);
    g.blocks = ((g.nodes + per - 1) / per + 7) / 8 * 8;
    first += g.blocks;
    g.F = s.F;
    g.G = s.G;
    g.base = s.base;
    g.stride = s.stride;
    g.phi_mask = s.phi_mask;
    g.kid0 = static_cast<short>(kids);
    g.kids = static_cast<short>(s.kids);
    g.lgM = static_cast<signed char>(s.lgM);
    g.lgA = static_cast<signed char>(s.lgA);
    g.reach = static_cast<signed char>(s.reach);
    for (int c = 0; c < s.kids; ++c) a.kid[kids++] = NodeKid{s.kid[c].g, s.kid[c].filt, s.kid[c].mask, s.kid[c].lgM};
    const double M = static_cast<double>(1 << s.lgM), nd = static_cast<double>(s.nodes);
    bytes += (nd / s.F + s.F) * (M * (1 << s.lgA)) * 4 + nd * M * (back ? 8 : s.dst ? 4 : 0) +
             (low ? nd * 4.0 * (1 << lgm) : 0.0);
    // transforms, filter product, modulus, lowpass; adjoint: children's products
    flops += nd * M * (5.0 * s.lgM * (back ? 3 : 1.5) + 4.0 * (1 << s.lgA) + 4.0 + (low ? 4.0 : 0.0));
    for (int c = 0; c < s.kids; ++c) {
      bytes += nd * 8.0 * (1 << s.kid[c].lgM) + 4.0 * M;
      flops += nd * 4.0 * M;
    }
  }
  if (first > 0x7fffffffull) return hipErrorInvalidValue;
  const unsigned blocks = static_cast<unsigned>(first);
  const std::string name = std::string("k_line_nodes<") + (back ? "true, " : "false, ") + (big ? "true>" : "false>");
  LaunchScope obs(name.c_str(), bytes, flops, st);
  if (back) return big ? run_nodes<true, true>(a, blocks, lds, st) : run_nodes<true, false>(a, blocks, lds, st);
  return big ? run_nodes<false, true>(a, blocks, lds, st) : run_nodes<false, false>(a, blocks, lds, st);
}

hipError_t launch_line_in(const float *x, float2 *spec, const LineEnd &e, hipStream_t st) {
  if (!end_ok(e)) return hipErrorInvalidValue;
  EndArgs a = end_args(e);
  a.xin = x;
  a.sout = spec;
  return run_end<kIn>(e.lg, a, st);
}

hipError_t launch_line_out(const float2 *spec, float *out, const LineEnd &e, hipStream_t st) {
  if (!end_ok(e)) return hipErrorInvalidValue;
  EndArgs a = end_args(e);
  a.sin = spec;
  a.xout = out;
  return run_end<kOut>(e.lg, a, st);
}

hipError_t launch_line_grad_out(const float *g, float2 *spec, const LineEnd &e, hipStream_t st) {
  if (!end_ok(e)) return hipErrorInvalidValue;
  EndArgs a = end_args(e);
  a.xin = g;
  a.sout = spec;
  return run_end<kGradOut>(e.lg, a, st);
}

hipError_t launch_line_grad_in(const float2 *spec, float *out, const LineEnd &e, hipStream_t st) {
  if (!end_ok(e)) return hipErrorInvalidValue;
  EndArgs a = end_args(e);
  a.sin = spec;
  a.xout = out;
  return run_end<kGradIn>(e.lg, a, st);
}

hipError_t launch_line_sum(const LineSum &s, hipStream_t st) {
  if (s.signals < 1 || s.J < 1 || s.J > kLineMaxOctaves || s.lgN > 13 || s.lgm > s.lgN) return hipErrorInvalidValue;
  SumArgs a{};
  a.dst = s.dst;
  a.gh = s.gh;
  a.phi = s.phi;
  a.filt = s.filt;
  a.list = s.list;
  for (int j = 0; j < s.J; ++j) {
    a.g[j] = s.g[j];
    a.lgM[j] = static_cast<signed char>(s.lgM[j]);
  }
  a.total = static_cast<unsigned long long>(s.signals) << s.lgN;
  a.lgN = s.lgN;
  a.lgm = s.lgm;
  a.K = s.K;
  a.Q = s.Q;
  const unsigned long long blocks = (a.total + 255) / 256;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  const double n = static_cast<double>(1 << s.lgN), signals = static_cast<double>(s.signals);
  double bytes = signals * (8.0 * n + 4.0 * (1 << s.lgm)) + 4.0 * n * (1 + s.J * s.Q);
  for (int j = 0; j < s.J; ++j) bytes += signals * 8.0 * s.Q * (1 << s.lgM[j]);
  LaunchScope obs("k_line_sum", bytes, signals * 4.0 * (n + (n < 256 ? n : 256.0) * s.listed), st);
  hipLaunchKernelGGL(k_line_sum, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace scat
