// Whole nodes of the 2-D cascade for grids of any shape: the nodes of at most 8192 points (sides
// 16 ... 128, square or 2 : 1) below an input or a first-order modulus whose spectrum is stored, and
// through k_node_half those of 128 x 128 in octave 0.
//
// One slab of N1 N2 / 16 threads (16 points each) computes a node: filter product with the source's
// half spectrum + periodisation, inverse 2-D transform, modulus, lowpass and subsampling as a
// separable FIR filter with the spatial taps of phi, and, for nodes with children, the forward
// transform of the modulus.  Against the passes that serve these nodes otherwise (k_rows_fused,
// k_col_fast, k_row_lowpass_fast) the node never goes to memory, between the row and the column
// transform as little as after the modulus: 8 + 8 + 4 bytes per point saved.  The nodes that fit
// take it, but for small calls of few angles (rect_pays in scat_capi.hip): 96 planes of 128 x 128, J = 3,
// L = 8, 600 -> 297 us (their 6144 + 6144 second-order nodes of octave 0: 331 -> 128 us); 48 planes of
// 200 x 120 543 -> 343 us.  With spectra as real and imaginary rows (below) 325 us for the latter; with
// octave 0 whole too (k_node_half) 227 us for the former.
// What bounds it: vector issue, with the loads' address path close behind.  6144 nodes of 64 x 64 under 128 x 128 take
// 83 us under the counters: 0.69 of the issue slots at 2.4 GHz, which is about 0.8 at the 2 GHz that the busy cycles show,
// and 0.57 (about 0.7) of the address path's cycles.  Without their loads they take 49, loads alone 47; more waves (5 and
// 7 a SIMD) or more loads in flight (12 ... 48 a lane) changed little.
#include <hip/hip_runtime.h>

#include <cmath>
#include <string>

#include "fft_regs.hpp"
#include "fir.hpp"
#include "scat_kernels.hpp"

namespace scat {

namespace {

// Row slots of the slab in LDS.  The lanes of one half-wavefront hold 32 / T2 rows x T2 adjacent
// columns, and a slot stride of (odd multiple of T2) mod 32 elements puts them on distinct banks;
// the row exchange is unpadded (16 T2 = N2 elements), which keeps a 64 x 64 node at 36 KB and so
// four workgroups on a compute unit.
constexpr int rect_row_stride(int N2) { return N2 + N2 / 16; }
// Columns that a wavefront loads
constexpr int rect_mask_width(int N2) { return N2 < 64 ? N2 : 64; }

struct RectArgs {
  const float *src;                // [NS][Sr/2+1][2][Sc]
  const float *filt;               // [F][Sr][Sc]
  const unsigned long long *mask;  // [F][4][N2 / CW]: see RectNode
  const float *taps_r, *taps_c;    // [2 R + 1]
  float *uout;
  float *out;
  unsigned nodes, blocks;
  int F, G, Sr, lgA;
  int chan_base, chan_src, chan_f, K;
  const float2 *tw;
  int tw_n;
};

template <int N1, int N2>
struct RectShape {
  static constexpr int T1 = N1 / 16, T2 = N2 / 16;
  static constexpr int TS = N1 * N2 / 16;
  static constexpr int NT = TS < 256 ? 256 : TS;
  static constexpr int SPW = NT / TS;
  static constexpr int CW = rect_mask_width(N2);
  static constexpr int RS = rect_row_stride(N2);
  static constexpr size_t lds_bytes = (static_cast<size_t>(SPW) * N1 * RS + N1 + N2) * sizeof(float2);
  static_assert(TS >= 16 && TS <= 512, "node shape");
};

// The slabs of a workgroup take consecutive nodes (filter fastest), and each XCD (workgroups are
// dealt to the eight in turn) a contiguous run of them: the filters of a source meet in one L2.
template <int N1, int N2, int DEC>
__global__ __launch_bounds__((RectShape<N1, N2>::NT), 4) void k_node_rect(RectArgs a) {
  using S = RectShape<N1, N2>;
  constexpr int T1 = S::T1, T2 = S::T2, TS = S::TS, RS = S::RS;
  constexpr bool WAVE = TS <= 64;  // a slab is (part of) one wavefront
  constexpr int MR = N1 / DEC, MC = N2 / DEC, R = kRectReach * DEC;
  extern __shared__ __attribute__((aligned(16))) float2 lds[];
  // (the slab is the same for all lanes of a wave from 64 threads on: its node stays scalar)
  const int slab = TS >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / TS) : threadIdx.x / TS;
  const int q = threadIdx.x % TS;
  const unsigned blk = (blockIdx.x & 7) * (a.blocks >> 3) + (blockIdx.x >> 3);
  if (blk * S::SPW >= a.nodes) return;
  const bool live = blk * S::SPW + slab < a.nodes;
  const unsigned node = live ? blk * S::SPW + slab : a.nodes - 1;  // idle slabs shadow the last node, store nothing
  const unsigned s = node / static_cast<unsigned>(a.F);
  const int f = static_cast<int>(node - s * a.F);
  float2 *area = lds + slab * (N1 * RS);
  float2 *wtab = lds + S::SPW * (N1 * RS);
  for (int i = threadIdx.x; i < N2; i += S::NT) wtab[i] = a.tw[(i / T2) * (i % T2) * (a.tw_n / N2)];
  for (int i = threadIdx.x; i < N1; i += S::NT) wtab[N2 + i] = a.tw[(i / T1) * (i % T1) * (a.tw_n / N1)];
  const int r = q / T2, t = q % T2;  // row layout: row r, columns t + T2 i
  const int c = q % N2;              // column layout: column c, rows t1 + T1 i
  const int t1 = N2 >= 64 ? __builtin_amdgcn_readfirstlane(q / N2) : q / N2;

  // ---- 1. spectrum of the node, lanes on adjacent columns (column c, rows t1 + T1 i).  The filter's
  // support is followed in blocks of a quarter of the node's rows x CW columns: for each, the alias blocks
  // in use.  What bounds this are the cycles that the loads take of the address path: 4 bytes a lane, 64
  // lanes side by side, take a quarter of the cycles of 8 bytes a lane, so real and imaginary parts come by
  // loads of their own, and all but a lane's fixed offset is scalar.
  float2 v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = make_float2(0.f, 0.f);
  {
    const int Sr = a.Sr, Sc = N2 << a.lgA, A = 1 << a.lgA;
    const float *re = a.src + static_cast<size_t>(s) * (Sr + 2) * Sc, *im = re + Sc;
    const float *filt = a.filt + static_cast<size_t>(f) * Sr * Sc;
    // byte offsets within a unit of T1 rows; mirrored: from its last row on
    const unsigned x_d = 4u * (t1 * 2 * Sc + c), x_w = 4u * (t1 * Sc + c);
    const unsigned x_m = 4u * ((T1 - 1 - t1) * 2 * Sc + ((N2 - c) & (N2 - 1)));
    auto at = [](const float *p, unsigned bytes) {
      return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p) + bytes);
    };
    int block = f * 4 * (N2 / S::CW) + c / S::CW;
    if (TS >= 64) block = __builtin_amdgcn_readfirstlane(block);
    struct Unit {
      float xr[4], xi[4], w[4], sign;
      bool own;
    };
    // rows N1 / 4 g + t1 + T1 i of alias block `bit`; own: the blocks that this node's filter uses
    auto load = [&](Unit &un, int g, int bit, unsigned long long own) {
      un.own = TS >= 64 || (own >> bit & 1ull) != 0ull;
      const int ar = bit >> a.lgA, ac = bit & (A - 1), kr = N1 / 4 * g + N1 * ar;
      const bool mir = kr >= Sr / 2;
      // mirrored: row Sr - kr, column -(c + N2 ac); the columns -c but 0 lie one block of N2 before
      const int row = (mir ? Sr - kr - (T1 - 1) : kr) * 2 * Sc;
      const float *pr = re + row, *pi = im + row, *pw = filt + (kr * Sc + N2 * ac);
      const unsigned back = static_cast<unsigned>(c != 0 ? A - 1 - ac : A - ac) & (A - 1);
      const unsigned x = mir ? x_m + 4u * N2 * back : x_d + 4u * N2 * ac;
      const int step = mir ? -2 * T1 * Sc : 2 * T1 * Sc;
      un.sign = mir ? -1.f : 1.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        un.xr[i] = at(pr + i * step, x);
        un.xi[i] = at(pi + i * step, x);
        un.w[i] = at(pw + i * T1 * Sc, x_w);
      }
    };
    // (a node takes its own filter's blocks and no others, whatever nodes it shares a wavefront with: its bits
    // do not depend on its place in the batch, and an infinity in a block that it leaves out does not reach it.
    // 16 planes of 64 x 64, J = 3, L = 8 74.7 -> 75.3 us, of 64 x 32, J = 2, 46.4 -> 47.2)
    auto add = [&](const Unit &un, int g) {
      if (!un.own) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float2 &z = v[4 * g + i];
        z.x = fmaf(un.xr[i], un.w[i], z.x);
        z.y = fmaf(un.xi[i], un.w[i] * un.sign, z.y);
      }
    };
    if (A == 1) {  // one block each: all of them at once
      Unit un[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) load(un[g], g, 0, 1ull);
#pragma unroll
      for (int g = 0; g < 4; ++g) add(un[g], g);
    } else {
      unsigned long long owns[4];  // (all before the first use of any: 16 planes of 64 x 64 75.9 -> 75.3 us)
#pragma unroll
      for (int g = 0; g < 4; ++g) owns[g] = a.mask[block + g * (N2 / S::CW)];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const unsigned long long own = owns[g];
        unsigned long long rem = own;
        if (TS < 64) {  // slabs that share a wavefront: what any of them uses
          rem |= __shfl_xor(rem, 32);
          if (TS < 32) rem |= __shfl_xor(rem, 16);
          rem = (static_cast<unsigned long long>(__builtin_amdgcn_readfirstlane(static_cast<int>(rem >> 32))) << 32) |
                static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(rem)));
        }
        auto next = [&] {
          const int bit = __ffsll(static_cast<long long>(rem)) - 1;
          rem &= rem - 1ull;
          return bit;
        };
        int n = __popcll(rem);
        for (; n >= 4; n -= 4) {
          Unit un[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) load(un[e], g, next(), own);
#pragma unroll
          for (int e = 0; e < 4; ++e) add(un[e], g);
        }
        if (n & 2) {
          Unit un[2];
          load(un[0], g, next(), own);
          load(un[1], g, next(), own);
          add(un[0], g);
          add(un[1], g);
        }
        if (n & 1) {
          Unit un;
          load(un, g, next(), own);
          add(un, g);
        }
      }
    }
  }
  __syncthreads();  // the twiddles

  // ---- 2. inverse transform: columns, transpose, rows
  fft_core_tab<16, T1, true, WAVE>(v, t1, area + c, T1 * RS, RS, wtab + N2 + t1, T1);
#pragma unroll
  for (int i = 0; i < 16; ++i) area[(t1 + T1 * i) * RS + c] = v[i];
  group_sync<WAVE>();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = area[r * RS + t + T2 * i];
  group_sync<WAVE>();
  fft_core_tab<16, T2, true, WAVE>(v, t, area + r * RS, T2, 1, wtab + t, T2);

  // ---- 3. modulus
  float u[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) u[i] = __builtin_amdgcn_sqrtf(v[i].x * v[i].x + v[i].y * v[i].y);

  // ---- 4. lowpass + subsampling by DEC: along the rows, then along the columns
  constexpr int US = N2 + 1, HS = MC + 4;
  static_assert(N1 * (US + HS) <= 2 * N1 * RS, "LDS of the lowpass");
  float *ub = reinterpret_cast<float *>(area);  // [N1][US]
  float *hb = ub + N1 * US;                     // [N1][HS]
#pragma unroll
  for (int i = 0; i < 16; ++i) ub[r * US + t + T2 * i] = u[i];
  group_sync<WAVE>();
  {
    constexpr int OPT = 16 / DEC;  // outputs per thread, adjacent columns
    const int rr = q % N1, mg = q / N1;
    float acc[OPT];
    fir<DEC, OPT, N2, 1>(acc, ub + rr * US, DEC * OPT * mg - R, a.taps_c);
#pragma unroll
    for (int j = 0; j < OPT; ++j) hb[rr * HS + OPT * mg + j] = acc[j];
  }
  group_sync<WAVE>();
  {
    constexpr int OPV = DEC >= 4 ? 1 : 16 / (DEC * DEC);  // outputs per thread, adjacent rows
    const int mc = q % MC, ng = q / MC;
    if (DEC <= 4 || ng < MR) {
      float acc[OPV];
      fir<DEC, OPV, N1, HS>(acc, hb + mc, DEC * OPV * ng - R, a.taps_r);
      if (live) {
        const unsigned plane = s / static_cast<unsigned>(a.G);
        const int g = static_cast<int>(s - plane * a.G);
        float *op = a.out + (static_cast<size_t>(plane) * a.K + a.chan_base + g * a.chan_src + f * a.chan_f) * (MR * MC);
#pragma unroll
        for (int j = 0; j < OPV; ++j) op[(OPV * ng + j) * MC + mc] = acc[j];
      }
    }
  }
  if (a.uout == nullptr) return;

  // ---- 5. spectrum of the modulus for the children (rows 0 .. N1/2)
  group_sync<WAVE>();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = make_float2(u[i], 0.f);
  fft_core_tab<16, T2, false, WAVE>(v, t, area + r * RS, T2, 1, wtab + t, T2);
#pragma unroll
  for (int i = 0; i < 16; ++i) area[r * RS + t + T2 * i] = v[i];
  group_sync<WAVE>();
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = area[(t1 + T1 * i) * RS + c];
  group_sync<WAVE>();
  fft_core_tab<16, T1, false, WAVE>(v, t1, area + c, T1 * RS, RS, wtab + N2 + t1, T1);
  if (live) {
    float *up = a.uout + static_cast<size_t>(node) * (N1 + 2) * N2 + c;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (t1 + T1 * i <= N1 / 2) {
        up[(t1 + T1 * i) * 2 * N2] = v[i].x;
        up[(t1 + T1 * i) * 2 * N2 + N2] = v[i].y;
      }
  }
}

double log2d(double n) { return n > 1 ? std::log2(n) : 0.0; }

template <int N1, int N2, int DEC>
hipError_t launch_rect_t(RectArgs &a, hipStream_t st) {
  using S = RectShape<N1, N2>;
  if (a.tw_n % N1 != 0 || a.tw_n % N2 != 0) return hipErrorInvalidValue;
  a.blocks = ((a.nodes + S::SPW - 1) / S::SPW + 7) / 8 * 8;
  const std::string name =
      "k_node_rect<" + std::to_string(N1) + ", " + std::to_string(N2) + ", " + std::to_string(DEC) + ">";
  const double nodes = static_cast<double>(a.nodes), pts = static_cast<double>(N1) * N2;
  const double spts = static_cast<double>(a.Sr) * (N2 << a.lgA);
  const double fft = 5.0 * pts * log2d(pts);
  LaunchScope obs(name.c_str(),
                  nodes / a.F * spts * 4 + a.F * spts * 4 + nodes * pts / (DEC * DEC) * 4 +
                      (a.uout ? nodes * pts * 4 : 0),
                  nodes * (4.0 * spts + fft * (a.uout ? 1.5 : 1.0) + 4.0 * pts +
                           2.0 * (2 * kRectReach * DEC + 1) * pts * (1.0 / DEC + 1.0 / (DEC * DEC))),
                  st);
  if (S::lds_bytes > 65536) {
    static unsigned long long lds_ok = 0;
    hipError_t e = allow_large_lds(reinterpret_cast<const void *>(k_node_rect<N1, N2, DEC>), lds_ok);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_node_rect<N1, N2, DEC>), dim3(static_cast<unsigned>(a.blocks)), dim3(S::NT), S::lds_bytes, st,
                     a);
  return hipGetLastError();
}

bool pow2i(int n) { return n > 0 && (n & (n - 1)) == 0; }

}  // namespace

int rect_reach(int dec) { return kRectReach * dec; }
int rect_mask_columns(int N2) { return rect_mask_width(N2); }

// (8 dec <= N2: plans on the fused row pass keep 16 points a row at their last octave, where dec is 2)
bool node_rect_supported(int N1, int N2, int A, int dec) {
  // 128 x 128 in octave 0 only: from larger sources k_node_half wants their filters in a layout of its own,
  // and the passes take 128 + 42 us there for the 1536 + 192 nodes of 24 planes of 256 x 256, which it would
  // not do in less.  Passes -> k_node_half, us: J = 3 on every batch and number of angles tried (1 ... 400 planes,
  // 1 ... 12): 1 plane, L = 8 107 -> 93, 400 planes 983 -> 807, first order only 357 -> 237; J = 4 for all but few nodes of
  // one or two angles (rect_pays): 1 plane, L = 8 155 -> 134, 256 planes 712 -> 574, first order only, L = 5, 172 -> 132.
  if (N1 == 128 && N2 == 128) return A == 1 && (dec == 8 || dec == 16);
  return pow2i(N1) && pow2i(N2) && N1 >= 16 && N2 >= 16 && N1 * N2 <= 8192 &&
         (N1 == N2 || N1 == 2 * N2 || N2 == 2 * N1) && (dec == 2 || dec == 4 || dec == 8) && 8 * dec <= N2 && pow2i(A) &&
         A <= 8;
}

hipError_t launch_node_rect(const RectNode &n, hipStream_t st) {
  if (n.NS <= 0) return hipSuccess;
  if (!node_rect_supported(n.N1, n.N2, n.A, n.dec) || n.F < 1 || n.G < 1 || n.mask == nullptr ||
      n.NS > 0x7fff0000L / n.F)
    return hipErrorInvalidValue;
  if (n.N1 * n.N2 > 8192) {  // 128 x 128: half a slab's threads, see k_node_half
    NodeLaunch h{};
    h.M = 128;
    h.A = 1;
    h.P = 1;
    h.dec = n.dec;
    h.src = reinterpret_cast<const float2 *>(n.src);
    h.filt = n.filt;
    h.taps_r = n.taps_r;
    h.taps_c = n.taps_c;
    h.uout = reinterpret_cast<float2 *>(n.uout);
    h.out = n.out;
    h.NS = n.NS;
    h.F = n.F;
    h.G = n.G;
    h.chan_base = n.chan_base;
    h.chan_src = n.chan_src;
    h.chan_f = n.chan_f;
    h.K = n.K;
    h.tw = n.tw;
    h.tw_n = n.tw_n;
    return launch_node(h, st);
  }
  RectArgs a;
  a.src = n.src;
  a.filt = n.filt;
  a.mask = n.mask;
  a.taps_r = n.taps_r;
  a.taps_c = n.taps_c;
  a.uout = n.uout;
  a.out = n.out;
  a.nodes = static_cast<unsigned>(n.NS * n.F);
  a.F = n.F;
  a.G = n.G;
  a.Sr = n.N1 * n.A;
  a.lgA = n.A == 1 ? 0 : n.A == 2 ? 1 : n.A == 4 ? 2 : 3;
  a.chan_base = n.chan_base;
  a.chan_src = n.chan_src;
  a.chan_f = n.chan_f;
  a.K = n.K;
  a.tw = n.tw;
  a.tw_n = n.tw_n;
#define SCAT_RECT(N1_, N2_, DEC_) \
  case (N1_ << 16) | (N2_ << 4) | DEC_: return launch_rect_t<N1_, N2_, DEC_>(a, st);
#define SCAT_RECT4(N1_, N2_) SCAT_RECT(N1_, N2_, 2) SCAT_RECT(N1_, N2_, 4)
#define SCAT_RECT8(N1_, N2_) SCAT_RECT4(N1_, N2_) SCAT_RECT(N1_, N2_, 8)
  switch ((n.N1 << 16) | (n.N2 << 4) | n.dec) {
    SCAT_RECT(16, 16, 2)
    SCAT_RECT4(16, 32)
    SCAT_RECT(32, 16, 2)
    SCAT_RECT4(32, 32)
    SCAT_RECT8(32, 64)
    SCAT_RECT4(64, 32)
    SCAT_RECT8(64, 64)
    SCAT_RECT8(64, 128)
    SCAT_RECT8(128, 64)
    default: return hipErrorInvalidValue;
  }
#undef SCAT_RECT8
#undef SCAT_RECT4
#undef SCAT_RECT
}

}  // namespace scat
