// Launch wrappers of the generic scattering kernels (see scat_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace scat {

// Optional per-thread hook called around every kernel launch of this file: `before` gets
// the kernel's name as a profiler prints it, the bytes the launch must move at the least
// (inputs and filter tables read once, outputs written once) and its model flops
// (5 n log2 n per transform plus the pointwise work).
struct LaunchObserver {
  virtual void before(const char *name, double bytes, double flops, hipStream_t st) = 0;
  virtual void after(hipStream_t st) = 0;
  virtual ~LaunchObserver() = default;
};
void set_launch_observer(LaunchObserver *o);

// Reports one launch to the installed observer: construct right before the launch,
// destroy right after it.
struct LaunchScope {
  LaunchScope(const char *name, double bytes, double flops, hipStream_t st);
  ~LaunchScope();
  LaunchScope(const LaunchScope &) = delete;
  LaunchScope &operator=(const LaunchScope &) = delete;

 private:
  hipStream_t st_;
  bool on_;
};

// Lets kernel `fn` use up to 160 KB of dynamic LDS on the current device.  The attribute is
// per device; `done` (one static per kernel at the call site) remembers the devices served.
inline hipError_t allow_large_lds(const void *fn, unsigned long long &done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (done & bit) return hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) done |= bit;
  return e;
}

// Where a kernel's node number g (within one input plane p) lands in the output:
// channel = base + (g / inner) * outer_stride + (g % inner), node = p * G + g.
struct ChanMap {
  int G, inner, outer_stride, base;
};

// mask (optional, device): per filter a 64-bit word, bit a_r * 2^fc + a_c set = the alias block
// (a_r, a_c) of (Sr >> fr) x (Sc >> fc) points holds values that matter; blocks whose bit is
// clear for every filter processed together are skipped (needs 2^(fr + fc) <= 64).
hipError_t launch_mulfold_invrow(const float2 *src, const float *filt, float2 *dst, long S, int F,
                                 int Sr, int Sc, int fr, int fc, int post_tw_m, const float2 *tw,
                                 int tw_n, hipStream_t st, const unsigned long long *mask = nullptr);

hipError_t launch_col(int mode, const void *src, long nodes, int Mr, int Mc, float2 *uc,
                      int post_tw_m, const float *phi_rows, int m_r, float *w_out, float *out,
                      ChanMap cm, int K, const float2 *tw, int tw_n, hipStream_t st,
                      bool uc_half = false);

// launch_col mode 1 with the four-step twiddle (post_tw_m = Mr * Mc) over up to kColMaxSegs
// arrays of nodes in one launch: segment i holds `nodes` signals of Mr x Mc elements at
// src + src_off and writes their column spectra to uc + uc_off (Mr = 256, Mc a multiple of 16).
constexpr int kColMaxSegs = 8;
struct ColSeg {
  long nodes;
  int Mc;
  long long src_off, uc_off;
};
// uc_half: the columns are real after the modulus, so only rows 0 .. Mr/2 of every node's
// spectrum are written ([nodes][Mr/2+1][Mc] at uc + uc_off; launch_rows1d with half_rows reads them)
hipError_t launch_col_segs(const float2 *src, float2 *uc, int Mr, const ColSeg *segs, int n, bool uc_half,
                           const float2 *tw, int tw_n, hipStream_t st);

// launch_col mode 2 for 256-row nodes of Mc <= 16 columns, over `nodes` nodes mapped by cm and,
// stored right behind them, `tail_nodes` nodes that are channel 0 of signals 0, 1, ...
bool col_out_tail_supported(int Mr, int Mc, int tw_n);
hipError_t launch_col_out_tail(const float2 *src, long nodes, long tail_nodes, int Mc, float *out, ChanMap cm, int K,
                               const float2 *tw, int tw_n, hipStream_t st);

// 1-D cascade: forward row FFT of src [nodes][Sr][Sc] (column spectra, left untouched) and,
// for each child, filter product + fold of the row by 2^lg_fold + inverse row FFT + four-step
// twiddle, stored to the child's dst [nodes][Sr][Sc >> lg_fold] (see k_rows1d).
constexpr int kRows1dMaxChildren = 32;
struct Rows1dChild {
  const float *filt;  // [Sr][Sc], carries the inverse-transform normalisation
  float2 *dst;
  int lg_fold;
  int post_tw_m;  // 0 = no twiddle, else Sr * (Sc >> lg_fold): the child's signal length
  // K > 0: node p * cm.G + g is stored as signal number p * K + channel(cm, g) instead of at
  // its own number (the lowpass children of a whole transform gathered channel-major)
  ChanMap cm;
  int K;
  // null, or cm.G device words: the channel of node g comes from this table instead of cm's
  // formula (nodes of several parent octaves in one launch)
  const int *chan_tab;
};
struct Rows1dArgs {
  int n;
  Rows1dChild c[kRows1dMaxChildren];
  // null, or where the forward row spectra themselves are stored ([nodes][Sr][Sc]; may be the
  // source: in place).  Register kernel with all rows stored only.
  float2 *spec_out = nullptr;
};
// half_rows: src holds rows 0 .. Sr/2 of every node only ([nodes][Sr/2+1][Sc], written by the
// column pass with uc_half for real columns); the other rows are derived from them
// (rows1d_half_supported: the row lengths for which that form exists)
bool rows1d_half_supported(int Sr, int Sc);
hipError_t launch_rows1d(const float2 *src, long nodes, int Sr, int Sc, const Rows1dArgs &a,
                         const float2 *tw, int tw_n, hipStream_t st, bool half_rows = false);

// Adjoint of launch_rows1d: dst [nodes][Sr][Sc] (= or +=) the inverse row FFT of
// sum_c filt_c * tile(forward row FFT of child c), child rows of Sc >> lg_fold points (see
// k_rows1d_adj).  Node g of dst reads node number
//   K == 0:  g * cm.G + cm.base                       (one of the cm.G nodes under each parent)
//   K  > 0:  (g / cm.G) * K + channel(cm, g % cm.G)   (channel-major arrays, as Rows1dChild)
// of c.src.
struct Rows1dAdjChild {
  const float2 *src;
  const float *filt;  // [Sr][Sc], the table of the forward pass
  int lg_fold;
  ChanMap cm;
  int K;
};
struct Rows1dAdjArgs {
  int n;
  int accumulate;  // 0: dst is overwritten; 1: added to
  Rows1dAdjChild c[kRows1dMaxChildren];
};
bool rows1d_adj_supported(int Sc);
hipError_t launch_rows1d_adj(float2 *dst, long nodes, int Sr, int Sc, const Rows1dAdjArgs &a,
                             const float2 *tw, int tw_n, hipStream_t st);

// 2-D: dst [nodes][Sr][Sc] (= or +=) sum_c filt_c * tile(src_c), child planes of
// (Sr >> lg_fr) x (Sc >> lg_fc) gradient spectra, then (inverse != 0) the inverse row
// transform (see k_rows2d_adj).  filt_row != nullptr: the filter is filt_row[kr] * filt[kc].
// Child nodes as in Rows1dAdjChild.  Row lengths 4 ... 512, with the inverse transform up to 256.
struct Rows2dAdjChild {
  const float2 *src;
  const float *filt;
  const float *filt_row;
  int lg_fr, lg_fc;
  ChanMap cm;
  int K;
  int pre_rows;  // 1: src is given before its forward row transform (lg_fc == 0, rows <= 256)
};
struct Rows2dAdjArgs {
  int n;
  int accumulate;
  int inverse;
  int lg_rows, any_pre_rows;  // set by the launcher
  Rows2dAdjChild c[kRows1dMaxChildren];
};
bool rows2d_adj_supported(int Sc, bool inverse);
hipError_t launch_rows2d_adj(float2 *dst, long nodes, int Sr, int Sc, const Rows2dAdjArgs &a,
                             const float2 *tw, int tw_n, hipStream_t st);

// planar: every row is left as its Mc real parts followed by its Mc imaginary parts (what k_node_rect
// reads; rows of 16 ... 256 points)
hipError_t launch_row_fwd(float2 *data, long rows, int Mc, const float2 *tw, int tw_n,
                          hipStream_t st, bool planar = false);

hipError_t launch_row_lowpass(const float *w, long nodes, int m_r, int Mc, int m_c,
                              const float *phi_cols, float *out, ChanMap cm, int K,
                              const float2 *tw, int tw_n, hipStream_t st);

// Column pass of whole square nodes (Mr x Mr) with both halves of the lowpass (length m on
// both axes) fused: like launch_col mode 0/1 followed by launch_row_lowpass, but S goes
// straight to `out` and the intermediate W never to memory.
bool col_node_supported(int Mr, int Mc, int m_r, int m_c, int tw_n);
hipError_t launch_col_node(int mode, const void *src, long nodes, int Mr, int m, float2 *uc,
                           bool uc_half, const float *phi_rows, const float *phi_cols, float *out,
                           ChanMap cm, int K, const float2 *tw, int tw_n, hipStream_t st);

// Leaf nodes (no children; 64 x 64 with a 32 x 32 output) from the row pass's output to the
// output coefficients in one kernel (see k_leaf_node).
bool leaf_node_supported(int Mr, int Mc, int m_r, int m_c, int tw_n);
hipError_t launch_leaf_node(const float2 *src, long nodes, int Mr, int m, const float *phi_rows,
                            const float *phi_cols, float *out, ChanMap cm, int K, const float2 *tw,
                            int tw_n, hipStream_t st);

// One level of the fused row pass: wavelets `filt` ([F][Sr][Sc] real, pre-scaled) applied
// with fold 2^f on both axes, outputs to dst [NS*F][Sr>>f][Sc>>f].
struct FusedLevel {
  int f, F;
  const float *filt;
  float2 *dst;
};

// True if launch_rows_fused can handle sources of Sr x Sc with largest fold 2^fmax.
bool rows_fused_supported(int Sr, int Sc, int fmax);

// Forward row FFT of column-transformed sources [NS][Sr][Sc] (or half, see below), then every level's filter
// multiply + fold + inverse row FFT (see k_rows_fused).
// src_half: the sources hold rows 0..Sr/2 only ([NS][Sr/2+1][Sc], column spectra of real
// signals as written by launch_col with uc_half); the other rows are their conjugates.
hipError_t launch_rows_fused(const float2 *src, bool src_half, long NS, int Sr, int Sc,
                             const FusedLevel *levels, int nlev, const float2 *tw, int tw_n,
                             hipStream_t st);

// Whole scattering tree of 32 x 32 planes at J = 2: one wavefront per first-order node keeps the
// node, the spectrum of its modulus and its second-order children in LDS and writes only S1 and S2;
// the planes' spectra and S0 by a launch before it, or, for few planes, in the same one (scat_tree.hip).
//   x         [planes][n_r][n_c] real, extended symmetrically to 32 x 32 (sides of 13 ... 32)
//   xh        [planes][32][32] space for the spectra of the extended planes
//   psi_j0/1  [L][32][32] first-order wavelets of octaves 0 and 1, pre-scaled by 1/1024
//   phi_cols* lowpass along a row (the column frequency axis) at resolutions 0 (32 samples)
//             and 1 (16 samples), Fourier domain, pre-scaled by 1/length
//   taps*     lowpass along a column at the same resolutions as spatial taps: the inverse
//             DFT (unnormalised) of the pre-scaled Fourier samples, 32 and 16 values
//   out       [planes][K][o_r][o_c], o_r, o_c <= 8
struct Tree32 {
  const float *x;
  float2 *xh;
  long planes;
  int n_r, n_c, o_r, o_c;
  int L, max_order, K;
  const float *psi_j0, *psi_j1, *phi_cols0, *phi_cols1, *taps0, *taps1;
  float *out;
  bool few;  // one launch
};
// Is one launch the faster way for a call of so many planes?  (of the whole call: its chunks go one way)
bool tree32_few(long planes, int L, int max_order);
bool tree_supported(int n_r, int n_c, int J);
hipError_t launch_tree32(const Tree32 &t, hipStream_t st);
// gx [planes][n_r][n_c]: the gradient for the output gradient gout [planes][K][o_r][o_c] (t.out and t.xh
// are not used).  parts: tree32_back_elems(L) elements per plane.
size_t tree32_back_elems(int L);
hipError_t launch_tree32_back(const Tree32 &t, const float *gout, float2 *parts, float *gx, hipStream_t st);

// Whole nodes of the 2-D tree in one kernel each (scat_node.hip): spectrum of the node from
// its parent's stored half spectra (P sources of S x S, S = M * A, with A x A aliases folded),
// inverse transform, modulus, lowpass to the 32 x 32 output grid by a separable FIR filter
// (taps: 2 R + 1 values, R = 4 M / 32; polyphase nodes: two sets, for p = 0 and p = 1), and
// optionally the half spectrum of the modulus for the node's children.
//   src    [NS][P][S/2+1][S]; filt [F][P][S][S]; items per source: F (poly: 4 F, the four
//          polyphase components of each filter's node, component index 2 p_r + p_c fastest)
//   mask   filters that vanish on whole M x M alias blocks of their table: the blocks to skip
//   uout   null or [NS * items][M/2+1][M] (poly: times w^(p.k), w = exp(-2 pi i / 2M))
//   out    [planes][K][32][32] with channel = chan_base + (source % G) * chan_src +
//          filter * chan_f and plane = source / G; poly: parts [NS * items][32][32]
struct NodeLaunch {
  int M, A, P;
  bool poly;
  bool full;  // src holds all S rows of one spectrum per node ([NS][S][S]) instead of rows 0 .. S/2
  int dec;    // 0: outputs of 32 x 32; else (M = 128, A = P = 1) subsampling 8 or 16, taps and spectra as in
              // RectNode
  const float2 *src;
  const float *filt;
  const unsigned long long *mask;  // null, or [F] device words: bit (q A + a_r) A + a_c set = block in use
  // null, or [F][words per workgroup] device words for the loaders whose source is twice the
  // node's size: per thread, which of its loads meet table values that are not negligible
  // (node_lane_mask builds them from the table itself)
  const unsigned *lane_mask;
  const float *taps_r, *taps_c;
  float2 *uout;
  float *out;
  long NS;
  int F, G;
  int chan_base, chan_src, chan_f, K;
  const float2 *tw;
  int tw_n;
};
bool node_supported(int M, int A, int P, bool poly, bool full = false);
hipError_t launch_node(const NodeLaunch &n, hipStream_t st);
// out[plane][chan_base + g][32][32] = sum of the four parts of node plane * G + g
hipError_t launch_sum4(const float *part, float *out, long nodes, int G, int K, int chan_base,
                       hipStream_t st);

// Whole nodes of N1 x N2 points for grids of any shape (scat_rect.hip): the spectrum from the
// source's half spectrum (S = A N1 x A N2 points, rows 0 .. A N1 / 2 stored), inverse transform,
// modulus, lowpass by a FIR filter of 2 rect_reach(dec) + 1 taps and subsampling by dec per axis.
//   src    [NS][A N1/2+1][2][A N2]: real, then imaginary parts of each row; filt [F][A N1][A N2], pre-scaled
//   mask   [F][4][N2 / w] device words, w = rect_mask_columns: bit a_r A + a_c of word (g, b) clear = in
//          that N1 x N2 alias block the filter is negligible on the g-th quarter of the rows of the b-th
//          w columns
//   uout   null or [NS * F][N1/2+1][2][N2] half spectra of the moduli
//   out    [planes][K][N1/dec][N2/dec], channels as in NodeLaunch
struct RectNode {
  int N1, N2, A, dec;
  const float *src;
  const float *filt;
  const unsigned long long *mask;
  const float *taps_r, *taps_c;
  float *uout;
  float *out;
  long NS;
  int F, G;
  int chan_base, chan_src, chan_f, K;
  const float2 *tw;
  int tw_n;
};
bool node_rect_supported(int N1, int N2, int A, int dec);
int rect_reach(int dec);
int rect_mask_columns(int N2);
hipError_t launch_node_rect(const RectNode &n, hipStream_t st);

// Modulus backward step of whole nodes in one pass (k_node_modback): data [nodes][Mr][Mc]
// gradient spectra in, gradient spectra of the taped y [nodes][Mr][Mc] out, in place.  The
// _low form starts from the node's adjoint lowpass instead (arguments as
// launch_lowpass_adj_rows; ghat is scratch for nodes * m_r * m_c elements); with y_rows, y is
// the node before its inverse column transform (the forward row pass's output) and the
// kernel transforms the columns itself.
bool node_modback_supported(int Mr, int Mc);
// ghat [node][m_r][m_c] = 2-D transform of the nodes' output gradient planes
bool small_fft2_supported(int m_r, int m_c);
hipError_t launch_small_fft2(const float *gout, long nodes, ChanMap cm, int K, int m_r, int m_c,
                             float2 *ghat, const float2 *tw, int tw_n, hipStream_t st);
hipError_t launch_node_modback(float2 *data, const float2 *y, long nodes, int Mr, int Mc,
                               const float2 *tw, int tw_n, hipStream_t st, bool y_rows = false);
// ... the same for leaves (y before its inverse column transform) with the lowpass as spatial taps instead of
// Fourier samples: taps_r, taps_c hold dec = Mr / m_r zeros and then phi at -leaf_reach(dec) ... leaf_reach(dec)
int leaf_reach(int dec);
bool leaf_modback_supported(int Mr, int Mc, int m_r, int m_c);
hipError_t launch_leaf_modback(const float *gout, long nodes, ChanMap cm, int K, int m_r, int m_c, int Mr, int Mc,
                               const float *taps_r, const float *taps_c, const float2 *y, float2 *dst,
                               const float2 *tw, int tw_n, hipStream_t st);
hipError_t launch_node_modback_low(const float *gout, long nodes, ChanMap cm, int K, int m_r, int m_c,
                                   int Mr, int Mc, const float *phi_rows, const float *phi_cols,
                                   float2 *ghat, const float2 *y, float2 *dst, const float2 *tw,
                                   int tw_n, hipStream_t st, bool y_rows = false);

// ---- backward pass (scat_backward.hip): plain 2-D transforms in place and the adjoints of
// the lowpass, the modulus and the filter-multiply-fold step.  Sides 4...512.
bool backward_side_supported(int m);
// rows only: data [rows][Mc]
hipError_t launch_fft_rows_inplace(float2 *data, long rows, int Mc, bool inverse, const float2 *tw,
                                   int tw_n, hipStream_t st);
// columns of data [nodes][Mr][Mc]: inverse transform, a = Re(a) y / |y| (0 where y = 0)
// against y of the same layout, forward transform
// tw_m > 0: with the four-step twiddles exp(+-2 pi i k1 b / tw_m) around the column passes
hipError_t launch_cols_modback(float2 *data, const float2 *y, long nodes, int Mr, int Mc,
                               const float2 *tw, int tw_n, hipStream_t st, int tw_m = 0,
                               bool y_rows = false);
// columns only (any power-of-two number of columns up to 512)
hipError_t launch_fft_cols_inplace(float2 *data, long nodes, int Mr, int Mc, bool inverse,
                                   const float2 *tw, int tw_n, hipStream_t st);
// 1-D signals as n1 x Mc matrices: data[node][k1][b] *= exp(-+2 pi i k1 b / (n1 Mc))
hipError_t launch_twiddle(float2 *data, long nodes, int n1, int Mc, bool conj, const float2 *tw,
                          int tw_n, hipStream_t st);
// dst[node][i] = (g_out[plane][chan(cm, g)][i], 0) for i < m
hipError_t launch_gather_real(const float *gout, long nodes, ChanMap cm, int K, int m, float2 *dst,
                              hipStream_t st);
// dst[node][k1][k2] = ghat[node][k1][k2 mod mc] * filt[k1][k2]
hipError_t launch_tile_filter(const float2 *ghat, const float *filt, float2 *dst, long nodes, int n1,
                              int Mc, int mc, hipStream_t st);
// the same followed by the inverse row transform, in one pass over dst; `ghat` is scratch
// of nodes * m_r * m_c elements
hipError_t launch_lowpass_adj_rows(const float *gout, long nodes, ChanMap cm, int K, int m_r,
                                   int m_c, int Mr, int Mc, const float *phi_rows,
                                   const float *phi_cols, float2 *ghat, float2 *dst,
                                   const float2 *tw, int tw_n, hipStream_t st);
hipError_t launch_take_real(const float2 *a, float *out, long count, hipStream_t st);
// dst [S][Sr][Sc] += sum_f filt[f] * G[s F + f][k_r mod Mr][k_c mod Mc]
hipError_t launch_tile_accum(float2 *dst, const float *filt, const float2 *G, long S, int F, int Sr,
                             int Sc, int Mr, int Mc, hipStream_t st);

// ---- 3-D solid harmonic scattering (scat_3d.hip): a 3-D transform in place over
// [volumes][n0][n1][n2] (sides 4...256) and the pointwise steps of the cascade
// fused 3-D passes (slabs of axes 1 and 2 held by one workgroup); see scat_3d.hip
bool fused3_supported(int n0, int n1, int n2, int J);
// A node of a fused 3-D launch (every launch takes a list of them, one per blockIdx.y):
//   src  F^ of its source [volumes][n0][n1][n2]; tab its M pair tables [M][n0][n1][n2]
//   W    its M signals [M][volumes][n0][n1][n2]
//   T    axis-0 spectra [volumes][n0/2+1][n1][n2] (backward, half == 0: [volumes][n0][n1][n2])
//   U    null, or where its own spectrum goes; chan its output channel
struct Node3 {
  const float2 *src, *tab;
  float2 *W, *T, *U;
  int M, chan, half;
};
constexpr int kMaxNodes3 = 24;
struct Nodes3 {
  int n;
  Node3 v[kMaxNodes3];
};
// T = inverse slab transform of (channel chan's lowpass adjoint + the spectra A[first ... first+count))
struct Sum3 {
  float2 *T;
  int first, count, chan;
};
constexpr int kMaxSpectra3 = 32;
struct Sums3 {
  int n;
  Sum3 v[kMaxNodes3];
  const float2 *A[kMaxSpectra3];
};
hipError_t launch3_slab_mul_inv(const Nodes3 &nodes, long volumes, int n0, int n1, int n2, const float2 *tw,
                                int tw_n, hipStream_t st);
// phi == nullptr: spectra only, no lowpass; P [volumes][K][n0][n1>>J][n2>>J]
hipError_t launch3_slab_fwd_low(const Nodes3 &nodes, const float *phi, float2 *P, long volumes, int n0, int n1,
                                int n2, int J, int K, const float2 *tw, int tw_n, hipStream_t st);
// xreal (one node, its T is written): real input, of user[0] x user[1] x user[2] samples extended
// symmetrically where user is not null; else the nodes' signals W
hipError_t launch3_axis0_rho(const Nodes3 &nodes, const float *xreal, const int *user, long volumes, int n0,
                             int n2, int Mc, const float2 *tw, int tw_n, hipStream_t st);
// W <- forward axis-0 transform of (gradient of rho in T) y / rho, in place
hipError_t launch3_axis0_back(const Nodes3 &nodes, long volumes, int n0, int Mc, const float2 *tw, int tw_n,
                              hipStream_t st);
hipError_t launch3_axis0_real(const float2 *src, float *out, long volumes, int n0, int Mc, const float2 *tw,
                              int tw_n, hipStream_t st);
// W_0 <- sum_p conj(c_p) forward slab transform of W_p
hipError_t launch3_slab_fwd_mulacc(const Nodes3 &nodes, long volumes, int n0, int n1, int n2, const float2 *tw,
                                   int tw_n, hipStream_t st);
hipError_t launch3_slab_sum_inv(const Sums3 &sums, const float *phi, const float2 *Gs, long volumes, int n0,
                                int n1, int n2, int J, int K, const float2 *tw, int tw_n, hipStream_t st);
hipError_t launch3_sum_spectra(const Sums3 &sums, float2 *dst, long total, hipStream_t st);
// output grids one workgroup holds: P -> the first o[0] x o[1] x o[2] output samples, and its adjoint
bool out3_supported(int m0, int m1, int m2);
hipError_t launch3_out(const float2 *P, float *out, long maps, int n0, int m0, int m1, int m2, const int *o,
                       hipStream_t st);
hipError_t launch3_out_adj(const float *gout, float2 *Gs, long maps, int m0, int m1, int m2, const int *o,
                           hipStream_t st);
hipError_t launch3_fold0(const float2 *P, float2 *Q, long groups, int n0, int m0, int slab,
                         hipStream_t st);
hipError_t launch3_real_part(const float2 *src, float *out, long total, hipStream_t st);
hipError_t launch3_fft(float2 *data, long volumes, int n0, int n1, int n2, bool inverse,
                       const float2 *tw, int tw_n, hipStream_t st);
hipError_t launch3_real_to_complex(const float *x, float2 *out, long total, hipStream_t st);
// dst[v][e] = src[v][e] * filt[e], e < n
hipError_t launch3_mul_table(const float2 *src, const float *filt, float2 *dst, long volumes, long n,
                             hipStream_t st, bool accumulate = false);
// backward pass of the 3-D transform: lowpass adjoint, gradient through rho
hipError_t launch3_tile_phi(const float2 *Gs, const float *phi, float2 *dst, long volumes, int K,
                            int chan, int n0, int n1, int n2, int J, bool accumulate, hipStream_t st);
hipError_t launch3_rho_back(const float2 *gu, const float *acc, float2 *y, long total,
                            hipStream_t st);
// acc[i] = |y[i]|^2 (first) or acc[i] + |y[i]|^2
hipError_t launch3_accum_abs2(const float2 *y, float *acc, long total, bool first, hipStream_t st);
// out[i] = (sqrt(acc[i]), 0)
hipError_t launch3_sqrt(const float *acc, float2 *out, long total, hipStream_t st);
// out[v][chan][a][b][c] = Re src[v][a 2^J][b 2^J][c 2^J], out has K channels per volume
hipError_t launch3_sample(const float2 *src, float *out, long volumes, int K, int chan, int n0,
                          int n1, int n2, int J, hipStream_t st);

// ---- backward pass of 2-D plans whose every node is one workgroup (scat_plane.hip)
constexpr int kPlaneMaxOctaves = 8;
struct PlaneKidNodes {
  const float2 *g;                 // [nodes][L][Mr][Mc] gradient spectra of the children
  const float *filt;               // their L wavelets on the parent's grid
  const unsigned long long *mask;  // as PlaneNodes::mask
  int Mr, Mc;
};
// NS * F nodes of N1 x N2 points: wavelet node % F on source node / F of A N1 x A N2 points
struct PlaneNodes {
  const float2 *src;  // [NS][A N1 / 2 + 1][A N2]
  long NS;
  int N1, N2, A;
  const float *filt;
  int F;
  // per wavelet three words: the alias blocks (bit a_r A + a_c) in use by the upper and by the lower
  // half of the node's rows; the sixteenths of the source's rows in use
  const unsigned long long *mask;
  float2 *dst;  // half spectra of the moduli; adjoint: gradient spectra
  // adjoint: spectra of the output gradients [planes][K][m_r][m_c], phi's factors; node of source s
  // and wavelet f: channel chan_base + (s % G) chan_src + f of plane s / G
  const float2 *gh;
  const float *phi_r, *phi_c;
  int m_r, m_c, G, chan_base, chan_src, K, L;
  PlaneKidNodes kid[kPlaneMaxOctaves];
  int kids;
  const float2 *tw;
  int tw_n;
};
bool plane_supported(int N1, int N2);
hipError_t launch_plane_nodes(const PlaneNodes &n, bool back, hipStream_t st);
hipError_t launch_plane_in(const float *x, float2 *spec, long planes, int N1, int N2, const float2 *tw, int tw_n,
                           hipStream_t st);
hipError_t launch_plane_real(const float2 *spec, float *out, long planes, int N1, int N2, const float2 *tw, int tw_n,
                             hipStream_t st);
struct PlaneSum {
  float2 *dst;
  const float2 *gh;
  const float *phi_r, *phi_c, *filt;
  const int *list;  // as LineSum::list, blocks of 256 points of the plane
  const float2 *g[kPlaneMaxOctaves];
  int res[kPlaneMaxOctaves];
  long planes, listed;
  int N1, N2, m_r, m_c, K, J, L;
};
hipError_t launch_plane_sum(const PlaneSum &s, hipStream_t st);

// ---- 1-D plans of at most 8192 samples, whole nodes (scat_line.hip).  Spectra in natural order;
// half spectra are [M/2+1].
constexpr int kLineMaxSegs = 28;    // pairs of octaves
constexpr int kLineMaxOctaves = 8;
struct LineKid {
  const float2 *g;    // [nodes][1 << lgM] gradient spectra of the children, numbered as their parents
  const float *filt;  // their wavelet on the parent's grid
  unsigned mask;      // blocks of line_block(parent's lgM) values on which it is not negligible
  int lgM;
};
// `nodes` nodes of 1 << lgM samples: wavelet node % F on source node / F, whose half spectra have
// 1 << (lgM + lgA) samples; output channel base + (node % G) stride of signal node / G
struct LineNodes {
  const float2 *src;
  const float *filt;
  const unsigned long long *mask;  // per wavelet two words: alias blocks in use by either half of the node
  const float *phi;
  float2 *dst;  // forward: half spectra for the children (or null); adjoint: gradient spectra
  long nodes;
  int F, G, base, stride, lgM, lgA, reach;
  unsigned phi_mask;   // as LineKid::mask
  const LineKid *kid;  // adjoint
  int kids;
};
int line_block(int lgM);  // samples between two that a thread holds
// low [signals][K][(1 << lgm)/2+1]: the outputs' half spectra, written (null: not formed), or with
// `back` those of the output gradients, read
hipError_t launch_line_nodes(const LineNodes *list, int n, float2 *low, int lgm, int K, const float2 *tw, bool back,
                             hipStream_t st);
// transforms of `rows` lines of 1 << lg samples, of which `len` are the caller's
struct LineEnd {
  long rows;
  int lg, len;
  float2 *low;  // launch_line_in: also the half spectrum of channel 0, or null
  const float *phi;
  int lgm, K, reach;
  const float2 *tw;
};
hipError_t launch_line_in(const float *x, float2 *spec, const LineEnd &e, hipStream_t st);
hipError_t launch_line_out(const float2 *spec, float *out, const LineEnd &e, hipStream_t st);
hipError_t launch_line_grad_out(const float *g, float2 *spec, const LineEnd &e, hipStream_t st);
hipError_t launch_line_grad_in(const float2 *spec, float *out, const LineEnd &e, hipStream_t st);
struct LineSum {
  float2 *dst;
  const float2 *gh;
  const float *phi, *filt;
  // per block of 256 frequencies the first-order wavelets in use: the blocks' starts in `list`
  // (one more than there are blocks), then the wavelets
  const int *list;
  const float2 *g[kLineMaxOctaves];
  int lgM[kLineMaxOctaves];
  long signals, listed;  // wavelets in the list, over all blocks
  int lgN, lgm, K, J, Q;
};
hipError_t launch_line_sum(const LineSum &s, hipStream_t st);

}  // namespace scat
