// Tall-skinny Householder QR with explicit Q (QR-based projector section,
// step 1: the isometries are re-orthonormalised by a QR decomposition after
// the power update).
//
// Communication-avoiding layout for N x k blocks with N >> k:
//  * the rows are split into `nb` leaves of at most kLeafRows rows (leaf 0
//    holds at least k rows); the columns are processed in panels of width
//    kPanel;
//  * per panel, every leaf factors its active rows of the panel with
//    Householder reflectors held in registers, forms the compact-WY factor T
//    (H_0...H_(w-1) = I - V T V^T) and updates its trailing columns with
//    C <- C - V T^T (V^T C), three small GEMMs on the FP64 matrix cores;
//  * the w x w triangles the leaves leave in their top rows are combined
//    eight at a time up a reduction tree (depth log8 of the leaf count);
//    combining stacked upper triangles gives reflectors [e_j; v] with v
//    upper triangular in each absorbed triangle, stored in its place, and
//    their own WY factor updates the trailing columns of the node's rows;
//  * a factorisation reads only the panel and a trailing update of the level
//    below writes only the trailing columns, so the two share one launch;
//  * the caller's block is read by panel 0 only; the factors live in a working
//    copy, and Q = prod_p L_p T_p [S; 0], S = diag(sign R_cc) (so that R has
//    a non-negative diagonal), is formed in the caller's block by applying
//    the tree and leaf WY factors (C <- C - V T (V^T C)) in reverse order on
//    the columns that can be non-trivial; rows of [S; 0] that no factor has
//    touched yet are taken as known, not read.
// Reflectors follow the LAPACK dlarfg convention: beta = -sign(alpha) * norm,
// tau = (beta - alpha) / beta, and tau = 0 (H = I) when the part below the
// diagonal is exactly zero, so rank-deficient blocks never divide by zero.

#include "common.h"

#include <type_traits>

namespace sictm {
namespace {

constexpr int kPanel = 32;
constexpr int kLeafRows = 192;       // of the four-wavefront leaves
constexpr int kWideLeafRows = 384;   // of the eight-wavefront ones
constexpr int kT = kPanel + 1;   // padded row length of the small LDS matrices

struct QrPlan {
  int N, k, nb, P, depth;
  bool wide;   // leaves of eight wavefronts
};

struct QrArgs {
  double* W[kMaxProb];   // the caller's blocks: read by panel 0, then Q
  double* A[kMaxProb];   // working copies holding V and R
  double* Tl;            // [count][P][nb][kPanel*kPanel] leaf WY factors
  double* Tn;            // [count][P][nb][kPanel*kPanel] tree WY factors (by right child)
  int count, N, k, nb, P;
  int rows, extra;       // leaves hold `rows` rows, the first `extra` one more
};

// First row of leaf i (no division: the kernels start with this).
__device__ __forceinline__ int leaf_start(const QrArgs& q, int i) {
  return i * q.rows + min(i, q.extra);
}

__device__ __forceinline__ long slot(int mat, int p, int leaf, int nb, int P) {
  return ((long)mat * P + p) * nb + leaf;
}

// ---------------------------------------------------------------------------
// Householder factorisation of one panel by the four wavefronts of a
// workgroup.  The panel sits in registers, a column per lane: lane c of a
// 16-lane row holds the panel columns c and c + 16 of the rows g + 16 r,
// r < R, where g = 0..15 numbers the 16-lane rows of the workgroup.  A step
// needs column j in every lane of its row, which is one DPP broadcast per
// register (row_newbcast), then 2 R multiply-adds give the row's share of
// x_j^T x_s for the lane's two columns s: the squared norm of the column
// (s = j) and the products of all others come from the same sums, so a step
// has one exchange between the wavefronts (through LDS, double-buffered by
// the parity of j) and one barrier.  With S_s the sum below the pivot and
// a_s the pivot row, the reflector (dlarfg: beta = -sign(a_j) |(a_j, x_j)|,
// v = x_j / (a_j - beta)) gives v^T x_s = a_s + S_s / (a_j - beta), and for
// the earlier columns the Gram column of the WY factor T.  Reflectors stay
// unscaled in their registers (each lane keeps the scale of its columns);
// the pivot row goes to Rs as it becomes a row of R and is zeroed from
// column j on, so that no later sum needs a mask.  Every wavefront forms the
// same reflector from the same sums in the same order, and writes the same
// values to the same places where only one would have to: a step without
// branches is faster than one with less to store.
//
// Bound by latency: 32 dependent steps.  Measured on 8 blocks of
// 5184 x 160, one row per lane with a 63-add transpose-reduction of the 32
// products per step, a second reduction for the norm and a second barrier
// took 51.7 us per launch of leaves (44.0 us of tree nodes); this form takes
// 28.3 us, of which the 32 steps are 17 us (1290 cycles each).
// ---------------------------------------------------------------------------

// 1/x and 1/sqrt(x) to full double precision from the hardware estimates (two
// Newton steps), for arguments away from the ends of the exponent range.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double fast_rsq(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, fma(-0.5 * x * y, y, 0.5), y);
  return fma(y, fma(-0.5 * x * y, y, 0.5), y);
}

// Lane L of each 16-lane row, in every lane of the row.
template <int L>
__device__ __forceinline__ double row_bcast(double x) {
  return __longlong_as_double(
      __builtin_amdgcn_update_dpp(0LL, __double_as_longlong(x), 0x150 + L, 0xf, 0xf, true));
}

constexpr int kGL = kPanel + 2;   // row length of Gt: 16-byte aligned rows

struct PanelLds {
  double part[2][8][kPanel];     // [buffer][wavefront][chunk a | chunk b]: x_j^T x_s below the pivot
  double alpha[2][32][kPanel];   // [buffer][16-lane row][chunk a | chunk b]: register row 0
  double Rs[kPanel][kT];         // R
  double Gt[kPanel][kGL];        // Gt[j][s] = v_s^T v_j for s < j, Gt[j][j] = tau_j
  double T[kPanel][kT];
};

// The pass over the columns works on a pair of column chunks: `a` holds the
// 16 pivots of this half of the panel, `b` the other 16 columns; register 0
// of each holds the pivot rows (of four wavefronts it has 16 rows, and the
// halves trade places between the passes; of eight it has all 32).
template <int R>
struct PanelRegs {
  double a[R], b[R];       // unscaled panel entries
  double sa, sb;           // scales of the lane's reflectors
};

// Column j = j0 + JL; j0 = 0 or 16, chunk a starts at column j0, chunk b at
// 16 - j0.
template <int JL, int R, int NW>
__device__ __forceinline__ void panel_step(PanelRegs<R>& x, int j0, int w, int lane, int wave,
                                           PanelLds& sh) {
  const int j = j0 + JL;
  if (j < w) {
    constexpr int buf = JL & 1;
    const int c = lane & 15, row = (lane >> 4) + 4 * wave;
    const int prow = NW == 8 ? j : JL;
    const bool piv = row == prow;   // this 16-lane row holds the pivot row
    const bool upper = lane >= 32;
    sh.alpha[buf][row][c] = x.a[0];
    sh.alpha[buf][row][16 + c] = x.b[0];
    double v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = row_bcast<JL>(x.a[r]);
    v[0] = piv ? 0.0 : v[0];
    double p0 = 0.0, p1 = 0.0, q0 = 0.0, q1 = 0.0;
#pragma unroll
    for (int r = 0; r < R; r += 2) {
      p0 = fma(v[r], x.a[r], p0);
      q0 = fma(v[r], x.b[r], q0);
      p1 = fma(v[r + 1], x.a[r + 1], p1);
      q1 = fma(v[r + 1], x.b[r + 1], q1);
    }
    double p = p0 + p1, q = q0 + q1;
    swap_halves32(p, q);   // lanes < 32 sum chunk a, the others chunk b
    p += q;
    q = p;
    swap_halves16(p, q);
    p += q;
    sh.part[buf][wave][(upper ? 16 : 0) + c] = p;
    __syncthreads();
    const double aa = sh.alpha[buf][prow][c], ab = sh.alpha[buf][prow][16 + c];
    auto sum4 = [&](int o, int w0) {
      return (sh.part[buf][w0][o] + sh.part[buf][w0 + 1][o]) +
             (sh.part[buf][w0 + 2][o] + sh.part[buf][w0 + 3][o]);
    };
    double Sa = sum4(c, 0), Sb = sum4(16 + c, 0);
    if (NW == 8) {
      Sa += sum4(c, 4);
      Sb += sum4(16 + c, 4);
    }
    const double ss = row_bcast<JL>(Sa), al = row_bcast<JL>(aa);
    // tau = (beta - alpha) / beta; H = I (tau = 0) when the part below the
    // pivot is exactly zero
    const double q2 = fma(al, al, ss);
    const double y = fast_rsq(q2);
    double nrm = q2 * y;
    nrm = fma(0.5 * y, fma(-nrm, nrm, q2), nrm);
    double tau = fma(fabs(al), y, 1.0), inv = fast_rcp(fabs(al) + nrm);
    // the estimates hold away from the ends of the exponent range (the
    // condition is the same in every lane)
    if (__builtin_expect(!__all(q2 > 1e-280 && q2 < 1e280), 0)) {
      nrm = sqrt(q2);
      tau = 1.0 + fabs(al) / nrm;
      inv = 1.0 / (fabs(al) + nrm);
    }
    const bool live = !(ss == 0.0);
    const double beta = live ? -copysign(nrm, al) : al;
    const double scal = live ? copysign(inv, al) : 0.0;
    tau = live ? tau : 0.0;
    const double da = fma(scal, Sa, aa), db = fma(scal, Sb, ab);
    const double fa = c > JL ? tau * da : 0.0, fb = j0 == 0 ? tau * db : 0.0;
    const double ga = -fa * scal, gb = -fb * scal;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      x.a[r] = fma(ga, v[r], x.a[r]);
      x.b[r] = fma(gb, v[r], x.b[r]);
    }
    x.a[0] = piv && c >= JL ? 0.0 : x.a[0];
    x.b[0] = piv && j0 == 0 ? 0.0 : x.b[0];
    // row j of Gt (columns below j count) and of R (columns from j on count)
    const int col = (upper ? 16 - j0 : j0) + c;
    const double gram = upper ? x.sb * db : (c == JL ? tau : x.sa * da);
    const double rrow = upper ? ab - fb : (c == JL ? beta : aa - fa);
    sh.Gt[j][col] = gram;
    sh.Rs[j][col] = rrow;
    x.sa = c == JL ? scal : x.sa;
  }
}

template <int R, int NW>
__device__ __forceinline__ void swap_chunks(PanelRegs<R>& x) {
  auto sw = [](double& p, double& q) {
    const double t = p;
    p = q;
    q = t;
  };
  if (NW == 4) {
    sw(x.a[0], x.a[1]);
    sw(x.b[0], x.b[1]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) sw(x.a[r], x.b[r]);
  sw(x.sa, x.sb);
}

// T (upper) of H_0...H_(w-1) = I - V T V^T from Gt.  The 8 x 8 diagonal
// blocks are built columnwise, T_jj = tau_j, T[i, j] = -tau_j sum_{l=i}^{j-1}
// T[i, l] G[l, j], one block per wavefront, a row per lane; two blocks side
// by side then merge with T_12 = -T_11 (G_12 T_22) (wavefronts beyond the
// fourth only take part in the barriers), to 16 x 16 and to
// 32 x 32.  (One wavefront building all 32 columns, a chain of 496
// multiply-adds fed from LDS, took 11000 cycles of a panel's 63000.)
__device__ __forceinline__ void build_T(PanelLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double (*Y)[kT] = sh.Rs;   // R has been stored
  if (wave < 4) {
    const int b = 8 * wave;
    double t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      double acc[2] = {0.0, 0.0};
#pragma unroll
      for (int l = 0; l < j; ++l) acc[l & 1] = fma(t[l], sh.Gt[b + j][b + l], acc[l & 1]);
      const double tj = sh.Gt[b + j][b + j];
      t[j] = lane < j ? -tj * (acc[0] + acc[1]) : (lane == j ? tj : 0.0);   // t[l] = 0 for l < lane
    }
    if (lane < 8) {
#pragma unroll
      for (int j = 0; j < kPanel; ++j) sh.T[b + lane][j] = 0.0;
#pragma unroll
      for (int j = 0; j < 8; ++j) sh.T[b + lane][b + j] = t[j];
    }
  }
  __syncthreads();
  // merges at width h: thread (i, c) forms one element
  auto merge = [&](int h, int i, int c, int o, bool on) {
    double y = 0.0;
    if (on) {
      for (int l = 0; l < h; ++l) y = fma(sh.Gt[o + h + l][o + i], sh.T[o + h + l][o + h + c], y);
      Y[o + i][c] = y;
    }
    __syncthreads();
    if (on) {
      double z = 0.0;
      for (int l = 0; l < h; ++l) z = fma(sh.T[o + i][o + l], Y[o + l][c], z);
      sh.T[o + i][o + h + c] = -z;
    }
    __syncthreads();
  };
  merge(8, lane >> 3, lane & 7, 16 * wave, wave < 2);
  merge(16, tid >> 4, tid & 15, 0, tid < 256);
}

// Loads the panel through ld(g, r, column), factors it, returns V and R
// through st(g, r, column, V entry, R entry) (row g + 4 NW r; the R entry is
// meaningful for the first 32 rows) and forms T.
template <int R, int NW, typename LD, typename ST>
__device__ __forceinline__ void panel_qr(int w, int lane, int wave, PanelLds& sh, LD ld, ST st) {
  static_assert(R >= 2 && R % 2 == 0, "register rows");
  PanelRegs<R> x;
  const int g = (lane >> 4) + 4 * wave, c = lane & 15;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    x.a[r] = ld(g, r, c);
    x.b[r] = ld(g, r, c + 16);
  }
  x.sa = x.sb = 0.0;
  // rows of Gt and Rs at or beyond w are never written
  for (int i = threadIdx.x; i < kPanel * kPanel; i += 64 * NW) {
    sh.Gt[i >> 5][i & 31] = 0.0;
    sh.Rs[i >> 5][i & 31] = 0.0;
  }
  __syncthreads();
  // two passes over one copy of the code (the instruction cache holds it)
#pragma unroll 1
  for (int j0 = 0; j0 < kPanel; j0 += 16) {
    panel_step<0, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<1, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<2, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<3, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<4, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<5, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<6, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<7, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<8, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<9, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<10, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<11, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<12, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<13, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<14, R, NW>(x, j0, w, lane, wave, sh);
    panel_step<15, R, NW>(x, j0, w, lane, wave, sh);
    swap_chunks<R, NW>(x);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool top = r < 8 / NW;
    st(g, r, c, x.sa * x.a[r], top ? sh.Rs[g + 4 * NW * r][c] : 0.0);
    st(g, r, c + 16, x.sb * x.b[r], top ? sh.Rs[g + 4 * NW * r][c + 16] : 0.0);
  }
  build_T(sh);
}

// ---------------------------------------------------------------------------
// leaf factorisation of panel p (the trailing columns: leaf_wy)
// ---------------------------------------------------------------------------
template <int R, int NW>
__device__ __forceinline__ void leaf_factor(const QrArgs& q, int p, int leaf, int mat,
                                            PanelLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k = q.k, nb = q.nb;
  const int c0 = p * kPanel, w = min(kPanel, k - c0);
  const int s = leaf_start(q, leaf), e = leaf_start(q, leaf + 1);
  const int a0 = (leaf == 0) ? c0 : s;
  const int m = e - a0;
  const double* src = (p == 0 ? q.W[mat] : q.A[mat]) + (long)a0 * k + c0;
  double* dst = q.A[mat] + (long)a0 * k + c0;
  // rows at or beyond m and columns at or beyond w are held as zeros
  constexpr int G = 4 * NW;
  panel_qr<R, NW>(
      w, lane, wave, sh,
      [&](int g, int r, int c) {
        return g + G * r < m && c < w ? (src + (long)(G * r) * k)[g * k + c] : 0.0;
      },
      [&](int g, int r, int c, double v, double rv) {
        const int row = g + G * r;
        if (row < m && c < w) (dst + (long)(G * r) * k)[g * k + c] = c >= row ? rv : v;
      });
  const long sl = slot(mat, p, leaf, nb, q.P);
  for (int idx = tid; idx < kPanel * kPanel; idx += 64 * NW)
    q.Tl[sl * kPanel * kPanel + idx] = sh.T[idx / kPanel][idx % kPanel];
}

// Top row of the w x w triangle a leaf holds during panel p.
__device__ __forceinline__ int top_row(const QrArgs& q, int leaf, int c0) {
  return leaf == 0 ? c0 : leaf_start(q, leaf);
}

// ---------------------------------------------------------------------------
// Reduction tree: a node at stride s combines the triangles of the leaves
// a, a + s, ..., a + (kArity - 1) s (those below nb), a = node * s * kArity;
// the first child keeps R, the others receive the reflector parts.  The
// node's WY factor is stored in the slot of child 1, s (kArity i + 1), which
// no other node at any stride shares (its odd part times a power of kArity).
// ---------------------------------------------------------------------------
constexpr int kArity = 8;
constexpr int kTrailN = 32;   // columns per workgroup in the block-reflector kernels
static_assert(kTrailN == kPanel, "the leaf and tree block-reflector chunks share one launch width");

__device__ __forceinline__ int node_children(int a, int s, int nb) {
  return min(kArity, (nb - a + s - 1) / s);
}

// The workgroup factors the stacked triangles [R_0; R_1; ...]; the
// reflectors are [e_j; v_j] with v_j in the upper triangles of the children
// after the first (the node's trailing columns: tree_wy).  Register row r
// holds rows g + 16 (r mod 2) of child r / 2 (of eight wavefronts, rows g of
// child r).  The rows of child 0 below the pivot are zero in the pivot column,
// so the panel code needs no mask for them.
template <int R, int NW>
__device__ __forceinline__ void tree_factor(const QrArgs& q, int p, int s, int a, int nch, int mat,
                                            PanelLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k = q.k, nb = q.nb;
  const int c0 = p * kPanel, w = min(kPanel, k - c0);
  double* A = q.A[mat];
  constexpr int H = 8 / NW;   // register rows of a child
  auto base = [&](int r) {   // register row r of the stack (the same in every lane)
    return A + (long)(top_row(q, a + r / H * s, c0) + 16 * (r % H)) * k + c0;
  };
  auto in = [&](int g, int r, int c) { return r / H < nch && g + 16 * (r % H) <= c && c < w; };
  panel_qr<R, NW>(
      w, lane, wave, sh,
      [&](int g, int r, int c) { return in(g, r, c) ? base(r)[g * k + c] : 0.0; },
      [&](int g, int r, int c, double v, double rv) {
        if (in(g, r, c)) base(r)[g * k + c] = r < H ? rv : v;
      });
  const long sl = slot(mat, p, a + s, nb, q.P);
  for (int idx = tid; idx < kPanel * kPanel; idx += 64 * NW)
    q.Tn[sl * kPanel * kPanel + idx] = sh.T[idx / kPanel][idx % kPanel];
}

template <int NW = 4>
__device__ __forceinline__ void tree_factor_node(const QrArgs& q, int p, int s, int node, int mat,
                                                 PanelLds& sh) {
  const int a = node * s * kArity;
  if (a + s >= q.nb) return;
  const int nch = node_children(a, s, q.nb);
  if (nch <= 2)
    tree_factor<16 / NW, NW>(q, p, s, a, nch, mat, sh);
  else if (nch <= 4)
    tree_factor<32 / NW, NW>(q, p, s, a, nch, mat, sh);
  else
    tree_factor<8 * kArity / NW, NW>(q, p, s, a, nch, mat, sh);
}

// ---------------------------------------------------------------------------
// Block reflectors applied to 32-column chunks, one chunk per workgroup, so
// that the chunks of a leaf or node run side by side.
// FORM = false: the trailing update of the factorisation, A <- H^T A on the
// columns [c0 + w, k) (H = I - V T V^T, so H^T uses T^T; panel 0 takes the
// columns from the caller's block); FORM = true: the Q formation, E <- H E
// on the columns [c0, k) of the caller's block, E = [S; 0] at first.  Of E
// in panel p, chunk 0 (its own columns) holds what this panel's earlier
// factors have written and [S; 0] elsewhere, and the later chunks what the
// later panels have written, which is everything but the rows
// c0 .. c0 + w - 1 (zero until the first factor of this panel reaches them).
// ---------------------------------------------------------------------------
struct WyLds {
  double Wp[4][kPanel][kT];
  double T[kPanel][kT], W2[kPanel][kT];
};

// S_cc from the diagonal of R.
__device__ __forceinline__ double diag_sign(const double* A, int k, int c) {
  return A[(long)c * k + c] < 0.0 ? -1.0 : 1.0;
}

// One chunk: C <- C - V op(T) (V^T C) for NW RW rows, of which this wavefront
// owns rows RW wave .. RW (wave + 1) - 1.  vval / cval(row, column) give the
// operands (zeros outside), put(row, column, value) stores the result.  The
// operands are read from global memory straight into the operand layout of
// v_mfma_f64_16x16x4 (lane l: row l/16 of a 4-row k-step, column l%16 of a
// 16-column block); the wavefronts' partial products V_w^T C_w meet in LDS,
// every wavefront forms one 16 x 16 block of W2 = op(T) W1 from their sum,
// and each then updates its own rows.  The second reading of V and C (in the
// layouts of the update) and T are requested before the barriers that
// separate the products, so one memory latency covers them; the update's
// products accumulate onto C itself.  `ksteps` k-steps of this wavefront have
// a C that is not known to be zero.  TREE: the rows are 32-row triangles
// stacked, whose rows 16 .. 31 are zero in columns 0 .. 15 (those products
// are left out).  50 KB of LDS lets three workgroups of four wavefronts share a
// CU (of eight, the second four add their partial products to the first's).
//
// Bound by latency (a chain of two memory round trips, 3 x 8 to 3 x 64
// dependent f64 MFMAs and three barriers): on 8 blocks of 5184 x 160 a launch
// forming Q took 20.2 us (nodes) and 38.6 us (leaves) with the second reading
// issued where it was used and the zeros multiplied, 15.7 and 25.7 us in this
// form.
template <bool FORM, bool TREE, int RW, int NW, typename VF, typename CF, typename PF>
__device__ __forceinline__ void wy_apply(const double* Tg, int rows, int ksteps, VF vval, CF cval,
                                         PF put, WyLds& sh) {
  constexpr int KS = RW / 4, RB = RW / 16;
  static_assert(kPanel == 32 && kTrailN == kPanel && RW % 16 == 0, "fragment shapes");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = RW * wave, li = lane & 15, lk = lane >> 4;
  constexpr int NT = 64 * NW;
  double tg[kPanel * kPanel / NT];
#pragma unroll
  for (int i = 0; i < kPanel * kPanel / NT; ++i) tg[i] = Tg[tid + NT * i];
  {
    double vf[KS][2], cf[KS][2];
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      const int rr = r0 + 4 * t + lk;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        vf[t][i] = t < ksteps && !(TREE && i == 0 && (t & 4)) ? vval(rr, 16 * i + li) : 0.0;
        cf[t][i] = t < ksteps ? cval(rr, 16 * i + li) : 0.0;
      }
    }
#pragma unroll
    for (int i = 0; i < kPanel * kPanel / NT; ++i)
      sh.T[(tid >> 5) + NT / 32 * i][tid & 31] = tg[i];
    v4d acc[2][2] = {{{0, 0, 0, 0}, {0, 0, 0, 0}}, {{0, 0, 0, 0}, {0, 0, 0, 0}}};
#pragma unroll
    for (int t = 0; t < KS; ++t)
      if (t < ksteps) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            if (!(TREE && i == 0 && (t & 4)))
              acc[i][j] =
                  __builtin_amdgcn_mfma_f64_16x16x4f64(vf[t][i], cf[t][j], acc[i][j], 0, 0, 0);
      }
    auto partial = [&](bool add) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double& d = sh.Wp[wave & 3][16 * i + lk + 4 * r][16 * j + li];
            d = add ? d + acc[i][j][r] : acc[i][j][r];
          }
    };
    if (wave < 4) partial(false);
    if (NW == 8) {
      __syncthreads();
      if (wave >= 4) partial(true);
    }
  }
  // the update's operands
  double v2[RB][kPanel / 4];
  v4d u[RB][2];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int rr0 = r0 + 16 * rb;
#pragma unroll
    for (int t = 0; t < kPanel / 4; ++t)
      v2[rb][t] = !(TREE && (rb & 1) && t < 4) ? vval(rr0 + li, 4 * t + lk) : 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) u[rb][j][r] = cval(rr0 + lk + 4 * r, 16 * j + li);
  }
  __syncthreads();
  if (wave < 4) {
    // W2 block (bi, bj) = op(T) W1 with W1 the sum of the partials in wave order
    const int bi = wave >> 1, bj = wave & 1;
    v4d a2 = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < kPanel / 4; ++t) {
      const int l = 4 * t + lk, i = 16 * bi + li, c = 16 * bj + li;
      const double tv = FORM ? sh.T[i][l] : sh.T[l][i];
      const double w1 = (sh.Wp[0][l][c] + sh.Wp[1][l][c]) + (sh.Wp[2][l][c] + sh.Wp[3][l][c]);
      a2 = __builtin_amdgcn_mfma_f64_16x16x4f64(tv, w1, a2, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.W2[16 * bi + lk + 4 * r][16 * bj + li] = a2[r];
  }
  __syncthreads();
  double w2[kPanel / 4][2];
#pragma unroll
  for (int t = 0; t < kPanel / 4; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) w2[t][j] = sh.W2[4 * t + lk][16 * j + li];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int rr0 = r0 + 16 * rb;
    if (rr0 < rows) {
#pragma unroll
      for (int t = 0; t < kPanel / 4; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          if (!(TREE && (rb & 1) && t < 4))
            u[rb][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-v2[rb][t], w2[t][j], u[rb][j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) put(rr0 + lk + 4 * r, 16 * j + li, u[rb][j][r]);
    }
  }
}

// Node rows, with V_0 = I: row 32 h + r of the stack is row r of child h, and
// wavefront w owns children 2w and 2w + 1; rows r >= w of a child are zero.
template <bool FORM>
__device__ __forceinline__ void tree_wy(const QrArgs& q, int p, int s, int node, int mat, int chunk,
                                        bool top, WyLds& sh) {
  constexpr int RW = kArity * kPanel / 4;
  static_assert(RW == 2 * kPanel, "two children per wavefront");
  const int a = node * s * kArity;
  const int k = q.k, nb = q.nb;
  if (a + s >= nb) return;
  const int nch = node_children(a, s, nb);
  const int c0 = p * kPanel, w = min(kPanel, k - c0);
  const int cb = (FORM ? c0 : c0 + w) + chunk * kTrailN;
  if (cb >= k) return;
  const int nc = min(kTrailN, k - cb);
  const double* A = q.A[mat];
  double* M = FORM ? q.W[mat] : q.A[mat];
  const int wave = threadIdx.x >> 6;
  // the wavefront's two children
  const long t0 = (long)top_row(q, a + 2 * wave * s, c0) * k;
  const long t1 = (long)top_row(q, a + (2 * wave + 1) * s, c0) * k;
  auto vval = [&](int u, int c) -> double {
    const int h = u >> 5, r = u & 31;
    if (h >= nch || r >= w || c >= w) return 0.0;
    if (h == 0) return r == c ? 1.0 : 0.0;
    return r <= c ? A[(h & 1 ? t1 : t0) + r * k + c0 + c] : 0.0;
  };
  auto cval = [&](int u, int c) -> double {
    const int h = u >> 5, r = u & 31;
    if (h >= nch || r >= w || c >= nc) return 0.0;
    if (FORM) {
      // child 0 was a child of the level above, except at the top (leaf 0);
      // the other children's rows are first reached here
      if (h == 0 && top) return chunk == 0 && r == c ? diag_sign(A, k, c0 + c) : 0.0;
      if (h > 0 && chunk == 0) return 0.0;
    }
    return M[(h & 1 ? t1 : t0) + r * k + cb + c];
  };
  auto put = [&](int u, int c, double v) {
    const int h = u >> 5, r = u & 31;
    if (h < nch && r < w && c < nc) M[(h & 1 ? t1 : t0) + r * k + cb + c] = v;
  };
  const int ksteps = FORM && chunk == 0 ? (wave == 0 ? kPanel / 4 : 0)
                                        : kPanel / 4 * max(0, min(2, nch - 2 * wave));
  wy_apply<FORM, true, RW, 4>(q.Tn + slot(mat, p, a + s, nb, q.P) * kPanel * kPanel, kPanel * nch,
                           ksteps, vval, cval, put, sh);
}

// Leaf rows: V is unit lower-trapezoidal (implicit ones, zeros above).
template <bool FORM, int NW>
__device__ __forceinline__ void leaf_wy(const QrArgs& q, int p, int leaf, int mat, int chunk,
                                        WyLds& sh) {
  constexpr int RW = kLeafRows / 4;
  const int k = q.k, nb = q.nb;
  const int c0 = p * kPanel, w = min(kPanel, k - c0);
  const int cb = (FORM ? c0 : c0 + w) + chunk * kPanel;
  if (cb >= k) return;
  const int nc = min(kPanel, k - cb);
  const int s = leaf_start(q, leaf), e = leaf_start(q, leaf + 1);
  const int a0 = (leaf == 0) ? c0 : s;
  const int m = e - a0;
  const double* A = q.A[mat];
  const double* V = A + (long)a0 * k + c0;
  const double* Cin = (FORM || p == 0 ? q.W[mat] : q.A[mat]) + (long)a0 * k + cb;
  double* C = (FORM ? q.W[mat] : q.A[mat]) + (long)a0 * k + cb;
  auto vval = [&](int r, int c) -> double {
    if (r >= m || c >= w) return 0.0;
    return r > c ? V[r * k + c] : (r == c ? 1.0 : 0.0);
  };
  auto cval = [&](int r, int c) -> double {
    if (r >= m || c >= nc) return 0.0;
    if (FORM) {
      // the tree has written the top rows; without one they are those of
      // [S; 0].  The rows below are first reached here in chunk 0
      if (nb == 1 && r < w) return chunk == 0 && r == c ? diag_sign(A, k, c0 + c) : 0.0;
      if (chunk == 0 && r >= w) return 0.0;
    }
    return Cin[r * k + c];
  };
  auto put = [&](int r, int c, double v) {
    if (r < m && c < nc) C[r * k + c] = v;
  };
  const int r0 = RW * (threadIdx.x >> 6);
  const int live = FORM && chunk == 0 ? w : m;   // rows of C that may be non-zero
  wy_apply<FORM, false, RW, NW>(q.Tl + slot(mat, p, leaf, nb, q.P) * kPanel * kPanel, m,
                            max(0, min(RW / 4, (live - r0 + 3) >> 2)), vval, cval, put, sh);
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
union StageLds {
  PanelLds panel;
  WyLds wy;
};

// R register rows of NW wavefronts hold leaves of up to 4 NW R rows.  ALONE: the
// leaf and the panel are the only ones, and Q is formed here, from what this
// workgroup has just written.  Eight blocks of 32 x 20 took 15.1 and 9.3 us in two
// launches and 23.2 in one, 243 x 32 32.9 and 15.1, and 46.1; the gap between the
// launches goes too.
template <int R, int NW, bool ALONE = false>
__global__ __launch_bounds__(64 * NW) void qr_leaf_factor(QrArgs q, int p) {
  __shared__ StageLds sh;
  leaf_factor<R, NW>(q, p, blockIdx.x, blockIdx.y, sh.panel);
  if (ALONE) {
    __syncthreads();
    leaf_wy<true, NW>(q, 0, 0, blockIdx.y, 0, sh.wy);
  }
}

// After the leaf factors of panel p: the first tree level's factors (`next`
// nodes per matrix; the first blocks, since the next launch waits for their
// 32 serial steps) beside the leaves' trailing columns.
template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void qr_leaf_trail(QrArgs q, int p, int trail, int next) {
  __shared__ StageLds sh;
  int x = blockIdx.x;
  if (x < next * q.count) {
    tree_factor_node<NW>(q, p, 1, x % next, x / next, sh.panel);
    return;
  }
  x -= next * q.count;
  const int per = q.nb * trail;
  leaf_wy<false, NW>(q, p, x % per / trail, x / per, x % trail, sh.wy);
}

// After the tree factors at stride s: the next level's factors beside those
// nodes' trailing columns.
__global__ __launch_bounds__(256, 2) void qr_tree_trail(QrArgs q, int p, int s, int nodes,
                                                        int trail, int next) {
  __shared__ StageLds sh;
  int x = blockIdx.x;
  if (x < next * q.count) {
    tree_factor_node(q, p, s * kArity, x % next, x / next, sh.panel);
    return;
  }
  x -= next * q.count;
  const int per = nodes * trail;
  tree_wy<false>(q, p, s, x % per / trail, x / per, x % trail, false, sh.wy);
}

__global__ __launch_bounds__(256, 2) void qr_tree_form(QrArgs q, int p, int s, int top) {
  __shared__ WyLds sh;
  tree_wy<true>(q, p, s, blockIdx.x, blockIdx.y, blockIdx.z, top != 0, sh);
}

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void qr_leaf_form(QrArgs q, int p) {
  __shared__ WyLds sh;
  leaf_wy<true, NW>(q, p, blockIdx.x, blockIdx.y, blockIdx.z, sh);
}

// wide: with eight-wavefront leaves where they pay.
QrPlan make_plan(int N, int k, bool wide = true) {
  QrPlan pl;
  pl.N = N;
  pl.k = k;
  int nb = N / (k > 128 ? k : 128);
  if (nb < 1) nb = 1;
  const int need = (N + kLeafRows - 1) / kLeafRows;
  if (nb < need) nb = need;
  if (nb > 1 && N / nb < k) nb = N / k;  // leaf 0 must hold k rows
  pl.nb = nb;
  pl.P = (k + kPanel - 1) / kPanel;
  auto levels = [](int leaves) {
    int depth = 0;
    for (long span = 1; span < leaves; span *= kArity) ++depth;
    return depth;
  };
  pl.depth = levels(nb);
  // twice as tall leaves where that saves a level of the tree (what the rows
  // above refuse stays refused)
  pl.wide = false;
  const int wnb = (N + kWideLeafRows - 1) / kWideLeafRows;
  if (wide && (N + nb - 1) / nb <= kLeafRows && levels(wnb) < pl.depth) {
    pl.wide = true;
    pl.nb = wnb;
    pl.depth = levels(wnb);
  }
  return pl;
}

}  // namespace

bool qr_plan_ok(int N, int k) {
  if (k <= 0 || N < k || k > kLeafRows) return false;
  const QrPlan pl = make_plan(N, k);
  return pl.wide || (N + pl.nb - 1) / pl.nb <= kLeafRows;
}

// The layout that N x k takes: its leaves, whether of eight wavefronts, and the
// levels of the tree above them (tests hold shapes to the branch they are there for).
void qr_plan_layout(int N, int k, int* leaves, int* wide, int* levels) {
  const QrPlan pl = make_plan(N, k);
  *leaves = pl.nb;
  *wide = pl.wide;
  *levels = pl.depth;
}

// Sized by the four-wavefront leaves, whose number grows with N: callers carve
// the workspace for their full N and also run fewer rows, whose plan may have more
// leaves than the full one's tall leaves (1152 rows 3, 1100 rows 8).
size_t qr_workspace_bytes(int count, int N, int k) {
  const QrPlan pl = make_plan(N, k, false);
  const size_t slots = (size_t)count * pl.P * pl.nb;
  const size_t n = 2 * slots * kPanel * kPanel + (size_t)count * N * k;
  return n * sizeof(double);
}

int launch_qr(int count, double* const* W, int N, int k, void* ws, hipStream_t s) {
  if (count <= 0 || k <= 0) return 0;
  if (count > kMaxProb || N < k || k > kLeafRows) {
    set_thread_error("launch_qr: need k <= N, k <= 192 and at most 8 matrices per launch");
    return 1;
  }
  const QrPlan pl = make_plan(N, k);
  if (!pl.wide && (N + pl.nb - 1) / pl.nb > kLeafRows) {
    set_thread_error("launch_qr: N too large for the leaf size (N/k too large)");
    return 1;
  }
  QrArgs q{};
  q.count = count;
  q.N = N;
  q.k = k;
  q.nb = pl.nb;
  q.P = pl.P;
  const size_t slots = (size_t)count * pl.P * pl.nb;
  q.Tl = (double*)ws;
  q.Tn = q.Tl + slots * kPanel * kPanel;
  double* work = q.Tn + slots * kPanel * kPanel;
  for (int i = 0; i < count; ++i) {
    q.W[i] = W[i];
    q.A[i] = work + (size_t)i * N * k;
  }
  q.rows = N / pl.nb;
  q.extra = N % pl.nb;
  const int leaf_rows = q.rows + (q.extra > 0);
  auto nodes_at = [&](int st) { return (pl.nb + st * kArity - 1) / (st * kArity); };

  for (int p = 0; p < pl.P; ++p) {
    const int c0 = p * kPanel, w = std::min(kPanel, k - c0);
    const int trail = (k - c0 - w + kTrailN - 1) / kTrailN;
    const dim3 leaves(pl.nb, count);
    auto factor = [&](auto alone) {
      constexpr bool A = decltype(alone)::value;
      if (leaf_rows <= 64)
        qr_leaf_factor<4, 4, A><<<leaves, 256, 0, s>>>(q, p);
      else if (leaf_rows <= 128)
        qr_leaf_factor<8, 4, A><<<leaves, 256, 0, s>>>(q, p);
      else if (leaf_rows <= kLeafRows)
        qr_leaf_factor<12, 4, A><<<leaves, 256, 0, s>>>(q, p);
      else if (leaf_rows <= 256)
        qr_leaf_factor<8, 8, A><<<leaves, 512, 0, s>>>(q, p);
      else
        qr_leaf_factor<12, 8, A><<<leaves, 512, 0, s>>>(q, p);
    };
    if (pl.nb == 1 && pl.P == 1) {
      factor(std::true_type{});
      CTM_HIP_TRY(hipGetLastError());
      return 0;
    }
    factor(std::false_type{});
    int next = pl.depth > 0 ? nodes_at(1) : 0;   // nodes of the next level to factor
    const int stage = count * (pl.nb * trail + next);
    if (stage && leaf_rows <= kLeafRows)
      qr_leaf_trail<4><<<stage, 256, 0, s>>>(q, p, trail, next);
    else if (stage)
      qr_leaf_trail<8><<<stage, 512, 0, s>>>(q, p, trail, next);
    for (int L = 0, st = 1; L < pl.depth; ++L, st *= kArity) {
      const int nodes = next;
      next = L + 1 < pl.depth ? nodes_at(st * kArity) : 0;
      if (nodes * trail + next)
        qr_tree_trail<<<count * (nodes * trail + next), 256, 0, s>>>(q, p, st, nodes, trail, next);
    }
  }
  for (int p = pl.P - 1; p >= 0; --p) {
    const int chunks = (k - p * kPanel + kTrailN - 1) / kTrailN;
    for (int L = pl.depth - 1; L >= 0; --L) {
      int st = 1;
      for (int i = 0; i < L; ++i) st *= kArity;
      qr_tree_form<<<dim3(nodes_at(st), count, chunks), 256, 0, s>>>(q, p, st, L == pl.depth - 1);
    }
    if (leaf_rows <= kLeafRows)
      qr_leaf_form<4><<<dim3(pl.nb, count, chunks), 256, 0, s>>>(q, p);
    else
      qr_leaf_form<8><<<dim3(pl.nb, count, chunks), 512, 0, s>>>(q, p);
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace sictm
