// SVD of the small (chi+p) x (chi+p) reduced matrix rho = Y M X (QR-based
// projector section, step 2), and of the chi x chi corners for the
// convergence measure.
//
// One-sided (Hestenes) Jacobi: U <- X V with V accumulating plane rotations
// until all column pairs of U are orthogonal to working precision; then
// s_j = |u_j|, u_j <- u_j / s_j.  One-sided Jacobi computes small singular
// values to high relative accuracy, which matters here because the
// pseudo-inverse s^-1/2 keeps directions down to a relative 1e-12.
// Preconditioning (Drmac & Veselic): the columns of A are sorted by norm
// (permutation P), A P = Q R by the Householder QR of this library, and the
// Jacobi iteration runs on X = R^T, which converges in a few sweeps where A
// itself needs dozens: R^T = Ut S V'^T gives A = (Q V') S (P Ut)^T.
//
// Up to n = 96 (128 for the values alone) one workgroup holds the columns of
// a matrix in LDS for all sweeps (svd_small).  Above that, and at every n where
// the caller asks for this order, block-pair parallel ordering: the columns are
// cut into blocks of kBlk; an outer sweep pairs the blocks in a round-robin
// tournament, four wavefronts per block pair and matrix, the rounds separated by
// the barriers of one workgroup (n <= 64), by grid barriers of one cooperative
// launch, or by launches inside a stream capture.  The columns of both blocks are
// loaded into LDS and the pairs across the two blocks rotated in kBlk steps of
// kBlk disjoint pairs (in the sweep's first round, where every block is visited
// once, the pairs within each block first, in kBlk - 1 more steps), so that
// every column pair meets once per sweep; 16 lanes per pair (rows spread over
// the lanes, dot products reduced by DPP row sums); the rotations of the visit
// are accumulated in a 2 kBlk x 2 kBlk matrix W and applied to the right vectors
// once at the end (V_cols <- V_cols W).  A per-matrix flag records whether a
// sweep rotated anything, and the sweeps end after one without rotations.
// Columns that end numerically zero (rank-deficient input) are replaced by an
// orthonormal completion so that u stays orthogonal.  Singular values are
// returned in descending order (ties by index).

#include "common.h"

#include <hip/hip_cooperative_groups.h>

namespace sictm {
namespace {

constexpr int kSvdMaxN = 192;   // the preconditioning QR holds n <= 192 rows per leaf
constexpr int kRPL = kSvdMaxN / 64;   // rows per lane in the finalisation
constexpr int kCompChunk = 32;       // non-zero columns staged per LDS pass of the completion
constexpr int kBlk = 16;              // columns per block
constexpr int kMaxSweeps = 24;
constexpr int kLanesPerPair = 16;

__device__ __forceinline__ double wsum(double x) { return wave_sum64(x); }

__device__ __forceinline__ double gsum16(double x) { return row_sum16(x); }

struct SvdArgs {
  const double* A[kMaxProb];   // matrices the Jacobi kernels act on (R^T)
  double* U[kMaxProb];         // Jacobi outputs: left vectors of R^T (Ut) ...
  double* S[kMaxProb];
  double* V[kMaxProb];         // ... and right vectors (V')
  double* work;       // [count][2][n][n] column-major working columns
  int* flags;         // [count][kMaxSweeps] "a rotation happened in sweep s"
  int n, nblk, want_v;
  // preconditioning
  const double* Ain[kMaxProb]; // the caller's matrices
  double* Wp[kMaxProb];        // A P, then Q
  double* Wc[kMaxProb];        // A P
  double* Ut[kMaxProb];        // left vectors of R^T
  int* perm;                   // [count][n]
  double* fro2;                // [count] squared Frobenius norm of each input
};

// Tournament position -> block / column index (position 0 fixed).
__device__ __forceinline__ int tour(int pos, int round, int m) {
  return pos == 0 ? 0 : ((pos - 1 + round) % (m - 1)) + 1;
}

__global__ void svd_init(SvdArgs a) {
  const int mat = blockIdx.y;
  const int n = a.n;
  double* Uc = a.work + (size_t)mat * 2 * n * n;
  double* Vc = Uc + (size_t)n * n;
  const double* A = a.A[mat];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n * n; i += gridDim.x * blockDim.x) {
    const int r = i / n, c = i % n;
    Uc[(size_t)c * n + r] = A[i];
    if (a.want_v) Vc[(size_t)c * n + r] = (r == c) ? 1.0 : 0.0;
  }
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < kMaxSweeps; i += blockDim.x) a.flags[mat * kMaxSweeps + i] = 0;
}

// Column norms, stable descending sort -> perm (the copy Wp = Wc = A[:, perm]
// follows in svd_prep_copy).  Thread c sums column c down the rows, so
// that each row is read by consecutive threads.
__global__ __launch_bounds__(256) void svd_prep(SvdArgs a) {
  __shared__ double nrm[kSvdMaxN];
  __shared__ int perm[kSvdMaxN];
  const int mat = blockIdx.x, n = a.n, tid = threadIdx.x;
  const double* A = a.Ain[mat];
  for (int c = tid; c < n; c += 256) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int r = 0;
    for (; r + 3 < n; r += 4) {
      const double x0 = A[(size_t)r * n + c], x1 = A[(size_t)(r + 1) * n + c];
      const double x2 = A[(size_t)(r + 2) * n + c], x3 = A[(size_t)(r + 3) * n + c];
      s0 += x0 * x0;
      s1 += x1 * x1;
      s2 += x2 * x2;
      s3 += x3 * x3;
    }
    for (; r < n; ++r) s0 += A[(size_t)r * n + c] * A[(size_t)r * n + c];
    nrm[c] = (s0 + s1) + (s2 + s3);
  }
  __syncthreads();
  if (tid == 0) {
    double f = 0.0;
    for (int c = 0; c < n; ++c) f += nrm[c];
    a.fro2[mat] = f;
  }
  for (int c = tid; c < n; c += 256) {
    int rank = 0;
    const double v = rank_key(nrm[c]);
    for (int o = 0; o < n; ++o) {
      const double w = rank_key(nrm[o]);
      rank += (w > v) || (w == v && o < c);
    }
    perm[rank] = c;
  }
  __syncthreads();
  int* pg = a.perm + (size_t)mat * n;
  for (int c = tid; c < n; c += 256) pg[c] = perm[c];
}

// Wp = Wc = A[:, perm], over the blocks of x (matrix blockIdx.y).
__global__ __launch_bounds__(256) void svd_prep_copy(SvdArgs a) {
  const int mat = blockIdx.y, n = a.n;
  const double* A = a.Ain[mat];
  const int* pg = a.perm + (size_t)mat * n;
  double* Wp = a.Wp[mat];
  double* Wc = a.Wc[mat];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n * n; i += gridDim.x * 256) {
    const int r = i / n, j = i % n;
    const double v = A[(size_t)r * n + pg[j]];
    Wp[i] = v;
    Wc[i] = v;
  }
}

// v[perm[i], :] = Ut[i, :]
__global__ void svd_unpermute_rows(SvdArgs a) {
  const int mat = blockIdx.y, n = a.n;
  const int* pg = a.perm + (size_t)mat * n;
  const double* Ut = a.Ut[mat];
  double* V = a.V[mat];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n * n; i += gridDim.x * blockDim.x) {
    const int r = i / n, c = i % n;
    V[(size_t)pg[r] * n + c] = Ut[i];
  }
}

// 1/sqrt(x) and 1/x to full double precision from the hardware estimates
// (Newton steps); used for the rotation angles, where x > 0.
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double h = 0.5 * x * y;
  y = fma(y, fma(-h, y, 0.5), y);
  h = 0.5 * x * y;
  return fma(y, fma(-h, y, 0.5), y);
}
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// The plane rotation that orthogonalises two columns with squared norms al,
// be and product ga (all divided by the squared norm of the matrix, which
// keeps their products in range): t, the smaller root of
// t^2 + 2 zeta t = 1 with zeta = (be - al) / (2 ga), c and s.  False when
// the pair is orthogonal to working precision (|ga| <= tol sqrt(al be), tol =
// 1e-15 sqrt(n)) or a column is numerically zero: below 1e-15 of the matrix norm,
// rotating cannot converge in the relative sense and does not change the
// result above roundoff; such columns are completed at the end.  `counts`:
// the rotation is clearly above roundoff (a pair left at |ga| ~ tol sqrt(al
// be) keeps being rotated but does not prevent the sweeps from stopping).
// The norms follow the rotation, al - t ga and be + t ga, and are summed anew
// from the columns every sweep (visit).
struct SvdScale {
  double scale, tol2, cut;
};
__device__ __forceinline__ SvdScale svd_scale(double fro2, int n) {
  const double scale = fro2 > 1e-300 ? 1.0 / fro2 : 1e300;
  return {scale, 1e-30 * n, 1e-30 * (fro2 * scale)};
}
__device__ __forceinline__ bool plane_rotation(double al, double be, double ga, const SvdScale& f,
                                               double& t, double& c, double& s, bool& counts) {
  const double g2 = ga * ga, thr = f.tol2 * (al * be);
  counts = g2 > 256.0 * thr;
  if (!(g2 > thr && al > f.cut && be > f.cut)) return false;
  const double d = be - al, h2 = fma(d, d, 4.0 * g2);
  const double h = h2 * fast_rsqrt(h2);
  t = copysign(2.0 * ga, d * ga) * fast_rcp(fabs(d) + h);
  c = fast_rsqrt(fma(t, t, 1.0));
  s = c * t;
  return true;
}

// All sweeps of a small matrix in one workgroup, with the columns of U (and
// of V) in LDS: a sweep is a sequence of halvings, each pairing the columns
// of the first half of every set with those of the second (h steps for
// halves of h columns, pair (i, (i + r) mod h) in step r), then the halves
// with themselves: n - 1 steps and a few more for odd sizes.  16 lanes hold
// a pair; the column of the first half stays in their registers for the h
// steps, so that a step moves one column through LDS, sums one product and
// has one barrier.  (Rotations with c left to a scale per column halve the
// arithmetic and measured 1 to 5 % slower: the scales lengthen the chain.)
//
// Bound by the latency of a step (a 16-lane sum, three reciprocal square
// roots and reciprocals, one LDS round trip).  Used where
// U and V (U alone for values only) fit the LDS; above that the block-pair
// kernels spread the columns over several CUs.  Measured, 4 random matrices with
// vectors, before (block pairs of 16 columns at every size) and after: n = 20
// 374 and 154 us, 64 872 and 480, 87 1724 and 950, 96 1630 and 1013; values
// only, n = 100: 1732 and 1066.
template <int RPL, bool WANT_V>
struct SmallSvd {
  static constexpr int ROWS = 16 * RPL;
  // columns 16 rows apart modulo 32 fall 32 banks apart for the two pairs of
  // a half wavefront; where that does not fit, an odd stride
  static constexpr int LD = ROWS <= 48 ? 48 : ROWS <= 80 ? 80 : ROWS + 1;
  double U[ROWS][LD];
  double V[WANT_V ? ROWS : 1][WANT_V ? LD : 1];
  double nrm[ROWS];
};

template <int RPL, bool WANT_V>
__global__ __launch_bounds__(8 * 16 * RPL) void svd_small(SvdArgs a) {
  using L = SmallSvd<RPL, WANT_V>;
  constexpr int NT = 8 * L::ROWS;
  __shared__ L sh;
  const int n = a.n, mat = blockIdx.x;
  const int tid = threadIdx.x, grp = tid >> 4, li = tid & 15;
  const double* A = a.A[mat];
  // U[c][r] = A[r][c], V = I; rows from n on hold zeros
  for (int i = tid; i < n * L::ROWS; i += NT) {
    const int r = i / n, c = i % n;
    sh.U[c][r] = r < n ? A[(size_t)r * n + c] : 0.0;
    if (WANT_V) sh.V[c][r] = r == c ? 1.0 : 0.0;
  }
  const SvdScale f = svd_scale(a.fro2[mat], n);
  __syncthreads();
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    for (int c = grp; c < n; c += NT / 16) {
      double x = 0.0;
#pragma unroll
      for (int t = 0; t < RPL; ++t) x = fma(sh.U[c][li + 16 * t], sh.U[c][li + 16 * t], x);
      x = gsum16(x) * f.scale;
      if (li == 0) sh.nrm[c] = x;
    }
    __syncthreads();
    int rotated = 0;
    int h = (n + 1) >> 1;   // columns of a half at this level
    for (int level = 0;; ++level) {
      // odd sizes leave more first-half columns than there are groups
      for (int g0 = 0; g0 < h << level; g0 += NT / 16) {
        // this group's set [base, base + size) and its place idx in the first half
        int base = 0, size = n;
        const int set = (g0 + grp) / h, idx = (g0 + grp) % h;
        bool in = set < (1 << level);
        for (int b = level - 1; b >= 0 && in; --b) {   // descend to the set
          const int half = (size + 1) >> 1;
          if ((set >> b) & 1) {
            base += half;
            size -= half;
          } else {
            size = half;
          }
        }
        const int half = (size + 1) >> 1;   // of this set: h or one less
        in = in && idx < half && size > 1;
        const int p = base + idx;
        double up[RPL], vp[RPL], al = 0.0;
        if (in) {
          al = sh.nrm[p];
#pragma unroll
          for (int t = 0; t < RPL; ++t) {
            up[t] = sh.U[p][li + 16 * t];
            if (WANT_V) vp[t] = sh.V[p][li + 16 * t];
          }
        }
        for (int r = 0; r < h; ++r) {
          int k = idx + r;
          k = k >= h ? k - h : k;   // place in the second half
          if (in && half + k < size) {
            const int q = base + half + k;
            double uq[RPL];
            double ga = 0.0, g1 = 0.0;
#pragma unroll
            for (int t = 0; t < RPL; ++t) uq[t] = sh.U[q][li + 16 * t];
            const double be = sh.nrm[q];
#pragma unroll
            for (int t = 0; t < RPL; t += 2) {
              ga = fma(up[t], uq[t], ga);
              if (t + 1 < RPL) g1 = fma(up[t + 1], uq[t + 1], g1);
            }
            ga = gsum16(ga + g1) * f.scale;
            double t_, c, s;
            bool counts;
            if (plane_rotation(al, be, ga, f, t_, c, s, counts)) {
              rotated |= counts;
#pragma unroll
              for (int t = 0; t < RPL; ++t) {
                const double x = up[t], y = uq[t];
                up[t] = c * x - s * y;
                sh.U[q][li + 16 * t] = s * x + c * y;
              }
              if (WANT_V) {
#pragma unroll
                for (int t = 0; t < RPL; ++t) {
                  const double x = vp[t], y = sh.V[q][li + 16 * t];
                  vp[t] = c * x - s * y;
                  sh.V[q][li + 16 * t] = s * x + c * y;
                }
              }
              al = fma(-t_, ga, al);
              if (li == 0) sh.nrm[q] = fma(t_, ga, be);
            }
          }
          __syncthreads();
        }
        if (in) {
          if (li == 0) sh.nrm[p] = al;
#pragma unroll
          for (int t = 0; t < RPL; ++t) {
            sh.U[p][li + 16 * t] = up[t];
            if (WANT_V) sh.V[p][li + 16 * t] = vp[t];
          }
        }
        __syncthreads();
      }
      if (h == 1) break;
      h = (h + 1) >> 1;
    }
    if (!__syncthreads_or(rotated)) break;
  }
  double* Uc = a.work + (size_t)mat * 2 * n * n;
  double* Vc = Uc + (size_t)n * n;
  for (int i = tid; i < n * n; i += NT) {
    const int c = i / n, r = i % n;
    Uc[i] = sh.U[c][r];
    if (WANT_V) Vc[i] = sh.V[c][r];
  }
}

// Where the one-workgroup kernel applies.
bool small_svd_fits(int n, bool want_v) { return n <= (want_v ? 96 : 128); }

template <bool WANT_V>
void launch_small_svd(const SvdArgs& a, int count, hipStream_t s) {
  const int n = a.n;
  if (n <= 32)
    svd_small<2, WANT_V><<<count, 256, 0, s>>>(a);
  else if (n <= 48)
    svd_small<3, WANT_V><<<count, 384, 0, s>>>(a);
  else if (n <= 64)
    svd_small<4, WANT_V><<<count, 512, 0, s>>>(a);
  else if (n <= 80)
    svd_small<5, WANT_V><<<count, 640, 0, s>>>(a);
  else if (n <= 96)
    svd_small<6, WANT_V><<<count, 768, 0, s>>>(a);
  else
    svd_small<8, false><<<count, 1024, 0, s>>>(a);
}

// One round of an outer sweep: block pair (tournament positions bp,
// nblk-1-bp).  The 2 kBlk columns of U live in LDS; the rotations of the
// visit are accumulated in a 2 kBlk x 2 kBlk matrix W (also in LDS) and the
// right vectors are updated once at the end, V_cols <- V_cols W.  RPL is the
// number of rows per lane (n <= 16 RPL).  Norms and products are summed anew in
// every step, in the order of the blocks: unit cells amplify the last bits of
// these vectors (cell.hip), so the order and the sums are part of what this
// computes (the fma calls fix its rounding).  Bound by the latency of a step, like
// svd_small, and by the grid barriers; across blocks a column of the first stays in
// registers.  4 random matrices with vectors, n = 100: 2200 us with both columns
// through LDS, 1715 so; 144: 3238, 2688; 160: 3329, 2789 (norms tracked from step to
// step and narrower blocks, a different order: 1570, 2560, 2691).
template <int RPL>
struct RoundLds {
  static constexpr int kC = 2 * kBlk;
  static constexpr int LD = 16 * RPL + 1;   // odd row length: no bank conflicts
  double Ul[kC][LD];
  double Vl[kC][LD];
  double Wl[kC][kC + 1];
  int rot;
};

template <int RPL>
__device__ __forceinline__ void block_round(const SvdArgs& a, int sweep, int round, int mat, int bp,
                                            RoundLds<RPL>& sh) {
  constexpr int kC = RoundLds<RPL>::kC;
  auto& Ul = sh.Ul;
  auto& Vl = sh.Vl;
  auto& Wl = sh.Wl;
  int& rot = sh.rot;
  const int n = a.n, nblk = a.nblk;
  const int b0 = tour(bp, round, nblk), b1 = tour(nblk - 1 - bp, round, nblk);
  const int tid = threadIdx.x & 255;   // of the block pair's four wavefronts
  double* Uc = a.work + (size_t)mat * 2 * n * n;
  double* Vc = Uc + (size_t)n * n;
  // local column j -> global column: j < kBlk from b0, else from b1
  auto gcol = [&](int j) { return (j < kBlk ? b0 : b1) * kBlk + (j % kBlk); };
  // the columns of U (and of V) into LDS, one column per wave at a time, rows
  // lane + 64 t: coalesced, with no index division; four columns per wave in
  // flight
  const int nv = a.want_v ? 2 : 1;
  const int wv = tid / 64, ln = tid % 64;
  constexpr int kRW = (16 * RPL + 63) / 64;   // row chunks per lane (n <= 16 RPL)
  const int ncol = nv * kC;
  for (int c0 = wv; c0 < ncol; c0 += 16) {
    double t[4][kRW];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = c0 + 4 * u, g = gcol(cc % kC);
      const double* src = (cc < kC ? Uc : Vc) + (size_t)g * n;
#pragma unroll
      for (int r = 0; r < kRW; ++r) {
        const int row = ln + 64 * r;
        t[u][r] = (cc < ncol && g < n && row < n) ? src[row] : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = c0 + 4 * u;
      if (cc < ncol) {
        double* dst = cc < kC ? Ul[cc] : Vl[cc - kC];
#pragma unroll
        for (int r = 0; r < kRW; ++r) {
          const int row = ln + 64 * r;
          if (row < n)
            dst[row] = t[u][r];
          else if (row < 16 * RPL)
            dst[row] = 0.0;   // rows n .. 16 RPL - 1 hold exact zeros
        }
      }
    }
  }
  for (int idx = tid; idx < kC * kC; idx += 256) Wl[idx / kC][idx % kC] = (idx / kC == idx % kC);
  if (tid == 0) rot = 0;
  __syncthreads();
  const int grp = tid / kLanesPerPair, li = tid % kLanesPerPair;   // 16 pair groups
  const double tol = 1e-15 * sqrt((double)n);
  // columns below 1e-15 of the matrix norm are numerically zero: rotating
  // them against the others cannot converge in the relative sense and does
  // not change the result above roundoff; they are completed at the end
  const double negl = 1e-30 * a.fro2[mat];
  int my_rot = 0;
  // The rotation of columns up (of the first index) and uq: its cosine and sine,
  // or false.
  auto rotation = [&](const double (&up)[RPL], const double (&uq)[RPL], double& c, double& s) {
    double al = fma(up[0], up[0], up[1] * up[1]), be = fma(uq[0], uq[0], uq[1] * uq[1]);
    double ga = fma(up[1], uq[1], up[0] * uq[0]);
#pragma unroll
    for (int t = 2; t < RPL; ++t) {   // rows n .. 16 RPL - 1 are zero: no guard
      al = fma(up[t], up[t], al);
      be = fma(uq[t], uq[t], be);
      ga = fma(up[t], uq[t], ga);
    }
    al = gsum16(al);
    be = gsum16(be);
    ga = gsum16(ga);
    const double thr = tol * sqrt(al) * sqrt(be);
    if (!(ga != 0.0 && fabs(ga) > thr && al > negl && be > negl)) return false;
    // tan of the rotation angle, the smaller root of t^2 + 2 zeta t = 1
    const double zeta = (be - al) * fast_rcp(2.0 * ga);
    const double z2 = fma(zeta, zeta, 1.0);
    const double t = (zeta >= 0.0 ? 1.0 : -1.0) * fast_rcp(fma(z2, fast_rsqrt(z2), fabs(zeta)));
    c = fast_rsqrt(fma(t, t, 1.0));
    s = c * t;
    // convergence counts only rotations clearly above roundoff: a pair
    // left at |gamma| ~ tol sqrt(alpha beta) keeps being rotated but does
    // not prevent the sweep loop from stopping
    my_rot |= fabs(ga) > 16.0 * thr;
    return true;
  };
  // the sweep's first round (every block in exactly one pair) also pairs the
  // columns within each block: kBlk - 1 steps of a round-robin per block,
  // kBlk / 2 pairs of each block per step
  for (int r = 0; r < (round == 0 ? kBlk - 1 : 0); ++r) {
    const int blk = grp / (kBlk / 2), k = grp % (kBlk / 2);
    const int ca = tour(k, r, kBlk), cb = tour(kBlk - 1 - k, r, kBlk);
    const int p = blk * kBlk + min(ca, cb), q = blk * kBlk + max(ca, cb);
    if (gcol(p) < n && gcol(q) < n) {
      double up[RPL], uq[RPL], c, s;
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        up[t] = Ul[p][li + 16 * t];
        uq[t] = Ul[q][li + 16 * t];
      }
      if (rotation(up, uq, c, s)) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          Ul[p][li + 16 * t] = fma(c, up[t], -(s * uq[t]));
          Ul[q][li + 16 * t] = fma(c, uq[t], s * up[t]);
        }
        if (a.want_v) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const double wp = Wl[li + 16 * t][p], wq = Wl[li + 16 * t][q];
            Wl[li + 16 * t][p] = fma(c, wp, -(s * wq));
            Wl[li + 16 * t][q] = fma(s, wp, c * wq);
          }
        }
      }
    }
    __syncthreads();
  }
  // then kBlk steps pair column i of the first block, which stays in the
  // registers of its lanes, with column (i + step) mod kBlk of the second, so
  // that a sweep meets every column pair exactly once
  {
    const int p = grp;
    const bool in = gcol(p) < n;
    double up[RPL], wp[2];
#pragma unroll
    for (int t = 0; t < RPL; ++t) up[t] = Ul[p][li + 16 * t];
#pragma unroll
    for (int t = 0; t < 2; ++t) wp[t] = Wl[li + 16 * t][p];
    for (int r = 0; r < kBlk; ++r) {
      const int q = kBlk + (grp + r) % kBlk;
      if (in && gcol(q) < n) {
        double uq[RPL], wq[2], c, s;
#pragma unroll
        for (int t = 0; t < RPL; ++t) uq[t] = Ul[q][li + 16 * t];
#pragma unroll
        for (int t = 0; t < 2; ++t) wq[t] = Wl[li + 16 * t][q];
        if (rotation(up, uq, c, s)) {
#pragma unroll
          for (int t = 0; t < RPL; ++t) {
            const double x = up[t], y = uq[t];
            up[t] = fma(c, x, -(s * y));
            Ul[q][li + 16 * t] = fma(c, y, s * x);
          }
          if (a.want_v) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const double x = wp[t], y = wq[t];
              wp[t] = fma(c, x, -(s * y));
              Wl[li + 16 * t][q] = fma(s, x, c * y);
            }
          }
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < RPL; ++t) Ul[p][li + 16 * t] = up[t];
#pragma unroll
    for (int t = 0; t < 2; ++t) Wl[li + 16 * t][p] = wp[t];
    __syncthreads();
  }
  if (li == 0 && my_rot) atomicOr(&rot, 1);
  for (int j = wv; j < kC; j += 4) {
    const int g = gcol(j);
    if (g < n) {
#pragma unroll
      for (int r = 0; r < kRW; ++r) {
        const int row = ln + 64 * r;
        if (row < n) Uc[(size_t)g * n + row] = Ul[j][row];
      }
    }
  }
  if (a.want_v) {
    // V_cols <- V_cols W, register-blocked over the whole workgroup: thread
    // (rg, cg) computes rows rg + 32 i of columns kVc cg .. kVc cg + kVc - 1
    // (each sum over l in ascending order from zero, 20 independent chains
    // per thread in place of one 32-long chain per row)
    constexpr int kVr = (16 * RPL + 31) / 32, kVc = kC / 8;
    const int rg = tid % 32, cg = tid / 32;
    double acc[kVr][kVc];
#pragma unroll
    for (int i = 0; i < kVr; ++i)
#pragma unroll
      for (int c = 0; c < kVc; ++c) acc[i][c] = 0.0;
#pragma unroll 4
    for (int l = 0; l < kC; ++l) {
      double w[kVc];
#pragma unroll
      for (int c = 0; c < kVc; ++c) w[c] = Wl[l][kVc * cg + c];
#pragma unroll
      for (int i = 0; i < kVr; ++i) {
        const int r = rg + 32 * i;
        const double v = r < n ? Vl[l][r] : 0.0;
#pragma unroll
        for (int c = 0; c < kVc; ++c) acc[i][c] += v * w[c];
      }
    }
#pragma unroll
    for (int c = 0; c < kVc; ++c) {
      const int g = gcol(kVc * cg + c);
      if (g < n) {
#pragma unroll
        for (int i = 0; i < kVr; ++i) {
          const int r = rg + 32 * i;
          if (r < n) Vc[(size_t)g * n + r] = acc[i][c];
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0 && rot) atomicOr(&a.flags[mat * kMaxSweeps + sweep], 1);
}

// One round per launch; later launches return at once after a sweep
// without rotations.
template <int RPL>
__global__ __launch_bounds__(256) void svd_block_round(SvdArgs a, int sweep, int round) {
  __shared__ RoundLds<RPL> sh;
  const int mat = blockIdx.y;
  if (sweep > 0 && a.flags[mat * kMaxSweeps + sweep - 1] == 0) return;   // converged
  block_round<RPL>(a, sweep, round, mat, blockIdx.x, sh);
}

// All sweeps in one cooperative launch: a grid-wide barrier separates the
// rounds, matrices whose last sweep rotated nothing stop working, and the
// launch ends when every matrix has converged (a decision every workgroup
// takes from the same flags after the barrier).
template <int RPL>
__global__ __launch_bounds__(256) void svd_sweeps(SvdArgs a, int count) {
  __shared__ RoundLds<RPL> sh;
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const int mat = blockIdx.y;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    const bool active = sweep == 0 || a.flags[mat * kMaxSweeps + sweep - 1] != 0;
    for (int round = 0; round < a.nblk - 1; ++round) {
      if (active) block_round<RPL>(a, sweep, round, mat, blockIdx.x, sh);
      grid.sync();
    }
    bool any = false;
    for (int m = 0; m < count; ++m) any |= a.flags[m * kMaxSweeps + sweep] != 0;
    if (!any) break;
  }
}

// All sweeps in one ordinary launch, where one workgroup holds all G block pairs of
// a matrix (n <= 64): its barriers separate the rounds.  A cooperative launch goes
// to a queue of its own, for which the stream waits both ways: a unit cell of one
// site, D 2, k = 40, took 6.0 ms an iteration beside other contexts, 3.9 so.  Kernel times are alike (4 matrices, n = 48: 780 us with two
// workgroups and both columns through LDS, 655 so; n = 64: 829 and 842); three pairs
// on one CU take 1544 us at n = 70, where the cooperative launch takes 1288.
template <int RPL, int G>
__global__ __launch_bounds__(256 * G) void svd_sweeps_one(SvdArgs a) {
  __shared__ RoundLds<RPL> sh[G];
  const int mat = blockIdx.x, pair = threadIdx.x >> 8;
  int* flags = a.flags + mat * kMaxSweeps;
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    for (int round = 0; round < a.nblk - 1; ++round) {
      block_round<RPL>(a, sweep, round, mat, pair, sh[pair]);
      __syncthreads();
    }
    if (!__hip_atomic_load(&flags[sweep], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
  }
}

// Singular values, normalisation, completion of zero columns, ordering.
__global__ __launch_bounds__(1024) void svd_finalize(SvdArgs a) {
  const int mat = blockIdx.x;
  const int n = a.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int nwaves = 1024 / 64;
  double* Uc = a.work + (size_t)mat * 2 * n * n;
  double* Vc = Uc + (size_t)n * n;
  __shared__ double snorm[kSvdMaxN];
  __shared__ int order[kSvdMaxN];
  // singular values = column norms
  for (int c = wave; c < n; c += nwaves) {
    double ss = 0.0;
    for (int r = lane; r < n; r += 64) ss += Uc[(size_t)c * n + r] * Uc[(size_t)c * n + r];
    ss = wsum(ss);
    if (lane == 0) snorm[c] = sqrt(ss);
  }
  __syncthreads();
  // normalise non-zero columns
  for (int c = wave; c < n; c += nwaves) {
    const double sn = snorm[c];
    if (sn > 0.0)
      for (int r = lane; r < n; r += 64) Uc[(size_t)c * n + r] /= sn;
  }
  __syncthreads();
  // orthonormal completion of numerically zero columns; the cut is the one
  // below which the rotations left a column alone.  The unit vectors are
  // projected on the complement of the non-zero columns at once
  // (X = I - U U^T), and the complement's basis is drawn from X's columns
  // in index order by Gram-Schmidt: the zero columns, in index order, take
  // the unit vectors e_0, e_1, ... that keep enough of their length after
  // the projection on the complement of the non-zero columns and of the
  // zero columns completed before.  Wavefront w keeps columns w, w + 16, ...
  // of X in registers, rows lane, lane + 64, lane + 128.  The errors of one
  // pass grow with the inverse of the length that is left, and from one
  // column to the next, so a candidate that keeps less than 0.7 of its length
  // is projected a second time, by all wavefronts, on the columns themselves.
  const double zero_cut = 1e-15 * sqrt(a.fro2[mat]);
  if (a.U[mat] != nullptr) {
    __shared__ int nzl[kSvdMaxN], zl[kSvdMaxN];
    __shared__ int cnt[2];
    __shared__ double qs[kSvdMaxN];
    __shared__ int took[2];
    __shared__ double ust[kCompChunk][kSvdMaxN];
    if (wave == 0) {
      int nr = 0, nz = 0;
      for (int base = 0; base < n; base += 64) {
        const int c = base + lane;
        const bool in = c < n;
        const bool live = in && snorm[c] > zero_cut;
        const unsigned long long ml = __ballot(live), mz = __ballot(in && !live);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (live) nzl[nr + __popcll(ml & below)] = c;
        else if (in) zl[nz + __popcll(mz & below)] = c;
        nr += __popcll(ml);
        nz += __popcll(mz);
      }
      if (lane == 0) {
        cnt[0] = nr;
        cnt[1] = nz;
      }
    }
    __syncthreads();
    const int nr = cnt[0], nz = cnt[1];
    if (nz > 0) {
      constexpr int CPW = kSvdMaxN / nwaves;   // columns per wavefront
      double x[CPW][kRPL];
#pragma unroll
      for (int q = 0; q < CPW; ++q)
#pragma unroll
        for (int e = 0; e < kRPL; ++e) {
          const int j = wave + nwaves * q, i = lane + 64 * e;
          x[q][e] = (i == j && j < n) ? 1.0 : 0.0;
        }
      // X -= U_nz U_nz^T, kCompChunk non-zero columns staged in LDS at a time
      for (int o0 = 0; o0 < nr; o0 += kCompChunk) {
        const int m = min(kCompChunk, nr - o0);
        for (int t = tid; t < m * n; t += 1024) {
          const int oo = t / n, i = t % n;
          ust[oo][i] = Uc[(size_t)nzl[o0 + oo] * n + i];
        }
        __syncthreads();
        for (int oo = 0; oo < m; ++oo) {
          double ui[kRPL];
#pragma unroll
          for (int e = 0; e < kRPL; ++e) {
            const int i = lane + 64 * e;
            ui[e] = i < n ? ust[oo][i] : 0.0;
          }
#pragma unroll
          for (int q = 0; q < CPW; ++q) {
            const int j = wave + nwaves * q;
            const double uj = j < n ? ust[oo][j] : 0.0;
#pragma unroll
            for (int e = 0; e < kRPL; ++e) x[q][e] -= uj * ui[e];
          }
        }
        __syncthreads();
      }
      // candidates in index order: a column of X that keeps more than
      // 1/(2 sqrt(n)) of its length (some column of the complement's
      // projector always does) becomes the next zero column and is removed
      // from the later candidates
      const double keep_min = 0.5 / sqrt((double)n);
      int t = 0;
      for (int cand = 0; cand < n && t < nz; ++cand) {
        if (wave == cand % nwaves) {
          const int qc = cand / nwaves;
          double xc[kRPL] = {};
#pragma unroll
          for (int q = 0; q < CPW; ++q)
            if (q == qc)
#pragma unroll
              for (int e = 0; e < kRPL; ++e) xc[e] = x[q][e];
          double ss = 0.0;
#pragma unroll
          for (int e = 0; e < kRPL; ++e) ss += xc[e] * xc[e];
          const double nn = sqrt(wsum(ss));
          const bool take = nn > keep_min;
          if (take) {
            const double inv = 1.0 / nn;
#pragma unroll
            for (int e = 0; e < kRPL; ++e) {
              const int i = lane + 64 * e;
              if (i < n) qs[i] = xc[e] * inv;
            }
          }
          if (lane == 0) took[cand & 1] = take ? (nn < 0.7 ? 2 : 1) : 0;
        }
        __syncthreads();
        const int how = took[cand & 1];
        if (!how) continue;
        if (how == 2) {
          double v[kRPL], y[kRPL];
#pragma unroll
          for (int e = 0; e < kRPL; ++e) {
            const int i = lane + 64 * e;
            v[e] = i < n ? qs[i] : 0.0;
            y[e] = 0.0;
          }
          for (int o = wave; o < nr + t; o += nwaves) {
            const double* u = Uc + (size_t)(o < nr ? nzl[o] : zl[o - nr]) * n;
            double uo[kRPL], d = 0.0;
#pragma unroll
            for (int e = 0; e < kRPL; ++e) {
              const int i = lane + 64 * e;
              uo[e] = i < n ? u[i] : 0.0;
              d += uo[e] * v[e];
            }
            d = wsum(d);
#pragma unroll
            for (int e = 0; e < kRPL; ++e) y[e] += d * uo[e];
          }
#pragma unroll
          for (int e = 0; e < kRPL; ++e) ust[wave][lane + 64 * e] = y[e];
          __syncthreads();
          if (wave == 0) {
            double ss = 0.0;
#pragma unroll
            for (int e = 0; e < kRPL; ++e) {
              double z = 0.0;
#pragma unroll
              for (int w = 0; w < nwaves; ++w) z += ust[w][lane + 64 * e];
              v[e] -= z;
              ss += v[e] * v[e];
            }
            const double inv = 1.0 / sqrt(wsum(ss));
#pragma unroll
            for (int e = 0; e < kRPL; ++e) {
              const int i = lane + 64 * e;
              if (i < n) qs[i] = v[e] * inv;
            }
          }
          __syncthreads();
        }
        if (tid < n) Uc[(size_t)zl[t] * n + tid] = qs[tid];
        ++t;
        if (t == nz) break;
        double qv[kRPL];
#pragma unroll
        for (int e = 0; e < kRPL; ++e) {
          const int i = lane + 64 * e;
          qv[e] = i < n ? qs[i] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < CPW; ++q) {
          const int j = wave + nwaves * q;
          if (j <= cand || j >= n) continue;
          double d = 0.0;
#pragma unroll
          for (int e = 0; e < kRPL; ++e) d += qv[e] * x[q][e];
          d = wsum(d);
#pragma unroll
          for (int e = 0; e < kRPL; ++e) x[q][e] -= d * qv[e];
        }
        __syncthreads();
      }
    }
  }
  __syncthreads();
  // descending order, ties by index
  for (int c = tid; c < n; c += 1024) {
    const double sc = rank_key(snorm[c]);
    int rank = 0;
    for (int o = 0; o < n; ++o) {
      const double so = rank_key(snorm[o]);
      rank += (so > sc) || (so == sc && o < c);
    }
    order[rank] = c;
  }
  __syncthreads();
  double* S = a.S[mat];
  double* U = a.U[mat];
  double* V = a.V[mat];
  for (int i = tid; i < n; i += 1024) S[i] = snorm[order[i]];
  for (int i = tid; i < n * n; i += 1024) {
    const int r = i / n, j = i % n;
    const int c = order[j];
    if (U) U[i] = Uc[(size_t)c * n + r];
    if (V) V[i] = Vc[(size_t)c * n + r];
  }
}

// The block-pair kernels: one workgroup per matrix up to n = 64, above that one
// cooperative launch, or inside a stream capture (where none can be recorded) one
// launch per round.
int launch_block_svd(const SvdArgs& a, int count, hipStream_t s) {
  const int n = a.n, nblk = a.nblk;
  if (nblk <= 4) {
    if (nblk == 2)
      svd_sweeps_one<2, 1><<<count, 256, 0, s>>>(a);
    else if (n <= 48)
      svd_sweeps_one<3, 2><<<count, 512, 0, s>>>(a);
    else
      svd_sweeps_one<4, 2><<<count, 512, 0, s>>>(a);
    CTM_HIP_TRY(hipGetLastError());
    return 0;
  }
  const dim3 grid(nblk / 2, count);
  const int rpl = (n + kLanesPerPair - 1) / kLanesPerPair;
  SvdArgs arg = a;
  int cnt = count;
  void* args[] = {&arg, &cnt};
  const void* fn = rpl <= 6    ? (const void*)svd_sweeps<6>
                   : rpl <= 8  ? (const void*)svd_sweeps<8>
                   : rpl <= 10 ? (const void*)svd_sweeps<10>
                               : (const void*)svd_sweeps<12>;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  (void)hipStreamIsCapturing(s, &cs);
  if (cs == hipStreamCaptureStatusNone &&
      hipLaunchCooperativeKernel(fn, grid, dim3(256), args, 0, s) == hipSuccess)
    return 0;
  (void)hipGetLastError();
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep)
    for (int round = 0; round < nblk - 1; ++round) {
      if (rpl <= 6)
        svd_block_round<6><<<grid, 256, 0, s>>>(a, sweep, round);
      else if (rpl <= 8)
        svd_block_round<8><<<grid, 256, 0, s>>>(a, sweep, round);
      else if (rpl <= 10)
        svd_block_round<10><<<grid, 256, 0, s>>>(a, sweep, round);
      else
        svd_block_round<12><<<grid, 256, 0, s>>>(a, sweep, round);
    }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

size_t svd_workspace_bytes(int count, int n) {
  const size_t nn = (size_t)n * n;
  return (size_t)count * (2 * nn + 5 * nn) * sizeof(double) +
         (size_t)count * (kMaxSweeps + n) * sizeof(int) + (size_t)count * sizeof(double) +
         std::max(qr_workspace_bytes(count, n, n), qr_ordered_workspace_bytes(count, n, n)) + 4096;
}

int launch_svd(int count, const double* const* A, double* const* U, double* const* S,
               double* const* V, int n, void* ws, hipStream_t s, bool ordered) {
  if (count <= 0 || n <= 0) return 0;
  if (count > kMaxProb || n > kSvdMaxN) {
    set_thread_error("launch_svd: n <= 192 and at most 8 matrices per launch");
    return 1;
  }
  const size_t nn = (size_t)n * n;
  double* base = (double*)ws;
  SvdArgs a{};
  a.n = n;
  a.work = base;                                   // 2 nn per matrix
  double* wp = a.work + (size_t)count * 2 * nn;    // A P -> Q
  double* wc = wp + (size_t)count * nn;            // A P
  double* rt = wc + (size_t)count * nn;            // R^T
  double* ut = rt + (size_t)count * nn;            // left vectors of R^T
  double* vp = ut + (size_t)count * nn;            // right vectors of R^T
  a.flags = (int*)(vp + (size_t)count * nn);
  a.perm = a.flags + (size_t)count * kMaxSweeps;
  a.fro2 = (double*)(((uintptr_t)(a.perm + (size_t)count * n) + 7) & ~(uintptr_t)7);
  char* qws = (char*)(a.fro2 + count);
  qws = (char*)(((uintptr_t)qws + 255) & ~(uintptr_t)255);
  int nblk = (n + kBlk - 1) / kBlk;
  nblk += nblk & 1;
  if (nblk < 2) nblk = 2;
  a.nblk = nblk;
  const bool want_u = U != nullptr, want_vout = V != nullptr;
  a.want_v = want_u ? 1 : 0;                       // V' is needed for u = Q V'
  double* qptr[kMaxProb];
  for (int i = 0; i < count; ++i) {
    a.Ain[i] = A[i];
    a.Wp[i] = wp + i * nn;
    a.Wc[i] = wc + i * nn;
    a.A[i] = rt + i * nn;
    a.Ut[i] = ut + i * nn;
    a.U[i] = want_vout ? a.Ut[i] : nullptr;
    a.S[i] = S[i];
    a.V[i] = want_u ? vp + i * nn : nullptr;
    qptr[i] = a.Wp[i];
  }
  svd_prep<<<count, 256, 0, s>>>(a);
  CTM_HIP_TRY(hipGetLastError());
  svd_prep_copy<<<dim3(std::max(1, std::min(64, n * n / 256)), count), 256, 0, s>>>(a);
  CTM_HIP_TRY(hipGetLastError());
  int r = ordered ? launch_qr_ordered(count, qptr, n, n, qws, s) : launch_qr(count, qptr, n, n, qws, s);
  if (r) return r;
  auto product = [&](const GemmBatch& x) {
    return ordered ? launch_gemm_ordered(x, nullptr, 0, s) : launch_gemm(x, DT::F64, DT::F64, DT::F64, s);
  };
  // R^T = (A P)^T Q
  GemmBatch g{};
  g.count = count;
  g.M = g.N = g.K = n;
  g.lda = g.ldb = n;
  gemm_set_rowmajor_c(g, n);
  g.nbatch = 1;
  g.alpha = 1.0;
  for (int i = 0; i < count; ++i) {
    g.A[i] = a.Wc[i];
    g.transA[i] = 1;
    g.B[i] = a.Wp[i];
    g.C[i] = rt + i * nn;
  }
  r = product(g);
  if (r) return r;
  if (!ordered && small_svd_fits(n, want_u)) {
    if (want_u) launch_small_svd<true>(a, count, s);
    else launch_small_svd<false>(a, count, s);
    CTM_HIP_TRY(hipGetLastError());
  } else {
    svd_init<<<dim3(std::max(1, std::min(64, n * n / 256)), count), 256, 0, s>>>(a);
    CTM_HIP_TRY(hipGetLastError());
    const int r2 = launch_block_svd(a, count, s);
    if (r2) return r2;
  }
  svd_finalize<<<count, 1024, 0, s>>>(a);
  CTM_HIP_TRY(hipGetLastError());
  if (want_u) {   // u = Q V'
    for (int i = 0; i < count; ++i) {
      g.A[i] = a.Wp[i];
      g.transA[i] = 0;
      g.B[i] = vp + i * nn;
      g.C[i] = U[i];
    }
    r = product(g);
    if (r) return r;
  }
  if (want_vout) {   // v = P Ut
    for (int i = 0; i < count; ++i) a.V[i] = V[i];
    svd_unpermute_rows<<<dim3(std::max(1, std::min(64, n * n / 256)), count), 256, 0, s>>>(a);
    CTM_HIP_TRY(hipGetLastError());
  }
  return 0;
}

}  // namespace sictm
