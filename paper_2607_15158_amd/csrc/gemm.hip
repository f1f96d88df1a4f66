// Batched, index-mapped GEMM on the gfx950 matrix cores.
//
// Every contraction of a CTMRG move -- the enlarged-corner build, the
// applications of the enlarged corners to the N x k isometry blocks, the
// reduced matrix rho, the projector products and the renormalisation of C
// and T (Fig. 1; QR-based projector section) -- is one launch of this kernel
// family.  Leg permutations are folded into the operand strides and into the
// two-level output map, so no tensor is ever transposed in memory.
//
// Design: 256-thread workgroups (4 wavefronts of 64), one BM x BN output tile
// per workgroup, K staged through LDS in BK slices with a register prefetch
// of the next slice.  Wavefronts own (BM/WGM) x (BN/WGN) sub-tiles built
// from 16x16 MFMA blocks:
//   float64: v_mfma_f64_16x16x4_f64  (A: lane -> (row l%16, k l/16))
//   float32: v_mfma_f32_16x16x4_f32  (same operand layout)
//   bf16   : v_mfma_f32_16x16x32_bf16 (A: lane -> (row l%16, k 8*(l/16)..+7))
// and accumulate in float64 (f64 inputs) or float32 (f32/bf16 inputs).
// Result element r = 0..3 of lane l lies in column l%16 and in row
// l/16 + 4r for the float64 instruction, row 4(l/16) + r for the others
// (both measured on gfx950).
// Workgroup ids are remapped so that consecutive tiles share an XCD (and its
// L2), since the hardware deals consecutive workgroups round-robin to the 8
// XCDs.

#include "common.h"

#include <algorithm>
#include <cmath>

namespace sictm {
namespace {

template <typename Dst, typename Src>
__device__ __forceinline__ Dst cvt(Src x) { return (Dst)x; }
template <>
__device__ __forceinline__ __bf16 cvt<__bf16, double>(double x) { return (__bf16)(float)x; }
template <>
__device__ __forceinline__ __bf16 cvt<__bf16, float>(float x) { return (__bf16)x; }

__device__ __forceinline__ int xcd_remap(int bid, int nb) {
  const int xcd = bid & 7, idx = bid >> 3;
  const int per = nb >> 3, rem = nb & 7;
  return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

__device__ __forceinline__ long map2(int i, int div, long s1, long s0) {
  return (long)(i / div) * s1 + (long)(i % div) * s0;
}

// ---------------------------------------------------------------------------
// 16x16x4 path (float64 or float32 compute type CT).
// ---------------------------------------------------------------------------
template <typename CT> struct Mfma4;
template <> struct Mfma4<double> {
  using acc_t = v4d;
  static __device__ __forceinline__ acc_t op(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct Mfma4<float> {
  using acc_t = v4f;
  static __device__ __forceinline__ acc_t op(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kK4BK = 16, kK4Pad = 2;

// One BM x BN output tile (tm, tn) of problem `prob`, inner batch `batch`.
// The K loop runs in ascending 16-wide slices whatever the tile shape, so an
// output element gets the same bits from every tile shape and grid.  The
// slices are double-buffered in LDS: the global loads of slice kt + 1 are in
// flight while slice kt is multiplied, then stored into the other buffer,
// one barrier per slice.
template <typename TA, typename TB, typename TC, typename CT, int BM, int BN, int WGM, int WGN>
__device__ __forceinline__ void k4_tile(const GemmBatch& g, int prob, int batch, int tm, int tn,
                                        CT (*As)[kK4BK][BM + kK4Pad],
                                        CT (*Bs)[kK4BK][BN + kK4Pad]) {
  constexpr int BK = kK4BK;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 16, NI = WTN / 16;
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;
  static_assert(WGM * WGN == 4, "four wavefronts");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "wave tile multiple of 16");
  static_assert((BM * BK) % 256 == 0 && (BN * BK) % 256 == 0, "tile loads");
  using Acc = typename Mfma4<CT>::acc_t;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int m0 = tm * BM, n0 = tn * BN;
  const int M = g.M, N = g.N, K = g.K;
  const int trans = g.transA[prob];
  const TA* A = (const TA*)g.A[prob] + (long)batch * g.a_bs;
  const TB* B = (const TB*)g.B[prob] + (long)batch * g.b_bs;
  TC* C = (TC*)g.C[prob] + (long)batch * g.c_bs;
  const long lda = g.lda, ldb = g.ldb;

  CT ra[EA], rb[EB];
  auto load_tiles = [&](int k0) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      const int gm = m0 + m, gk = k0 + kk;
      CT v = (CT)0;
      if (gm < M && gk < K) v = cvt<CT>(trans ? A[(long)gk * lda + gm] : A[(long)gm * lda + gk]);
      ra[e] = v;
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      const int n = i % BN, kk = i / BN;
      const int gn = n0 + n, gk = k0 + kk;
      CT v = (CT)0;
      if (gn < N && gk < K) v = cvt<CT>(B[(long)gk * ldb + gn]);
      rb[e] = v;
    }
  };
  auto store_tiles = [&](int buf) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      As[buf][kk][m] = ra[e];
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      Bs[buf][i / BN][i % BN] = rb[e];
    }
  };

  Acc acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = Acc{0, 0, 0, 0};

  const int nk = (K + BK - 1) / BK;
  load_tiles(0);
  store_tiles(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load_tiles((kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      CT a[MI], b[NI];
      const int kr = ks + (lane >> 4);
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = As[buf][kr][wm * WTM + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = Bs[buf][kr][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = Mfma4<CT>::op(a[i], b[j], acc[i][j]);
    }
    if (kt + 1 < nk) store_tiles(buf ^ 1);
    __syncthreads();
  }

  // epilogue: two-level output map
  long offn[NI];
  bool okn[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int n = n0 + wn * WTN + j * 16 + (lane & 15);
    okn[j] = n < N;
    offn[j] = okn[j] ? map2(n, g.cdiv_n, g.cs_n1, g.cs_n0) : 0;
  }
  const double alpha = g.alpha;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * WTM + i * 16 + Mfma4<CT>::row(lane, r);
      if (m >= M) continue;
      const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (!okn[j]) continue;
        TC* p = C + offm + offn[j];
        double v = alpha * (double)acc[i][j][r];
        if (g.accumulate) v += (double)*p;
        *p = cvt<TC>(v);
      }
    }
  }
}

template <typename TA, typename TB, typename TC, typename CT, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void gemm_k4(GemmBatch g, int tiles_m, int tiles_n) {
  __shared__ CT As[2][kK4BK][BM + kK4Pad];
  __shared__ CT Bs[2][kK4BK][BN + kK4Pad];
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int prob = blockIdx.y / g.nbatch, batch = blockIdx.y % g.nbatch;
  k4_tile<TA, TB, TC, CT, BM, BN, WGM, WGN>(g, prob, batch, tile / tiles_n, tile % tiles_n, As, Bs);
}

typedef double v2d __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Double-buffered tile as wide as B, for the float32
// contractions with long K (the site absorptions of the corners and of the
// edges' renormalisation, 20736 x 1296 x 1296 per corner at D = 6, and
// Zc = Ct P_l): operands of type TA / TB are rounded to float32 on their way
// into LDS and multiplied on v_mfma_f32_16x16x4f32 with float32
// accumulation (operand layout as the float64 instruction; result element r
// of lane l in row 4 (l / 16) + r).
// ---------------------------------------------------------------------------
template <int BM, int BK>
struct SkinnyAF {
  static constexpr int LT = BM + 16;
  static constexpr int LN = BK + 1;
  static constexpr int SIZE = (BK * LT > BM * LN) ? BK * LT : BM * LN;
};

template <typename TA, typename TB, typename TC, int BM, int BN, int WGM, int WGN, bool TRANS>
__device__ __forceinline__ void skinny_tile_f32(const GemmBatch& g, int tiles_m, int tiles_n,
                                                int lin, float (*As)[SkinnyAF<BM, 16>::SIZE],
                                                float (*Bs)[16][BN + 16]) {
  constexpr int BK = 16;
  using AL = SkinnyAF<BM, BK>;
  using VA2 = TA __attribute__((ext_vector_type(2)));
  using VB2 = TB __attribute__((ext_vector_type(2)));
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 16, NI = WTN / 16;
  constexpr int NT = 64 * WGM * WGN;
  constexpr int NA = BM * BK / 2, NB = BN * BK / 2;
  constexpr int VA = (NA + NT - 1) / NT, VB = (NB + NT - 1) / NT;
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "wave tile multiple of 16");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int per_prob = tiles_m * tiles_n;
  const int pb = lin / per_prob, tile = lin % per_prob;
  const int prob = pb / g.nbatch, batch = pb % g.nbatch;
  const int tn = tile % tiles_n, tm = tile / tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  const int M = g.M, N = g.N, K = g.K;
  const TA* A = (const TA*)g.A[prob] + (long)batch * g.a_bs;
  const TB* B = (const TB*)g.B[prob] + (long)batch * g.b_bs;
  TC* C = (TC*)g.C[prob] + (long)batch * g.c_bs;
  const long lda = g.lda, ldb = g.ldb;

  VA2 ra[VA];
  VB2 rb[VB];
  auto load = [&](int k0) {
#pragma unroll
    for (int e = 0; e < VA; ++e) {
      const int i = tid + e * NT;
      VA2 v = {(TA)0, (TA)0};
      if (i < NA) {
        if (TRANS) {
          const int gk = k0 + i / (BM / 2), gm = m0 + 2 * (i % (BM / 2));
          if (gk < K) {
            const TA* p = A + (long)gk * lda + gm;
            if (gm + 1 < M) v = *(const VA2*)p;
            else if (gm < M) v.x = p[0];
          }
        } else {
          const int gm = m0 + i / (BK / 2), gk = k0 + 2 * (i % (BK / 2));
          if (gm < M) {
            const TA* p = A + (long)gm * lda + gk;
            if (gk + 1 < K) v = *(const VA2*)p;
            else if (gk < K) v.x = p[0];
          }
        }
      }
      ra[e] = v;
    }
#pragma unroll
    for (int e = 0; e < VB; ++e) {
      const int i = tid + e * NT;
      const int gk = k0 + i / (BN / 2), gn = n0 + 2 * (i % (BN / 2));
      VB2 v = {(TB)0, (TB)0};
      if (i < NB && gk < K) {
        const TB* p = B + (long)gk * ldb + gn;
        if (gn + 1 < N) v = *(const VB2*)p;
        else if (gn < N) v.x = p[0];
      }
      rb[e] = v;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < VA; ++e) {
      const int i = tid + e * NT;
      if (i < NA) {
        if (TRANS) {
          const int kk = i / (BM / 2), m = 2 * (i % (BM / 2));
          As[buf][kk * AL::LT + m] = (float)ra[e].x;
          As[buf][kk * AL::LT + m + 1] = (float)ra[e].y;
        } else {
          const int m = i / (BK / 2), kk = 2 * (i % (BK / 2));
          As[buf][m * AL::LN + kk] = (float)ra[e].x;
          As[buf][m * AL::LN + kk + 1] = (float)ra[e].y;
        }
      }
    }
#pragma unroll
    for (int e = 0; e < VB; ++e) {
      const int i = tid + e * NT;
      if (i < NB) {
        Bs[buf][i / (BN / 2)][2 * (i % (BN / 2))] = (float)rb[e].x;
        Bs[buf][i / (BN / 2)][2 * (i % (BN / 2)) + 1] = (float)rb[e].y;
      }
    }
  };

  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  const int nk = (K + BK - 1) / BK;
  load(0);
  store(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load((kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      float a[MI], b[NI];
      const int kr = ks + (lane >> 4);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int m = wm * WTM + i * 16 + (lane & 15);
        a[i] = TRANS ? As[buf][kr * AL::LT + m] : As[buf][m * AL::LN + kr];
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = Bs[buf][kr][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) store(buf ^ 1);
    __syncthreads();
  }

  long offn[NI];
  bool okn[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int n = n0 + wn * WTN + j * 16 + (lane & 15);
    okn[j] = n < N;
    offn[j] = okn[j] ? map2(n, g.cdiv_n, g.cs_n1, g.cs_n0) : 0;
  }
  const double alpha = g.alpha;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * WTM + i * 16 + 4 * (lane >> 4) + r;
      if (m >= M) continue;
      const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (!okn[j]) continue;
        TC* p = C + offm + offn[j];
        double v = alpha * (double)acc[i][j][r];
        if (g.accumulate) v += (double)*p;
        *p = cvt<TC>(v);
      }
    }
  }
}

template <typename TA, typename TB, typename TC, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN, 512 / (64 * WGM * WGN)) void gemm_skinny_f32x(
    GemmBatch g, int tiles_m, int tiles_n) {
  __shared__ float As[2][SkinnyAF<BM, 16>::SIZE];
  __shared__ float Bs[2][16][BN + 16];
  const int per_prob = tiles_m * tiles_n;
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int prob = lin / per_prob / g.nbatch;
  if (g.transA[prob])
    skinny_tile_f32<TA, TB, TC, BM, BN, WGM, WGN, true>(g, tiles_m, tiles_n, lin, As, Bs);
  else
    skinny_tile_f32<TA, TB, TC, BM, BN, WGM, WGN, false>(g, tiles_m, tiles_n, lin, As, Bs);
}

// ---------------------------------------------------------------------------
// Split products (stream-K style): C = op(A) B with long K.  A launch of one
// tile per workgroup leaves CUs idle or half loaded when the tiles do not fill
// the chip evenly.  Here one workgroup of 8 wavefronts per CU takes an equal, contiguous range of the (tile,
// 16-wide K slice) space.  A tile inside one range is written directly; a
// tile cut by range boundaries leaves partial tiles in scratch (slot 2w for
// the segment that starts range w, 2w+1 for the one that ends it), which a
// second kernel sums in workgroup order, so results do not depend on timing.
// ---------------------------------------------------------------------------
struct StreamK {
  int nslices;    // BK-slices of K per tile
  int tiles_m, tiles_n;
  int nwg;        // workgroups (ranges) of the main kernel
  int per, rem;   // units per range; the first `rem` ranges have one more
  int unit;       // slices per unit: 1, or nslices where no tile is cut
  int total;      // ordered sums: all slices, whose range w begins at w total / nwg; else 0
  double* part;   // 2 * nwg partial BM x BN tiles (row-major)
};

__device__ __forceinline__ int sk_begin(int w, const StreamK& sk) {
  if (sk.total) return (int)((long)w * sk.total / sk.nwg);
  return (w * sk.per + min(w, sk.rem)) * sk.unit;
}

__device__ __forceinline__ int sk_owner(int p, const StreamK& sk) {
  if (sk.total) return (int)(((long)(p + 1) * sk.nwg - 1) / sk.total);   // the last w with w total / nwg <= p
  p /= sk.unit;
  const int wide = sk.rem * (sk.per + 1);
  return p < wide ? p / (sk.per + 1) : sk.rem + (p - wide) / sk.per;
}

// Two adjacent doubles by one 16-byte load; global loads need no more than
// the 8-byte alignment every double has (odd leading dimensions included).
typedef double v2du __attribute__((ext_vector_type(2), aligned(8)));

// The 8 wavefronts stand WM x WN; each owns MI x NI blocks of 16 x 16.  The
// rows of a wavefront are its own, so its elements of A go from global
// memory straight into the operand registers of the matrix instruction (of a
// 16-wide slice lane l takes k = 2 (l / 16), + 1, + 8 and + 9 of row l % 16,
// one for each of the slice's four instructions, which multiply them with
// the same rows of B: the order of the sum within a slice is free) and only
// B, which all share, is staged in LDS, one barrier per slice.  Loads run a
// slice (A) and two slices (B) ahead and stand between the matrix
// instructions of a slice, so that their issue and the LDS stores hide in
// the 64 cycles each of those takes.
// Rows and columns past the edge are read from clamped addresses and never
// stored; the last slice of K, when it is not full, is filled up with zeros.
//
// Bound by the f64 matrix cores.  8 products of 5184 x 5184 x 160: 1.185 ms
// with A staged in LDS beside B, loads under per-element bounds checks at the
// slice's start and the LDS stores at its end (matrix cores busy 73%), now
// 1.065 ms (82%; 1.0 ms with no loads at all).  8 of 1024 x 1024 x 72:
// 68 -> 39 us; 8 of 1875 x 1875 x 87 (odd rows, which took one-tile kernels
// before): 328 -> 127 us; 6 of 2500 x 2500 x 105: 210 -> 156 us.
//
// SEQ: the matrix instructions take k in ascending order, four adjacent ones
// each, so that a sum within a range has the bits of the tile kernels' (ordered
// products, below).  A is then read 8 bytes at a time: four of 2500 x 105 x 2500
// take 164 us on 192 x 128, where 256 x 112 with 16-byte loads takes 105.
template <int MI, int NI, int WN, bool SEQ>
struct SkTile {
  static constexpr int WM = 8 / WN;
  static constexpr int BM = 16 * MI * WM, BN = 16 * NI * WN;
  static constexpr int BK = 16, NT = 512;
  static constexpr int LB = BN + (SEQ ? 16 : 8);   // B rows in LDS: the rows of two lanes fall 32 banks apart
  static constexpr int NB = BN * BK / 2;              // 16-byte loads of B per slice
  static constexpr int VB = (NB + NT - 1) / NT;
  // k of matrix instruction t, beyond the lane's first
  static constexpr int kof(int t) { return SEQ ? 4 * t : 8 * (t >> 1) + (t & 1); }
  static __device__ __forceinline__ int kfirst(int lk) { return SEQ ? lk : 2 * lk; }
};

// acc += op(A)[m0 .. m0+BM) x B[.. n0 .. n0+BN) over the K slices [s0, s1) of
// problem prob (n0 < N, even).
// ONE: N == 1 (B has no pairs of columns).
template <int MI, int NI, int WN, bool TRANS, bool ONE, bool SEQ>
__device__ __forceinline__ void sk_segment(const GemmBatch& g, int prob, int batch, int m0, int n0, int s0, int s1,
                                           double (*Bs)[16][SkTile<MI, NI, WN, SEQ>::LB],
                                           v4d (&acc)[MI][NI]) {
  using S = SkTile<MI, NI, WN, SEQ>;
  constexpr int BK = S::BK;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int M = g.M, N = g.N, K = g.K;
  const long lda = g.lda, ldb = g.ldb;
  const double* A = (const double*)g.A[prob] + (long)batch * g.a_bs;
  const double* B = (const double*)g.B[prob] + (long)batch * g.b_bs;
  const int full = K / BK;   // slices before the partial one
  const int sf = min(s1, full);

  // A: this lane's rows at its first k of the slice the next load takes
  const double* pa[MI];
  const long astep = TRANS ? BK * lda : BK;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const long m = min(m0 + (wm * MI + i) * 16 + li, M - 1);
    const long k = s0 * BK + S::kfirst(lk);
    pa[i] = TRANS ? A + k * lda + m : A + m * lda + k;
  }
  auto load_a = [&](double (&ra)[MI][4]) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (TRANS || SEQ) {
#pragma unroll
        for (int t = 0; t < 4; ++t) ra[i][t] = pa[i][S::kof(t) * (TRANS ? lda : 1)];
      } else {
        const v2du v0 = *(const v2du*)pa[i], v1 = *(const v2du*)(pa[i] + S::kof(2));
        ra[i][0] = v0.x;
        ra[i][1] = v0.y;
        ra[i][2] = v1.x;
        ra[i][3] = v1.y;
      }
      pa[i] += astep;
    }
  };
  auto load_a_last = [&](double (&ra)[MI][4]) {   // the partial slice
    const int k = full * BK + S::kfirst(lk);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        ra[i][t] = k + S::kof(t) < K ? pa[i][S::kof(t) * (TRANS ? lda : 1)] : 0.0;
  };
  // B: pair e of this thread in row kb of a slice (threads beyond the slice's
  // pairs repeat its last one); the last column of an odd N is read as the
  // second of its pair
  const double* pb[S::VB];
  int kb[S::VB], lb[S::VB];
  bool second[S::VB];
#pragma unroll
  for (int e = 0; e < S::VB; ++e) {
    const int i = min(tid + e * S::NT, S::NB - 1);
    const int kk = i / (S::BN / 2), nl = 2 * (i % (S::BN / 2)), n = n0 + nl;
    second[e] = !ONE && n + 1 == N;
    pb[e] = B + (long)(s0 * BK + kk) * ldb + (n + 1 < N ? n : second[e] ? n - 1 : ONE ? 0 : N - 2);
    kb[e] = kk;
    lb[e] = kk * S::LB + nl;
  }
  const long bstep = BK * ldb;
  auto ld_b = [&](const double* q) {
    v2du v;
    if (ONE)
      v.x = v.y = *q;
    else
      v = *(const v2du*)q;
    return v;
  };
  auto load_b = [&](v2du (&rb)[S::VB]) {
#pragma unroll
    for (int e = 0; e < S::VB; ++e) {
      rb[e] = ld_b(pb[e]);
      pb[e] += bstep;
    }
  };
  auto load_b_last = [&](v2du (&rb)[S::VB]) {
#pragma unroll
    for (int e = 0; e < S::VB; ++e) {
      rb[e].x = rb[e].y = 0.0;
      if (full * BK + kb[e] < K) rb[e] = ld_b(pb[e]);
    }
  };
  auto store_b = [&](int buf, const v2du (&rb)[S::VB]) {
    double* base = &Bs[buf][0][0];
#pragma unroll
    for (int e = 0; e < S::VB; ++e) {
      v2d v;
      v.x = second[e] ? rb[e].y : rb[e].x;
      v.y = rb[e].y;
      *(v2d*)(base + lb[e]) = v;
    }
  };
  double ra[MI][4], rn[MI][4];
  v2du rb[S::VB];
  auto mul = [&](int buf, int t) {
    const double* bp = &Bs[buf][S::kof(t) + S::kfirst(lk)][wn * NI * 16 + li];
    double b[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) b[j] = bp[16 * j];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[i][t], b[j], acc[i][j], 0, 0, 0);
  };
  auto advance = [&]() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) ra[i][t] = rn[i][t];
  };

  if (s0 < full) {
    load_b(rb);
    load_a(ra);
  } else {
    load_b_last(rb);
    load_a_last(ra);
  }
  store_b(0, rb);
  if (s0 + 1 < s1) {
    if (s0 + 1 < full) load_b(rb);
    else load_b_last(rb);
  }
  // nothing is in flight where the loop begins: its waits are then only those
  // of its own loads, in their order
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  __syncthreads();
  int s = s0, buf = 0;
  for (; s + 2 < sf; ++s, buf ^= 1) {
    // matrix instructions and LDS reads may move across these marks, loads,
    // LDS stores and the waits they need may not
    mul(buf, 0);
    __builtin_amdgcn_sched_barrier(0x108);
    load_a(rn);
    mul(buf, 1);
    __builtin_amdgcn_sched_barrier(0x108);
    store_b(buf ^ 1, rb);
    load_b(rb);
    mul(buf, 2);
    __builtin_amdgcn_sched_barrier(0x108);
    mul(buf, 3);
    __syncthreads();
    advance();
  }
  for (; s < s1; ++s, buf ^= 1) {   // the last slices: what comes after may be partial or absent
    if (s + 1 < s1) {
      if (s + 1 < full) load_a(rn);
      else load_a_last(rn);
      store_b(buf ^ 1, rb);
    }
    if (s + 2 < s1) {
      if (s + 2 < full) load_b(rb);
      else load_b_last(rb);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) mul(buf, t);
    __syncthreads();
    advance();
  }
}

template <int MI, int NI, int WN, bool ONE, bool SEQ>
__global__ __launch_bounds__(512, 2) void gemm_streamk_f64(GemmBatch g, StreamK sk) {
  using S = SkTile<MI, NI, WN, SEQ>;
  constexpr int BM = S::BM, BN = S::BN;
  __shared__ __attribute__((aligned(16))) double Bs[2][16][S::LB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int begin = sk_begin(w, sk), end = sk_begin(w + 1, sk);
  const int M = g.M, N = g.N;
  // segments last to first: a range of L <= nslices slices then reads slice
  // t of its second tile, and later slice t + nslices - L of its first, at
  // step t, so the ranges sharing a problem (and an XCD) walk K in two
  // phases and reuse each B slice from L2
  int pend = end;
  while (pend > begin) {
    const int at = (pend - 1) / sk.nslices;
    const int pos = max(at * sk.nslices, begin);
    const int s0 = pos - at * sk.nslices, s1 = pend - at * sk.nslices;
    // cut tiles go down the rows first (ranges side by side share B).  Whole ones
    // are dealt out in turn along the columns, so that neighbouring columns are
    // worked on side by side: where the output map sends columns of different
    // tiles to one cache line, they meet in one L2 (four transposed 5184 x 5184 x
    // 144 with every 144th column adjacent: 3.25 ms in contiguous ranges, 1.34 so)
    const bool whole = sk.unit > 1;
    const int tile = whole ? (at - begin / sk.nslices) * sk.nwg + w : at;
    const int per = sk.tiles_m * sk.tiles_n, pb = tile / per, tt = tile % per;
    const int m0 = (whole ? tt / sk.tiles_n : tt % sk.tiles_m) * BM;
    const int n0 = (whole ? tt % sk.tiles_n : tt / sk.tiles_m) * BN;
    const int prob = pb / g.nbatch, batch = pb % g.nbatch;
    v4d acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = v4d{0, 0, 0, 0};
    if (g.transA[prob])
      sk_segment<MI, NI, WN, true, ONE, SEQ>(g, prob, batch, m0, n0, s0, s1, Bs, acc);
    else
      sk_segment<MI, NI, WN, false, ONE, SEQ>(g, prob, batch, m0, n0, s0, s1, Bs, acc);
    const int mw = wm * MI * 16 + (lane >> 4), nw = wn * NI * 16 + (lane & 15);
    if (s0 == 0 && s1 == sk.nslices) {
      // the whole tile: written here
      double* C = (double*)g.C[prob] + (long)batch * g.c_bs;
      long offn[NI];
      bool okn[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n = n0 + nw + j * 16;
        okn[j] = n < N;
        offn[j] = okn[j] ? map2(n, g.cdiv_n, g.cs_n1, g.cs_n0) : 0;
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + mw + i * 16 + 4 * r;
          if (m >= M) continue;
          const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            if (!okn[j]) continue;
            double* p = C + offm + offn[j];
            double v = g.alpha * acc[i][j][r];
            if (g.accumulate) v += *p;
            *p = v;
          }
        }
      }
    } else {
      // part of a tile: into the slot of this segment
      double* P = sk.part + (long)(2 * w + (pos == begin ? 0 : 1)) * (BM * BN) + mw * BN + nw;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < NI; ++j) P[(i * 16 + 4 * r) * BN + j * 16] = acc[i][j][r];
    }
    pend = pos;
  }
}

// Float32 form of the split SI application (contraction precision f32): the
// same ranges of (tile, K-slice) space as gemm_streamk_f64 over 192 x 160
// tiles, with A (the enlarged corner) in float32, B (the float64 block)
// rounded to float32 on its way into LDS, 32-wide slices (the bytes of the
// float64 kernel's 16) and v_mfma_f32_16x16x4f32 with float32 accumulation.
// Whole tiles are widened to float64 on store; cut tiles leave their partial
// sums in float64 in the same scratch slots, summed by gemm_streamk_fixup.
namespace skf32 {
constexpr int BM = 192, BN = 160, BK = 32, WGM = 4, WGN = 2, NT = 64 * WGM * WGN;
constexpr int WTM = BM / WGM, WTN = BN / WGN;   // 48 x 80 per wavefront
constexpr int MI = WTM / 16, NI = WTN / 16;     // 3 x 5 accumulator blocks
constexpr int LT = BM + 16;                     // transposed A in LDS: [k][m]
constexpr int LN = BK + 1;                      // plain A in LDS: [m][k]
constexpr int ASZ = (BK * LT > BM * LN) ? BK * LT : BM * LN;
constexpr int LB = BN + 16;                     // B in LDS: [k][n]
constexpr int NA = BM * BK / 4;                 // 16-byte loads of A per slice (4 floats)
constexpr int NB = BK * BN / 2;                 // 16-byte loads of B per slice (2 doubles)
constexpr int VA = (NA + NT - 1) / NT, VB = (NB + NT - 1) / NT;
}  // namespace skf32

template <bool TRANS>
__device__ __forceinline__ void sk_segment_f32(const GemmBatch& g, int prob, int m0, int s0, int s1,
                                               float (*As)[skf32::ASZ],
                                               float (*Bs)[skf32::BK][skf32::LB],
                                               v4f (&acc)[skf32::MI][skf32::NI]) {
  using namespace skf32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int M = g.M, N = g.N, K = g.K;
  const float* A = (const float*)g.A[prob];
  const double* B = (const double*)g.B[prob];
  const long lda = g.lda, ldb = g.ldb;
  v4f ra[VA];
  v2d rb[VB];
  auto load = [&](int k0) {
#pragma unroll
    for (int e = 0; e < VA; ++e) {
      const int i = tid + e * NT;
      v4f v = {0.f, 0.f, 0.f, 0.f};
      if (i < NA) {
        if (TRANS) {
          const int gk = k0 + i / (BM / 4), gm = m0 + 4 * (i % (BM / 4));
          if (gk < K) {
            const float* q = A + (long)gk * lda + gm;
            if (gm + 3 < M) {
              v = *(const v4f*)q;
            } else {
              if (gm < M) v.x = q[0];
              if (gm + 1 < M) v.y = q[1];
              if (gm + 2 < M) v.z = q[2];
            }
          }
        } else {
          const int gm = m0 + i / (BK / 4), gk = k0 + 4 * (i % (BK / 4));
          if (gm < M) {
            const float* q = A + (long)gm * lda + gk;
            if (gk + 3 < K) {
              v = *(const v4f*)q;
            } else {
              if (gk < K) v.x = q[0];
              if (gk + 1 < K) v.y = q[1];
              if (gk + 2 < K) v.z = q[2];
            }
          }
        }
      }
      ra[e] = v;
    }
#pragma unroll
    for (int e = 0; e < VB; ++e) {
      const int i = tid + e * NT;
      const int gk = k0 + i / (BN / 2), gn = 2 * (i % (BN / 2));
      v2d v = {0.0, 0.0};
      if (i < NB && gk < K) {
        const double* q = B + (long)gk * ldb + gn;
        if (gn + 1 < N) v = *(const v2d*)q;
        else if (gn < N) v.x = q[0];
      }
      rb[e] = v;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < VA; ++e) {
      const int i = tid + e * NT;
      if (i < NA) {
        if (TRANS) {
          const int kk = i / (BM / 4), m = 4 * (i % (BM / 4));
          *(v4f*)&As[buf][kk * LT + m] = ra[e];
        } else {
          const int m = i / (BK / 4), kk = 4 * (i % (BK / 4));
          float* q = &As[buf][m * LN + kk];
          q[0] = ra[e].x;
          q[1] = ra[e].y;
          q[2] = ra[e].z;
          q[3] = ra[e].w;
        }
      }
    }
#pragma unroll
    for (int e = 0; e < VB; ++e) {
      const int i = tid + e * NT;
      if (i < NB) {
        float* q = &Bs[buf][i / (BN / 2)][2 * (i % (BN / 2))];
        q[0] = (float)rb[e].x;
        q[1] = (float)rb[e].y;
      }
    }
  };
  load(s0 * BK);
  store(0);
  __syncthreads();
  for (int kt = s0; kt < s1; ++kt) {
    const int buf = (kt - s0) & 1;
    if (kt + 1 < s1) load((kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      float a[MI], b[NI];
      const int kr = ks + (lane >> 4);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int m = wm * WTM + i * 16 + (lane & 15);
        a[i] = TRANS ? As[buf][kr * LT + m] : As[buf][m * LN + kr];
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) b[j] = Bs[buf][kr][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < s1) store(buf ^ 1);
    __syncthreads();
  }
}

__global__ __launch_bounds__(skf32::NT, 1) void gemm_streamk_f32(GemmBatch g, StreamK sk) {
  using namespace skf32;
  __shared__ float As[2][ASZ];
  __shared__ float Bs[2][BK][LB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int begin = sk_begin(w, sk), end = sk_begin(w + 1, sk);
  const int M = g.M, N = g.N;
  // segments last to first, as in the float64 kernel
  int pend = end;
  while (pend > begin) {
    const int tile = (pend - 1) / sk.nslices;
    const int pos = max(tile * sk.nslices, begin);
    const int s0 = pos - tile * sk.nslices, s1 = pend - tile * sk.nslices;
    const int prob = tile / sk.tiles_m, m0 = (tile % sk.tiles_m) * BM;
    v4f acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    if (g.transA[prob])
      sk_segment_f32<true>(g, prob, m0, s0, s1, As, Bs, acc);
    else
      sk_segment_f32<false>(g, prob, m0, s0, s1, As, Bs, acc);
    // float32 MFMA result element r of lane l: row 4 (l / 16) + r, column l % 16
    if (s0 == 0 && s1 == sk.nslices) {
      double* C = (double*)g.C[prob];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm * WTM + i * 16 + 4 * (lane >> 4) + r;
          if (m >= M) continue;
          double* row = C + (long)m * g.cs_m0;
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const int n = wn * WTN + j * 16 + (lane & 15);
            if (n >= N) continue;
            double v = g.alpha * (double)acc[i][j][r];
            if (g.accumulate) v += row[n];
            row[n] = v;
          }
        }
      }
    } else {
      double* P = sk.part + (long)(2 * w + (pos == begin ? 0 : 1)) * (BM * BN);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ml = wm * WTM + i * 16 + 4 * (lane >> 4) + r;
#pragma unroll
          for (int j = 0; j < NI; ++j)
            P[ml * BN + wn * WTN + j * 16 + (lane & 15)] = (double)acc[i][j][r];
        }
    }
    pend = pos;
  }
}

// Sums the partial tiles of every tile cut by range boundaries, in
// workgroup order, and writes them through C's index map (alpha and
// accumulate as in the main kernel).  kFixRows-row strips of a tile per block
// of 256 threads, two adjacent columns per thread, four partials in flight.
// Ranges are never empty here (the split runs only with at least 8 slices
// per workgroup), so every workgroup between the first and the last owner of
// a tile left a partial in slot 2w.
constexpr int kFixRows = 8;

template <int BM, int BN>
__global__ __launch_bounds__(256) void gemm_streamk_fixup(GemmBatch g, StreamK sk) {
  static_assert(BM % kFixRows == 0 && BN % 2 == 0, "strip shape");
  const int tile = blockIdx.x / (BM / kFixRows);
  const int r0 = (blockIdx.x % (BM / kFixRows)) * kFixRows;
  const int t0 = tile * sk.nslices, t1 = t0 + sk.nslices;
  const int wf = sk_owner(t0, sk), wl = sk_owner(t1 - 1, sk);
  if (wf == wl) return;
  const int col = tile / sk.tiles_m, m0 = (tile % sk.tiles_m) * BM;
  const int pb = col / sk.tiles_n, n0 = (col % sk.tiles_n) * BN;
  const int first_slot = sk_begin(wf, sk) < t0 ? 2 * wf + 1 : 2 * wf;
  double* C = (double*)g.C[pb / g.nbatch] + (long)(pb % g.nbatch) * g.c_bs;
  constexpr int PR = BN / 2;   // column pairs per row
  for (int q = threadIdx.x; q < kFixRows * PR; q += 256) {
    const int ml = r0 + q / PR, nl = 2 * (q % PR), m = m0 + ml, n = n0 + nl;
    if (m >= g.M || n >= g.N) continue;
    const double* P = sk.part + (long)ml * BN + nl;
    v2d v = *(const v2d*)(P + (long)first_slot * (BM * BN));
    int w = wf + 1;
    for (; w + 3 <= wl; w += 4) {
      v2d x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = *(const v2d*)(P + (long)(2 * (w + i)) * (BM * BN));
#pragma unroll
      for (int i = 0; i < 4; ++i) v += x[i];
    }
    for (; w <= wl; ++w) v += *(const v2d*)(P + (long)(2 * w) * (BM * BN));
    const bool two = n + 1 < g.N;
    const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
    double* p0 = C + offm + map2(n, g.cdiv_n, g.cs_n1, g.cs_n0);
    double* p1 = two ? C + offm + map2(n + 1, g.cdiv_n, g.cs_n1, g.cs_n0) : p0;
    double o0 = g.alpha * v.x, o1 = g.alpha * v.y;
    if (g.accumulate) {
      o0 += *p0;
      if (two) o1 += *p1;
    }
    *p0 = o0;
    if (two) *p1 = o1;
  }
}

// ---------------------------------------------------------------------------
// Small products: a workgroup of 8 wavefronts owns 16 rows and 16 NT columns
// and splits K over the wavefronts (wavefront w takes the 16-wide slices w,
// w + 8, ...), each with its operands straight from global memory to the
// matrix cores' registers; the 8 partial tiles are summed in LDS in wavefront
// order.  A product whose tiles do not fill the chip is bound by the latency
// of one tile's walk over K, which this cuts to an eighth, in one launch.  The
// bits depend on K alone, not on NT or the grid.
// ---------------------------------------------------------------------------
template <int NT>
struct ShortTile {
  static constexpr int LD = 16 * (NT | 1);   // two rows fall 32 banks apart
  double red[8][16][LD];
};

template <int NT, bool TRANS>
__device__ __forceinline__ void short_tile(const GemmBatch& g, int prob, int tm, int tn, ShortTile<NT>& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int M = g.M, N = g.N, K = g.K, m0 = tm * 16, n0 = tn * 16 * NT;
  const long lda = g.lda, ldb = g.ldb;
  const int m = min(m0 + li, M - 1);
  const double* A = (const double*)g.A[prob] + (TRANS ? (long)m : (long)m * lda);
  const double* B = (const double*)g.B[prob];
  int nc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) nc[j] = min(n0 + 16 * j + li, N - 1);
  const int ns = (K + 15) >> 4, full = K >> 4;
  // k of matrix instruction t of a slice: 2 lk + {0, 1, 8, 9}
  auto load = [&](int s, double (&a)[4], double (&b)[4][NT]) {
    const int k = 16 * s + 2 * lk;
    if (s < full) {
      if (TRANS) {
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = A[(long)(k + 8 * (t >> 1) + (t & 1)) * lda];
      } else {
        const v2du x = *(const v2du*)(A + k), y = *(const v2du*)(A + k + 8);
        a[0] = x.x;
        a[1] = x.y;
        a[2] = y.x;
        a[3] = y.y;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) b[t][j] = B[(long)(k + 8 * (t >> 1) + (t & 1)) * ldb + nc[j]];
    } else {   // the partial slice
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int kk = k + 8 * (t >> 1) + (t & 1);
        const bool in = kk < K;
        a[t] = in ? A[TRANS ? (long)kk * lda : (long)kk] : 0.0;
#pragma unroll
        for (int j = 0; j < NT; ++j) b[t][j] = in ? B[(long)kk * ldb + nc[j]] : 0.0;
      }
    }
  };
  v4d acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = v4d{0, 0, 0, 0};
  double a[2][4], b[2][4][NT];
  auto mul = [&](const double (&x)[4], const double (&y)[4][NT]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t], y[t][j], acc[j], 0, 0, 0);
  };
  int s = wave;
  if (s < ns) load(s, a[0], b[0]);
  for (; s < ns; s += 16) {
    if (s + 8 < ns) load(s + 8, a[1], b[1]);
    mul(a[0], b[0]);
    if (s + 8 >= ns) break;
    if (s + 16 < ns) load(s + 16, a[0], b[0]);
    mul(a[1], b[1]);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.red[wave][lk + 4 * r][16 * j + li] = acc[j][r];
  __syncthreads();
  double* C = (double*)g.C[prob];
  for (int i = tid; i < 256 * NT; i += 512) {
    const int r = i / (16 * NT), c = i % (16 * NT), mm = m0 + r, n = n0 + c;
    if (mm >= M || n >= N) continue;
    double v = sh.red[0][r][c];
#pragma unroll
    for (int w = 1; w < 8; ++w) v += sh.red[w][r][c];
    v *= g.alpha;
    double* q = C + map2(mm, g.cdiv_m, g.cs_m1, g.cs_m0) + map2(n, g.cdiv_n, g.cs_n1, g.cs_n0);
    *q = g.accumulate ? v + *q : v;
  }
}

template <int NT>
__global__ __launch_bounds__(512, 2) void gemm_short_f64(GemmBatch g, int tiles_m, int tiles_n) {
  __shared__ ShortTile<NT> sh;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int per = tiles_m * tiles_n, prob = w / per, t = w % per;
  if (g.transA[prob])
    short_tile<NT, true>(g, prob, t / tiles_n, t % tiles_n, sh);
  else
    short_tile<NT, false>(g, prob, t / tiles_n, t % tiles_n, sh);
}

// ---------------------------------------------------------------------------
// Grouped launches: the products of several GemmBatch descriptors of
// different shapes (one per context of a batched move) in one persistent
// launch.  The descriptors sit in device memory with the prefix sums of
// their work items (tiles x problems x inner batches); workgroup w takes
// items w, w + grid, ... and finds each one's descriptor by binary search.
// Every item runs the tile code of the ungrouped kernels, whose results do
// not depend on the grid, so a grouped product equals the same product
// launched alone, bit for bit.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int group_of(const GroupItem* items, int n, long w) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].first <= w) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int NT>
__global__ __launch_bounds__(512, 2) void gemm_short_grouped(const GroupItem* items, int nitems, long total) {
  __shared__ ShortTile<NT> sh;
  for (long w = blockIdx.x; w < total; w += gridDim.x) {
    const GroupItem& it = items[group_of(items, nitems, w)];
    const int lin = (int)(w - it.first), per = it.tiles_m * it.tiles_n;
    const int prob = lin / per, t = lin % per;
    if (it.g.transA[prob])
      short_tile<NT, true>(it.g, prob, t / it.tiles_n, t % it.tiles_n, sh);
    else
      short_tile<NT, false>(it.g, prob, t / it.tiles_n, t % it.tiles_n, sh);
    __syncthreads();   // the sums are read before the next item overwrites them
  }
}

template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void gemm_k4_grouped(const GroupItem* items, int nitems,
                                                       long total) {
  __shared__ double As[2][kK4BK][BM + kK4Pad];
  __shared__ double Bs[2][kK4BK][BN + kK4Pad];
  for (long w = blockIdx.x; w < total; w += gridDim.x) {
    const GroupItem& it = items[group_of(items, nitems, w)];
    const int lin = (int)(w - it.first);
    const int per = it.tiles_m * it.tiles_n;
    const int pb = lin / per, tile = lin % per;
    k4_tile<double, double, double, double, BM, BN, WGM, WGN>(
        it.g, pb / it.g.nbatch, pb % it.g.nbatch, tile / it.tiles_n, tile % it.tiles_n, As, Bs);
  }
}

// ---------------------------------------------------------------------------
// bf16 path: v_mfma_f32_16x16x32_bf16, float32 accumulation.
// LDS keeps k contiguous per row so that a lane reads its 8 k-values at once.
// ---------------------------------------------------------------------------
template <typename TA, typename TB, typename TC, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void gemm_bf16(GemmBatch g, int tiles_m, int tiles_n) {
  constexpr int BK = 32;
  constexpr int PAD = 8;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 16, NI = WTN / 16;
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;
  static_assert(WGM * WGN == 4, "four wavefronts");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "wave tile multiple of 16");

  __shared__ __attribute__((aligned(16))) __bf16 As[BM][BK + PAD];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[BN][BK + PAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int tn = tile % tiles_n, tm = tile / tiles_n;
  const int prob = blockIdx.y / g.nbatch, batch = blockIdx.y % g.nbatch;
  const int m0 = tm * BM, n0 = tn * BN;
  const int M = g.M, N = g.N, K = g.K;
  const int trans = g.transA[prob];
  const TA* A = (const TA*)g.A[prob] + (long)batch * g.a_bs;
  const TB* B = (const TB*)g.B[prob] + (long)batch * g.b_bs;
  TC* C = (TC*)g.C[prob] + (long)batch * g.c_bs;
  const long lda = g.lda, ldb = g.ldb;

  __bf16 ra[EA], rb[EB];
  auto load_tiles = [&](int k0) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      const int gm = m0 + m, gk = k0 + kk;
      __bf16 v = (__bf16)0.0f;
      if (gm < M && gk < K)
        v = cvt<__bf16>(trans ? A[(long)gk * lda + gm] : A[(long)gm * lda + gk]);
      ra[e] = v;
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      const int n = i % BN, kk = i / BN;
      const int gn = n0 + n, gk = k0 + kk;
      __bf16 v = (__bf16)0.0f;
      if (gn < N && gk < K) v = cvt<__bf16>(B[(long)gk * ldb + gn]);
      rb[e] = v;
    }
  };
  auto store_tiles = [&]() {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      As[m][kk] = ra[e];
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      Bs[i % BN][i / BN] = rb[e];
    }
  };

  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0, 0, 0, 0};

  const int nk = (K + BK - 1) / BK;
  load_tiles(0);
  for (int kt = 0; kt < nk; ++kt) {
    store_tiles();
    __syncthreads();
    if (kt + 1 < nk) load_tiles((kt + 1) * BK);
    const int kc = 8 * (lane >> 4);
    v8bf a[MI], b[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
      a[i] = *reinterpret_cast<const v8bf*>(&As[wm * WTM + i * 16 + (lane & 15)][kc]);
#pragma unroll
    for (int j = 0; j < NI; ++j)
      b[j] = *reinterpret_cast<const v8bf*>(&Bs[wn * WTN + j * 16 + (lane & 15)][kc]);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  }

  long offn[NI];
  bool okn[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int n = n0 + wn * WTN + j * 16 + (lane & 15);
    okn[j] = n < N;
    offn[j] = okn[j] ? map2(n, g.cdiv_n, g.cs_n1, g.cs_n0) : 0;
  }
  const float alpha = (float)g.alpha;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * WTM + i * 16 + 4 * (lane >> 4) + r;
      if (m >= M) continue;
      const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (!okn[j]) continue;
        TC* p = C + offm + offn[j];
        float v = alpha * acc[i][j][r];
        if (g.accumulate) v += (float)*p;
        *p = cvt<TC>(v);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Split bfloat16 path (three bf16 products per step): every operand value x
// is rounded to float32 and written as hi + lo with hi = bf16(x) and
// lo = bf16(x - hi) (16 significant bits together); A B is then
// A_hi B_hi + A_hi B_lo + A_lo B_hi on v_mfma_f32_16x16x32_bf16 with float32
// accumulation, dropping only A_lo B_lo (relative 2^-16).  This keeps the
// bf16 matrix-core rate at close to float32 accuracy (Henry, Tang and
// Heinecke, ARITH 2019).  Same LDS layout as the bf16 path, hi and lo
// halves side by side.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

template <typename TA, typename TB, typename TC, int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void gemm_bf16x3(GemmBatch g, int tiles_m, int tiles_n) {
  constexpr int BK = 32;
  constexpr int PAD = 8;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 16, NI = WTN / 16;
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;
  static_assert(WGM * WGN == 4, "four wavefronts");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0, "wave tile multiple of 16");

  __shared__ __attribute__((aligned(16))) __bf16 Ah[BM][BK + PAD];
  __shared__ __attribute__((aligned(16))) __bf16 Al[BM][BK + PAD];
  __shared__ __attribute__((aligned(16))) __bf16 Bh[BN][BK + PAD];
  __shared__ __attribute__((aligned(16))) __bf16 Bl[BN][BK + PAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int tn = tile % tiles_n, tm = tile / tiles_n;
  const int prob = blockIdx.y / g.nbatch, batch = blockIdx.y % g.nbatch;
  const int m0 = tm * BM, n0 = tn * BN;
  const int M = g.M, N = g.N, K = g.K;
  const int trans = g.transA[prob];
  const TA* A = (const TA*)g.A[prob] + (long)batch * g.a_bs;
  const TB* B = (const TB*)g.B[prob] + (long)batch * g.b_bs;
  TC* C = (TC*)g.C[prob] + (long)batch * g.c_bs;
  const long lda = g.lda, ldb = g.ldb;

  float ra[EA], rb[EB];
  auto load_tiles = [&](int k0) {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      const int gm = m0 + m, gk = k0 + kk;
      float v = 0.0f;
      if (gm < M && gk < K) v = (float)(trans ? A[(long)gk * lda + gm] : A[(long)gm * lda + gk]);
      ra[e] = v;
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      const int n = i % BN, kk = i / BN;
      const int gn = n0 + n, gk = k0 + kk;
      float v = 0.0f;
      if (gn < N && gk < K) v = (float)B[(long)gk * ldb + gn];
      rb[e] = v;
    }
  };
  auto store_tiles = [&]() {
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int i = tid + e * 256;
      int m, kk;
      if (trans) { m = i % BM; kk = i / BM; } else { m = i / BK; kk = i % BK; }
      split_bf16(ra[e], Ah[m][kk], Al[m][kk]);
    }
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      const int i = tid + e * 256;
      split_bf16(rb[e], Bh[i % BN][i / BN], Bl[i % BN][i / BN]);
    }
  };

  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = v4f{0, 0, 0, 0};

  const int nk = (K + BK - 1) / BK;
  load_tiles(0);
  for (int kt = 0; kt < nk; ++kt) {
    store_tiles();
    __syncthreads();
    if (kt + 1 < nk) load_tiles((kt + 1) * BK);
    const int kc = 8 * (lane >> 4);
    v8bf ah[MI], al[MI], bh[NI], bl[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      ah[i] = *reinterpret_cast<const v8bf*>(&Ah[wm * WTM + i * 16 + (lane & 15)][kc]);
      al[i] = *reinterpret_cast<const v8bf*>(&Al[wm * WTM + i * 16 + (lane & 15)][kc]);
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      bh[j] = *reinterpret_cast<const v8bf*>(&Bh[wn * WTN + j * 16 + (lane & 15)][kc]);
      bl[j] = *reinterpret_cast<const v8bf*>(&Bl[wn * WTN + j * 16 + (lane & 15)][kc]);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
      }
    __syncthreads();
  }

  long offn[NI];
  bool okn[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int n = n0 + wn * WTN + j * 16 + (lane & 15);
    okn[j] = n < N;
    offn[j] = okn[j] ? map2(n, g.cdiv_n, g.cs_n1, g.cs_n0) : 0;
  }
  const float alpha = (float)g.alpha;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * WTM + i * 16 + 4 * (lane >> 4) + r;
      if (m >= M) continue;
      const long offm = map2(m, g.cdiv_m, g.cs_m1, g.cs_m0);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        if (!okn[j]) continue;
        TC* p = C + offm + offn[j];
        float v = alpha * acc[i][j][r];
        if (g.accumulate) v += (float)*p;
        *p = cvt<TC>(v);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// tile selection
// ---------------------------------------------------------------------------
struct TileCfg {
  int bm, bn;
};

// Available (BM, BN) shapes; each has a fixed wavefront arrangement below.
constexpr TileCfg kTiles[] = {{128, 128}, {128, 144}, {64, 160}, {64, 80}, {64, 64}, {32, 32}};

int pick_tile(const GemmBatch& g) {
  int best = -1;
  double best_cost = 1e300;
  const long blocks_y = (long)g.count * g.nbatch;
  for (int c = 0; c < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++c) {
    const int bm = kTiles[c].bm, bn = kTiles[c].bn;
    const long tm = ceil_div(g.M, bm), tn = ceil_div(g.N, bn);
    const long wgs = tm * tn * blocks_y;
    // padded work, penalised when the grid cannot fill 256 compute units, and
    // slightly by the per-tile overhead of small tiles
    const double work = (double)tm * bm * tn * bn * blocks_y;
    const double fill = wgs >= 256 ? 1.0 : 256.0 / (double)wgs;
    const double small = 1.0 + 2048.0 / (double)(bm * bn);
    const double cost = work * fill * small;
    if (cost < best_cost) { best_cost = cost; best = c; }
  }
  return best;
}

template <typename TA, typename TB, typename TC, typename CT>
int launch_k4(const GemmBatch& g, hipStream_t s) {
  const int c = pick_tile(g);
  const int bm = kTiles[c].bm, bn = kTiles[c].bn;
  const int tm = ceil_div(g.M, bm), tn = ceil_div(g.N, bn);
  dim3 grid(tm * tn, g.count * g.nbatch), block(256);
  switch (c) {
    case 0: gemm_k4<TA, TB, TC, CT, 128, 128, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 1: gemm_k4<TA, TB, TC, CT, 128, 144, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 2: gemm_k4<TA, TB, TC, CT, 64, 160, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 3: gemm_k4<TA, TB, TC, CT, 64, 80, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 4: gemm_k4<TA, TB, TC, CT, 64, 64, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    default: gemm_k4<TA, TB, TC, CT, 32, 32, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

template <typename TA, typename TB, typename TC>
int launch_b16(const GemmBatch& g, hipStream_t s) {
  const int c = pick_tile(g);
  const int bm = kTiles[c].bm, bn = kTiles[c].bn;
  const int tm = ceil_div(g.M, bm), tn = ceil_div(g.N, bn);
  dim3 grid(tm * tn, g.count * g.nbatch), block(256);
  switch (c) {
    case 0: gemm_bf16<TA, TB, TC, 128, 128, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 1: gemm_bf16<TA, TB, TC, 128, 144, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 2: gemm_bf16<TA, TB, TC, 64, 160, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 3: gemm_bf16<TA, TB, TC, 64, 80, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 4: gemm_bf16<TA, TB, TC, 64, 64, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    default: gemm_bf16<TA, TB, TC, 32, 32, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

template <typename TA, typename TB, typename TC>
int launch_bx3(const GemmBatch& g, hipStream_t s) {
  const int c = pick_tile(g);
  const int bm = kTiles[c].bm, bn = kTiles[c].bn;
  const int tm = ceil_div(g.M, bm), tn = ceil_div(g.N, bn);
  dim3 grid(tm * tn, g.count * g.nbatch), block(256);
  switch (c) {
    case 0: gemm_bf16x3<TA, TB, TC, 128, 128, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 1: gemm_bf16x3<TA, TB, TC, 128, 144, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 2: gemm_bf16x3<TA, TB, TC, 64, 160, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 3: gemm_bf16x3<TA, TB, TC, 64, 80, 4, 1><<<grid, block, 0, s>>>(g, tm, tn); break;
    case 4: gemm_bf16x3<TA, TB, TC, 64, 64, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
    default: gemm_bf16x3<TA, TB, TC, 32, 32, 2, 2><<<grid, block, 0, s>>>(g, tm, tn); break;
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

// Workgroups of a small product with 16 nt columns each, and its estimated
// microseconds: the launch with the first loads and the sums, and for each 256
// workgroups the longest wavefront's slices (within 15 % of kernel times
// measured from 32 x 20 x 32 to 1875 x 83 x 1875).
double short_groups(const GemmBatch& g, int nt) {
  return (double)ceil_div(g.M, 16) * ceil_div(g.N, 16 * nt) * g.count;
}
double short_us(const GemmBatch& g, int nt) {
  return 3.9 + std::ceil(short_groups(g, nt) / 256.0) * ceil_div(ceil_div(g.K, 16), 8) * (0.31 + 0.32 * nt);
}

// Column blocks per workgroup that fit a set of small products best.
int short_columns(const GemmBatch* gs, int n) {
  int best = 1;
  double cost = 1e300;
  for (int nt = 1; nt <= 5; ++nt) {
    double c = 0.0;
    for (int i = 0; i < n; ++i) c += short_us(gs[i], nt);
    if (c < cost) {
      cost = c;
      best = nt;
    }
  }
  return best;
}

int launch_short(const GemmBatch& g, hipStream_t s) {
  const int nt = short_columns(&g, 1);
  const int tm = ceil_div(g.M, 16), tn = ceil_div(g.N, 16 * nt), wgs = tm * tn * g.count;
  switch (nt) {
    case 1: gemm_short_f64<1><<<wgs, 512, 0, s>>>(g, tm, tn); break;
    case 2: gemm_short_f64<2><<<wgs, 512, 0, s>>>(g, tm, tn); break;
    case 3: gemm_short_f64<3><<<wgs, 512, 0, s>>>(g, tm, tn); break;
    case 4: gemm_short_f64<4><<<wgs, 512, 0, s>>>(g, tm, tn); break;
    default: gemm_short_f64<5><<<wgs, 512, 0, s>>>(g, tm, tn); break;
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

}  // namespace

// Small: up to 24 estimated us, and two rounds of 256 workgroups, or one where a
// wavefront has a single slice (K <= 128): beyond, the split kernel's tiles win,
// which read their operands less often.  Measured kernel times, us, on the
// kernels used before, on those tiles and here: 8 of 32 x 20 x 32 11, 5 and 4.5,
// 8 of 512 x 37 x 512 24, 21 and 10, 105 x 105 x 2500 27, 70 and 15, 4 of 1024 x 64
// x 1024 30, 38 and 19.5, 1875 x 83 x 1875 27, 61 and 23, 1024 x 64 x 64 17, 7 and
// 4; beyond the line, 8 of 1024 x 72 x 1024 42, 50 and 50, 8 of 1024 x 72 x 72 21,
// 9 and 13, 4 of 2500 x 100 x 105 18, 13 and 22, 512 x 512 x 64 11, 9 and 14.
bool gemm_short_applies(const GemmBatch& g) {
  if (g.nbatch != 1 || g.split || g.M <= 0 || g.N <= 0 || g.count <= 0 || g.K <= 0) return false;
  const int nt = short_columns(&g, 1);
  return short_us(g, nt) <= 24.0 && short_groups(g, nt) <= (g.K <= 128 ? 256.0 : 512.0);
}

int grouped_kind(const GemmBatch* gs, int n) {
  if (n > 0 && gemm_short_applies(gs[0])) return -short_columns(gs, n);
  int big = 0;
  double most = -1.0;
  for (int i = 0; i < n; ++i) {
    const double f = (double)gs[i].M * gs[i].N * (double)gs[i].K * gs[i].count * gs[i].nbatch;
    if (f > most) { most = f; big = i; }
  }
  return pick_tile(gs[big]);
}

long grouped_fill(const GemmBatch* gs, int n, int kind, GroupItem* items) {
  const int bm = kind < 0 ? 16 : kTiles[kind].bm, bn = kind < 0 ? -16 * kind : kTiles[kind].bn;
  long total = 0;
  for (int i = 0; i < n; ++i) {
    items[i].g = gs[i];
    items[i].tiles_m = gs[i].M > 0 ? ceil_div(gs[i].M, bm) : 0;
    items[i].tiles_n = gs[i].N > 0 ? ceil_div(gs[i].N, bn) : 0;
    items[i].first = total;
    total += (long)items[i].tiles_m * items[i].tiles_n * gs[i].count * gs[i].nbatch;
  }
  return total;
}

int launch_gemm_grouped(const GroupItem* items, int n, long total, int kind, hipStream_t s) {
  if (n <= 0 || total <= 0) return 0;
  // persistent grid: at most two workgroups per CU of 256
  const int grid = (int)std::min<long>(total, 512);
  if (kind < 0) {
    switch (-kind) {
      case 1: gemm_short_grouped<1><<<grid, 512, 0, s>>>(items, n, total); break;
      case 2: gemm_short_grouped<2><<<grid, 512, 0, s>>>(items, n, total); break;
      case 3: gemm_short_grouped<3><<<grid, 512, 0, s>>>(items, n, total); break;
      case 4: gemm_short_grouped<4><<<grid, 512, 0, s>>>(items, n, total); break;
      default: gemm_short_grouped<5><<<grid, 512, 0, s>>>(items, n, total); break;
    }
  } else {
    switch (kind) {
      case 0: gemm_k4_grouped<128, 128, 2, 2><<<grid, 256, 0, s>>>(items, n, total); break;
      case 1: gemm_k4_grouped<128, 144, 4, 1><<<grid, 256, 0, s>>>(items, n, total); break;
      case 2: gemm_k4_grouped<64, 160, 2, 2><<<grid, 256, 0, s>>>(items, n, total); break;
      case 3: gemm_k4_grouped<64, 80, 4, 1><<<grid, 256, 0, s>>>(items, n, total); break;
      case 4: gemm_k4_grouped<64, 64, 2, 2><<<grid, 256, 0, s>>>(items, n, total); break;
      default: gemm_k4_grouped<32, 32, 2, 2><<<grid, 256, 0, s>>>(items, n, total); break;
    }
  }
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

size_t gemm_si_scratch_bytes() { return (size_t)2 * kSplitMaxCus * 192 * 160 * sizeof(double); }

// Ranges of the split: ncu, or fewer so that each holds at least 8 slices.
static int sk_ranges(long pairs, int ncu) { return (int)std::min<long>(ncu, pairs / 8); }

// Rows of a tile of the split kernel: 192 (4 x 2 wavefronts) where N needs
// more than seven 16-column blocks; else 8 wavefronts one above the other
// with one or two 16-row blocks each and as many columns as N needs (less of
// the matrix work is padding than on 128 or 160 columns).  256 rows read B
// half as often; 128 where the taller tile would add more than a tenth of
// rows past the edge.
static int sk_rows(int M, int N) {
  if (N > 112) return 192;
  const long tall = (long)ceil_div(M, 256) * 256, low = (long)ceil_div(M, 128) * 128;
  return 10 * tall > 11 * low ? 128 : 256;
}

bool gemm_si_balanced_useful(int count, int M, int N, int K, int ncu) {
  // the split pays whenever each tile holds several slices: its ranges keep
  // every CU busy for the same time whatever the tile count, where the
  // plain kernel leaves CUs idle through whole K walks once the tiles are
  // fewer than the slots or do not divide them
  if (ncu < 1 || ncu > kSplitMaxCus || N > 160 || M <= 0 || count <= 0 || K <= 0) return false;
  const long tiles = (long)ceil_div(M, sk_rows(M, N)) * count, ns = ceil_div(K, 16);
  return ns >= 16 && sk_ranges(tiles * ns, ncu) >= 1 && tiles * ns <= (1L << 30);
}

bool gemm_si_balanced_applies(const GemmBatch& g, const void* scratch, int ncu) {
  if (!scratch || ((uintptr_t)scratch & 15) || g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch != 1)
    return false;
  return gemm_si_balanced_useful(g.count, g.M, g.N, g.K, ncu);
}

// One of the tile shapes on the ranges of sk (nwg, per, rem and unit set).
template <int MI, int NI, int WN, bool ONE = false, bool SEQ = false>
static int launch_streamk_f64(const GemmBatch& g, const StreamK& sk, hipStream_t s) {
  using S = SkTile<MI, NI, WN, SEQ>;
  static_assert((size_t)S::BM * S::BN <= 192 * 160, "scratch slots");
  gemm_streamk_f64<MI, NI, WN, ONE, SEQ><<<sk.nwg, S::NT, 0, s>>>(g, sk);
  CTM_HIP_TRY(hipGetLastError());
  if (sk.unit > 1) return 0;   // no tile is cut
  gemm_streamk_fixup<S::BM, S::BN>
      <<<g.count * g.nbatch * sk.tiles_m * sk.tiles_n * (S::BM / kFixRows), 256, 0, s>>>(g, sk);
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

// rows x cols: 128 or 256 rows with 16 to 112 columns, 192 with 128 or 160.
static int launch_streamk_shape(const GemmBatch& g, const StreamK& sk, int rows, int cols, hipStream_t s) {
  const bool tall = rows == 256;
  if (rows == 192)
    return cols == 160 ? launch_streamk_f64<3, 5, 2>(g, sk, s) : launch_streamk_f64<3, 4, 2>(g, sk, s);
  if (g.N == 1)
    return tall ? launch_streamk_f64<2, 1, 1, true>(g, sk, s) : launch_streamk_f64<1, 1, 1, true>(g, sk, s);
  switch (cols / 16) {
    case 1: return tall ? launch_streamk_f64<2, 1, 1>(g, sk, s) : launch_streamk_f64<1, 1, 1>(g, sk, s);
    case 2: return tall ? launch_streamk_f64<2, 2, 1>(g, sk, s) : launch_streamk_f64<1, 2, 1>(g, sk, s);
    case 3: return tall ? launch_streamk_f64<2, 3, 1>(g, sk, s) : launch_streamk_f64<1, 3, 1>(g, sk, s);
    case 4: return tall ? launch_streamk_f64<2, 4, 1>(g, sk, s) : launch_streamk_f64<1, 4, 1>(g, sk, s);
    case 5: return tall ? launch_streamk_f64<2, 5, 1>(g, sk, s) : launch_streamk_f64<1, 5, 1>(g, sk, s);
    case 6: return tall ? launch_streamk_f64<2, 6, 1>(g, sk, s) : launch_streamk_f64<1, 6, 1>(g, sk, s);
    default: return tall ? launch_streamk_f64<2, 7, 1>(g, sk, s) : launch_streamk_f64<1, 7, 1>(g, sk, s);
  }
}

int launch_gemm_si_balanced(const GemmBatch& g, double* scratch, int ncu, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch <= 0) return 0;
  if (!gemm_si_balanced_applies(g, scratch, ncu)) return launch_gemm(g, DT::F64, DT::F64, DT::F64, s);
  const int rows = sk_rows(g.M, g.N);
  StreamK sk{};
  sk.nslices = ceil_div(g.K, 16);
  sk.part = scratch;
  sk.tiles_m = ceil_div(g.M, rows);
  sk.tiles_n = 1;
  sk.unit = 1;
  const int total = g.count * sk.tiles_m * sk.nslices;
  sk.nwg = sk_ranges(total, ncu);
  sk.per = total / sk.nwg;
  sk.rem = total % sk.nwg;
  return launch_streamk_shape(g, sk, rows, rows == 192 ? (g.N > 128 ? 160 : 128) : (g.N + 15) / 16 * 16, s);
}

// Tile and ranges of a split product of any width, by estimated cycles.  A
// range of whole tiles needs no second kernel but leaves CUs idle where the
// tiles do not divide evenly; cut ranges keep all busy and pay for the partial
// tiles.  The constants are rounded from measured launches.  Products whose few
// tiles each walked all of K on the tile kernels, before and after, us: 1024 x
// 1024 x 1024 200 -> 50 (whole tiles of 128 x 32), four transposed 256 x 256 x
// 4096 750 -> 44 + 9 for the second kernel (cut tiles of 256 x 32), 1024 x 64 x
// 1024 185 -> 10 + 5, four 1024 x 1024 x 576 148 -> 98 (256 x 64), 4096 x 256 x
// 256 29 -> 19.  Bound by the matrix cores where K is long (50 TF/s on these,
// 61 on 192 x 160), else by the start of the ranges and the partial tiles.
// Short K on whole tiles, where the tile kernels waited for a tile's first loads
// and stores: eight 2500 x 2500 x 100 409 -> 257 us, four 5184 x 5184 x 144 639 ->
// 618 (476 at the matrix cores' rate), 3600 x 3600 x 64 253 -> 172, 8192 x 64 x 64
// 27 -> 14.
namespace {
struct SplitPlan {
  StreamK sk;
  int rows, cols;
  double cycles;
};

bool plan_split(const GemmBatch& g, bool cut_ok, int ncu, SplitPlan* best) {
  best->cycles = 1e300;
  const long ns = ceil_div(g.K, 16);
  auto consider = [&](int rows, int cols) {
    const int tm = ceil_div(g.M, rows), tn = ceil_div(g.N, cols);
    const long tiles = (long)tm * tn * g.count * g.nbatch;
    if (tiles * ns > (1L << 30)) return;
    // a slice: 2 matrix instructions of 64 cycles per SIMD, k step and 16 x 16
    // block of a wavefront, at the rate they reach with the loads between
    // them, and the barrier; or its operands from L2
    const double blocks = (double)rows * cols / (128 * 16);
    const double slice = std::max(620.0 * blocks + 800.0, (rows + cols) * 128.0 / 12.0);
    auto take = [&](long nwg, long units, int unit, double extra) {
      const double cyc = (double)((units + nwg - 1) / nwg) * unit * slice + extra;
      if (cyc >= best->cycles) return;
      best->cycles = cyc;
      best->rows = rows;
      best->cols = cols;
      best->sk.nslices = (int)ns;
      best->sk.tiles_m = tm;
      best->sk.tiles_n = tn;
      best->sk.nwg = (int)nwg;
      best->sk.per = (int)(units / nwg);
      best->sk.rem = (int)(units % nwg);
      best->sk.unit = unit;
    };
    // a tile's first loads, and its stores beside the other CUs' products
    const long whole = std::min<long>(tiles, ncu);
    take(whole, tiles, (int)ns, (tiles + whole - 1) / whole * (3000.0 + rows * cols / 2.0));
    const long nwg = sk_ranges(tiles * ns, ncu);
    // the second kernel's launch, and the partials written and read
    if (cut_ok && nwg >= 1) take(nwg, tiles * ns, 1, 14000.0 + (double)nwg * rows * cols * 16.0 / 1250.0);
  };
  for (int cols = 16; cols <= 112; cols += 16) {
    consider(128, cols);
    consider(256, cols);
  }
  consider(192, 128);
  consider(192, 160);
  return best->cycles < 1e300;
}
}  // namespace

// Few rows leave much of the split kernel's tiles of 128 or more empty, which
// long K makes up for by spreading the work: four of 64 x 8192 x 64 take 15.6 us on
// the tile kernels and 17.5 here, of 64 x 8192 x 300 70 and 49.
bool gemm_whole_applies(const GemmBatch& g) {
  return !g.split && g.M >= (g.K >= 256 ? 64 : 97) && g.N > 0 && g.K > 16 && g.count > 0 &&
         g.nbatch > 0 && !gemm_short_applies(g);
}

// Tiles are cut where K >= 256: below that the partial tiles outweigh what
// the CUs would idle (243 x 32 x 243: 14 + 4 us cut, 10 us on a tile kernel).
int launch_gemm_f64_any(const GemmBatch& g, double* scratch, int ncu, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch <= 0) return 0;
  SplitPlan p{};
  if (scratch && ((uintptr_t)scratch & 15) == 0 && g.K >= 256 && ncu >= 1 && ncu <= kSplitMaxCus &&
      gemm_whole_applies(g) && plan_split(g, true, ncu, &p)) {
    p.sk.part = scratch;
    return launch_streamk_shape(g, p.sk, p.rows, p.cols, s);
  }
  return launch_gemm(g, DT::F64, DT::F64, DT::F64, s);
}

// Ordered products: thin ones with long K on tiles of 192 rows in ranges that
// begin at w total / nwg, where rows and bases are aligned for 16-byte loads, all
// others whole, every sum over ascending k.  An element's bits then depend on this
// rule alone, not on how the products are tiled elsewhere.
int launch_gemm_ordered(const GemmBatch& g, double* scratch, int ncu, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch <= 0) return 0;
  StreamK sk{};
  sk.nslices = ceil_div(g.K, 16);
  sk.tiles_m = ceil_div(g.M, 192);
  sk.tiles_n = 1;
  sk.part = scratch;
  sk.unit = 1;
  auto run = [&](int cols) {
    return cols == 160 ? launch_streamk_f64<3, 5, 2, false, true>(g, sk, s)
                       : launch_streamk_f64<3, 4, 2, false, true>(g, sk, s);
  };
  bool cut = scratch && !((uintptr_t)scratch & 15) && ncu >= 1 && ncu <= kSplitMaxCus && g.nbatch == 1 &&
             g.N > 1 && g.N <= 160 && sk.nslices >= 16 && !(g.lda & 1);
  for (int i = 0; i < g.count; ++i)
    cut = cut && !((uintptr_t)g.A[i] & 15) && !((uintptr_t)g.B[i] & ((g.ldb & 1) ? 7 : 15));
  const long tiles = (long)sk.tiles_m * g.count;
  if (cut && tiles * sk.nslices >= 8 && tiles * sk.nslices <= (1L << 30)) {
    sk.total = (int)(tiles * sk.nslices);
    sk.nwg = sk_ranges(sk.total, ncu);
    return run(g.N > 128 ? 160 : 128);
  }
  // whole tiles where they fill the chip (eight 2500 x 2500 x 100 313 us, 423 on the
  // tile kernels), else the tile kernels
  const int cols = g.N > 128 && g.N <= 160 ? 160 : 128;
  sk.tiles_n = ceil_div(g.N, cols);
  const long all = (long)sk.tiles_m * sk.tiles_n * g.count * g.nbatch;
  if (g.K > 16 && g.N > 64 && all >= 128 && all * sk.nslices <= (1L << 30)) {
    sk.nwg = (int)std::min<long>(all, kSplitMaxCus);
    sk.per = (int)(all / sk.nwg);
    sk.rem = (int)(all % sk.nwg);
    sk.unit = sk.nslices;
    return run(cols);
  }
  return launch_k4<double, double, double, double>(g, s);
}

bool gemm_si_f32_balanced_applies(const GemmBatch& g, const void* scratch, int ncu) {
  if (!scratch || ((uintptr_t)scratch & 15) || g.M <= 0 || g.N <= 0 || g.count <= 0 ||
      g.nbatch != 1 || g.N > skf32::BN)
    return false;
  if ((g.lda & 3) || (g.ldb & 1)) return false;
  for (int i = 0; i < g.count; ++i)
    if (((uintptr_t)g.A[i] & 15) || ((uintptr_t)g.B[i] & 15)) return false;
  const bool rowmajor_c = g.cdiv_m >= g.M && g.cdiv_n >= g.N && g.cs_n0 == 1;
  // at least 8 slices per range, so that no range is empty, and 8 per tile
  const long tiles = (long)g.count * ceil_div(g.M, skf32::BM), ns = ceil_div(g.K, skf32::BK);
  return rowmajor_c && ncu >= 1 && ncu <= kSplitMaxCus && ns >= 8 && tiles * ns >= 8L * ncu &&
         tiles * ns <= (1L << 30);
}

int launch_gemm_si_f32_balanced(const GemmBatch& g, double* scratch, int ncu, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch <= 0) return 0;
  if (!gemm_si_f32_balanced_applies(g, scratch, ncu)) return launch_gemm_si_f32(g, s);
  const int tm = ceil_div(g.M, skf32::BM);
  StreamK sk{};
  sk.nslices = ceil_div(g.K, skf32::BK);
  sk.tiles_m = tm;
  sk.tiles_n = 1;
  sk.unit = 1;
  const int total = g.count * tm * sk.nslices;
  sk.nwg = ncu;
  sk.per = total / ncu;
  sk.rem = total % ncu;
  sk.part = scratch;
  gemm_streamk_f32<<<ncu, skf32::NT, 0, s>>>(g, sk);
  CTM_HIP_TRY(hipGetLastError());
  gemm_streamk_fixup<192, 160><<<(int)((long)g.count * tm * (192 / kFixRows)), 256, 0, s>>>(g, sk);
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

namespace {
// 8-byte aligned pairs of float32 / float64 operands for the float32 skinny tile.
bool pairs_ok(const GemmBatch& g) {
  if ((g.lda & 1) || (g.ldb & 1) || (g.a_bs & 1) || (g.b_bs & 1)) return false;
  for (int i = 0; i < g.count; ++i)
    if (((uintptr_t)g.A[i] & 15) || ((uintptr_t)g.B[i] & 15)) return false;
  return true;
}

// float32 contractions long enough for the double-buffered float32 tile.
template <typename TA, typename TB, typename TC>
bool launch_f32_db(const GemmBatch& g, hipStream_t s, int* rc) {
  if (g.K < 512 || g.M < 256 || !pairs_ok(g)) return false;
  auto go = [&](auto kern, int bm, int bn, int threads) {
    const int tm = ceil_div(g.M, bm), tn = ceil_div(g.N, bn);
    kern<<<dim3(tm * tn * g.count * g.nbatch), dim3(threads), 0, s>>>(g, tm, tn);
    const hipError_t e = hipGetLastError();
    *rc = e == hipSuccess ? 0 : hip_fail(e, "float32 skinny tile", __LINE__);
  };
  if (g.N <= 160)
    go(gemm_skinny_f32x<TA, TB, TC, 96, 160, 2, 2>, 96, 160, 256);
  else if ((long)g.M * g.count * g.nbatch >= 16384)
    go(gemm_skinny_f32x<TA, TB, TC, 256, 144, 8, 1>, 256, 144, 512);
  else
    go(gemm_skinny_f32x<TA, TB, TC, 128, 144, 4, 1>, 128, 144, 256);
  return true;
}

}  // namespace

// Compute type: float64 when any operand is float64 and the mode is f64;
// the caller selects the mode through the operand types:
//   (F64, F64, *)   -> float64 MFMA
//   (F32, *, *)     -> float32 MFMA (f64 B operands are rounded to f32)
//   (BF16, *, *)    -> bf16 MFMA with f32 accumulation
int launch_gemm(const GemmBatch& g, DT ta, DT tb, DT tc, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.count <= 0 || g.nbatch <= 0) return 0;
  if (g.K <= 0 && !g.accumulate) {
    // empty sum: the kernels still write zeros (load loop does not run)
  }
  if (g.split) {
    // split bfloat16 products of float32-stored contraction operands
    if (ta == DT::F64 && tb == DT::F32 && tc == DT::F32) return launch_bx3<double, float, float>(g, s);
    if (ta == DT::F32 && tb == DT::F64 && tc == DT::F64) return launch_bx3<float, double, double>(g, s);
    if (ta == DT::F32 && tb == DT::F32 && tc == DT::F64) return launch_bx3<float, float, double>(g, s);
    if (ta == DT::F64 && tb == DT::F32 && tc == DT::F64) return launch_bx3<double, float, double>(g, s);
    set_thread_error("launch_gemm: unsupported type combination for split bfloat16");
    return 1;
  }
  if (ta == DT::F64 && tb == DT::F64) {
    if (tc == DT::F64 && gemm_short_applies(g)) return launch_short(g, s);
    SplitPlan p{};
    if (tc == DT::F64 && gemm_whole_applies(g) && plan_split(g, false, kSplitMaxCus, &p))
      return launch_streamk_shape(g, p.sk, p.rows, p.cols, s);
    if (tc == DT::F64) return launch_k4<double, double, double, double>(g, s);
    if (tc == DT::F32) return launch_k4<double, double, float, double>(g, s);
  }
  {
    // the float32 contractions with long K on the double-buffered tile
    int rc = 0;
    if (ta == DT::F32 && tb == DT::F64 && tc == DT::F64 &&
        launch_f32_db<float, double, double>(g, s, &rc))
      return rc;
    if (ta == DT::F64 && tb == DT::F32 && tc == DT::F32 &&
        launch_f32_db<double, float, float>(g, s, &rc))
      return rc;
    if (ta == DT::F64 && tb == DT::F32 && tc == DT::F64 &&
        launch_f32_db<double, float, double>(g, s, &rc))
      return rc;
  }
  if (ta == DT::F32) {
    if (tb == DT::F64 && tc == DT::F64) return launch_k4<float, double, double, float>(g, s);
    if (tb == DT::F64 && tc == DT::F32) return launch_k4<float, double, float, float>(g, s);
    if (tb == DT::F32 && tc == DT::F32) return launch_k4<float, float, float, float>(g, s);
    if (tb == DT::F32 && tc == DT::F64) return launch_k4<float, float, double, float>(g, s);
  }
  if (ta == DT::F64 && tb == DT::F32) {
    if (tc == DT::F32) return launch_k4<double, float, float, float>(g, s);
    if (tc == DT::F64) return launch_k4<double, float, double, float>(g, s);
  }
  if (ta == DT::F64 && tb == DT::BF16) {
    if (tc == DT::BF16) return launch_b16<double, __bf16, __bf16>(g, s);
    if (tc == DT::F32) return launch_b16<double, __bf16, float>(g, s);
    if (tc == DT::F64) return launch_b16<double, __bf16, double>(g, s);
  }
  if (ta == DT::F64 && tb == DT::F32 && tc == DT::BF16) return launch_k4<double, float, __bf16, float>(g, s);
  if (ta == DT::BF16) {
    if (tb == DT::BF16 && tc == DT::F64) return launch_b16<__bf16, __bf16, double>(g, s);
    if (tb == DT::F64 && tc == DT::F64) return launch_b16<__bf16, double, double>(g, s);
    if (tb == DT::F64 && tc == DT::F32) return launch_b16<__bf16, double, float>(g, s);
    if (tb == DT::F32 && tc == DT::F32) return launch_b16<__bf16, float, float>(g, s);
    if (tb == DT::F32 && tc == DT::F64) return launch_b16<__bf16, float, double>(g, s);
  }
  if (ta == DT::F64 && tb == DT::F64 && tc == DT::BF16)
    return launch_k4<double, double, __bf16, double>(g, s);
  if (ta == DT::F64 && tb == DT::F64) return launch_k4<double, double, double, double>(g, s);
  set_thread_error("launch_gemm: unsupported type combination");
  return 1;
}

}  // namespace sictm
