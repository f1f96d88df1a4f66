// Site absorption of the enlarged corners through the single-layer tensor.
//
// The enlarged corner of the CTMRG move (Fig. 1, the corner C T T a) ends
// with the absorption Ct[(x, o1), (y, o2)] = sum_(p, q) W[(x, y), p, q]
// a[(p, q), (o1, o2)] of the double-layer site tensor a, whose legs pair a
// ket and a bra index (p = pk D + pb, ket-major) with
// a = sum_s A[s, pk, qk, o1k, o2k] A[s, pb, qb, o1b, o2b].  Contracted as one
// D^4 x D^4 matrix that costs 2 chi^2 D^8 flops per corner.  Here the ket
// layer is absorbed first and the bra layer (with the physical index) second:
//   X[(x, y), pb, qb, (s, o1k, o2k)] = sum_(pk, qk) W[(x, y), (pk pb), (qk qb)] A[s, pk, qk, o1k, o2k]
//   Ct[(x, o1k o1b), (y, o2k o2b)]   = sum_(pb, qb, s) X[...] A[s, pb, qb, o1b, o2b]
// the same tensor for 4 d chi^2 D^6 flops (9x less at D = 6, d = 2).
//
// A wavefront takes one (x, y) pair at a time, on its own: with rows (pb, qb)
// and K = (pk, qk), the first product leaves X_s in the matrix cores' result
// layout (row l / 16 + 4 r, column l % 16), which is their operand layout for
// the second product, out^T[(o1b, o2b), (o1k, o2k)] += A_s^T X_s with
// K = (pb, qb), so X never leaves the registers and no wavefront waits for
// another.  Both products read the same fragments of A_s, from a table every
// workgroup sets up once (the workgroups are persistent); the pair's W and
// its output block pass through one buffer per wavefront, so that global
// memory is read and written in runs.  D^2 = 36 is padded to 48 rows and
// columns (324 matrix instructions per pair where 182 would hold the
// numbers), which costs less than sharing rows between wavefronts.
//
// Bound by the f64 matrix cores (0.70 ms for the four corners of D = 6,
// chi = 144, against 0.35 ms of memory traffic).  Two pairs per workgroup, with X and the
// output staged in LDS for all four wavefronts and A permuted anew by every
// workgroup, took 2.64 ms; this form 0.89 ms (D = 5, chi = 75: 387 and
// 108 us; D = 4, chi = 64: 136 and 16 us).

#include "common.h"
#include "elem.h"

namespace sictm {
namespace {

constexpr int kAbsMaxDl = 36;     // D^2 up to D = 6
constexpr int kAbsMaxN = 72;      // d D^2 up to d = 2 at D = 6
constexpr int kAbsWaves = 8;

constexpr int kAbsMaxProb = 8;

struct AbsArgs {
  const double* W[kAbsMaxProb];    // [nR][Dl][Dl] per problem
  void* Ct[kAbsMaxProb];           // output (TO) per problem, element (R, o1, o2) at
                                   // (R / n2) sR1 + (R % n2) sR2 + o1 so1 + o2 so2
  const double* A[kAbsMaxProb];    // single-layer site tensor [s][u][l][d][r] per problem
  long sA[kAbsMaxProb][4];         // per problem: strides in A of the legs p, q, o1, o2
  long nR, sR1, sR2, so1, so2;
  int n2, d;
};

// Sizes for a bond dimension D (a compile-time constant, so that index
// divisions become multiplies).
template <int D>
struct AbsTile {
  static constexpr int Dl = D * D;
  static constexpr int RB = (Dl + 15) / 16;        // 16-row (and column) blocks
  static constexpr int KS = (Dl + 3) / 4;          // k-steps
  static constexpr int LA = RB == 1 ? 16 : 48;     // table row: rows 1 apart fall 32 banks apart
  static constexpr int SA = 4 * KS * LA;           // table of one s
  static constexpr int SW = Dl * Dl + (Dl & 1);    // one pair's W or output block
  static constexpr int NP = (Dl * Dl / 2 + 63) / 64;   // 16-byte loads per lane
  static constexpr int dmax = kAbsMaxN / Dl;
};

typedef double v2da __attribute__((ext_vector_type(2), aligned(8)));

template <int D, typename TO>
__global__ __launch_bounds__(64 * kAbsWaves, 2) void k_absorb_corner(AbsArgs a) {
  using S = AbsTile<D>;
  constexpr int Dl = S::Dl, RB = S::RB, KS = S::KS, LA = S::LA;
  constexpr int D4 = Dl * Dl;
  // As: [s][(p, q)][(o1, o2)], zeros outside
  __shared__ __attribute__((aligned(16))) double As[S::dmax * S::SA], bufs[kAbsWaves][S::SW];
  const int prob = blockIdx.y, d = a.d;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  double* buf = bufs[wave];
  const long* st = a.sA[prob];
  for (int i = tid; i < d * S::SA; i += 64 * kAbsWaves) {
    const int s = i / S::SA, k = i % S::SA / LA, n = i % LA;
    As[i] = k < Dl && n < Dl ? a.A[prob][(long)s * D4 + (k / D) * st[0] + (k % D) * st[1] +
                                         (n / D) * st[2] + (n % D) * st[3]]
                             : 0.0;
  }
  __syncthreads();
  // offsets in a pair's block of (hi, lo) as the ket halves (of K = (pk, qk)
  // and of (o1k, o2k)) and as the bra halves (of (pb, qb) and of (o1b, o2b))
  auto ket = [](int i) { return (i / D) * D * Dl + (i % D) * D; };
  auto bra = [](int i) { return (i / D) * Dl + i % D; };
  int kk[KS], kb[KS];   // of 4 t + lk
  bool kin[KS];
#pragma unroll
  for (int t = 0; t < KS; ++t) {
    kin[t] = 4 * t + lk < Dl;
    kk[t] = kin[t] ? ket(4 * t + lk) : 0;
    kb[t] = kin[t] ? bra(4 * t + lk) : 0;
  }
  int rb[RB];   // of 16 i + li
  bool rin[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    rin[i] = 16 * i + li < Dl;
    rb[i] = rin[i] ? bra(16 * i + li) : 0;
  }
  const double* W = a.W[prob];
  TO* C = (TO*)a.Ct[prob];
  const long step = (long)gridDim.x * kAbsWaves;
  for (long R = (long)blockIdx.x * kAbsWaves + wave; R < a.nR; R += step) {
    {
      const double* q = W + R * D4;
      v2da w[S::NP];
#pragma unroll
      for (int e = 0; e < S::NP; ++e) {
        const int i = lane + 64 * e;
        if (i < D4 / 2) w[e] = *(const v2da*)(q + 2 * i);
      }
#pragma unroll
      for (int e = 0; e < S::NP; ++e) {
        const int i = lane + 64 * e;
        if (i < D4 / 2) *(v2da*)(buf + 2 * i) = w[e];
      }
      if ((D4 & 1) && lane == 0) buf[D4 - 1] = q[D4 - 1];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double wf[RB][KS];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        const double v = buf[rb[i] + kk[t]];
        wf[i][t] = rin[i] && kin[t] ? v : 0.0;
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // one column block at a time (unrolled, its fragments would not fit the registers)
#pragma unroll 1
    for (int j = 0; j < RB; ++j) {
      const int col = 16 * j + li;
      v4d out[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) out[i] = v4d{0, 0, 0, 0};
#pragma unroll 1
      for (int s = 0; s < d; ++s) {
        const double* F = As + s * S::SA + lk * LA + li;
        v4d x[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) x[i] = v4d{0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          const double f = F[4 * t * LA + 16 * j];
#pragma unroll
          for (int i = 0; i < RB; ++i)
            x[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(wf[i][t], f, x[i], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < KS; ++t)
#pragma unroll
          for (int i = 0; i < RB; ++i)
            out[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(F[4 * t * LA + 16 * i], x[t >> 2][t & 3],
                                                          out[i], 0, 0, 0);
      }
      // row 4 t + lk = (o1b, o2b), column 16 j + li = (o1k, o2k)
#pragma unroll
      for (int t = 0; t < KS; ++t)
        if (kin[t] && col < Dl) buf[ket(col) + kb[t]] = out[t >> 2][t & 3];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    TO* o = C + (R / a.n2) * a.sR1 + (R % a.n2) * a.sR2;
    if (D % 2 == 0 && a.so2 == 1) {
      using V2 = TO __attribute__((ext_vector_type(2), aligned(sizeof(TO))));
#pragma unroll
      for (int e = 0; e < S::NP; ++e) {
        const int i = 2 * (lane + 64 * e);
        if (i < D4) {
          const v2da v = *(const v2da*)(buf + i);
          V2 u;
          u.x = (TO)v.x;
          u.y = (TO)v.y;
          *(V2*)(o + (i / Dl) * a.so1 + i % Dl) = u;
        }
      }
    } else {
      for (int i = lane; i < D4; i += 64) o[(i / Dl) * a.so1 + (i % Dl) * a.so2] = (TO)buf[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

}  // namespace

bool absorb_corner_fits(int D, int d) {
  return d >= 1 && D >= 2 && D * D <= kAbsMaxDl && d * D * D <= kAbsMaxN;
}

// Persistent workgroups: as many as the chip holds side by side (LDS, and
// the registers of D = 6), shared by the problems.
template <int D, typename TO>
static int launch_absorb_d(const AbsArgs& a, int count, hipStream_t s) {
  const long per = (256L * (D >= 6 ? 1 : D == 5 ? 2 : 4) + count - 1) / count;
  const long need = (a.nR + kAbsWaves - 1) / kAbsWaves;
  k_absorb_corner<D, TO><<<dim3((unsigned)(need < per ? need : per), count), 64 * kAbsWaves, 0, s>>>(a);
  CTM_HIP_TRY(hipGetLastError());
  return 0;
}

template <typename TO>
static int launch_absorb_t(const AbsArgs& a, int count, int D, hipStream_t s) {
  switch (D) {
    case 2: return launch_absorb_d<2, TO>(a, count, s);
    case 3: return launch_absorb_d<3, TO>(a, count, s);
    case 4: return launch_absorb_d<4, TO>(a, count, s);
    case 5: return launch_absorb_d<5, TO>(a, count, s);
    default: return launch_absorb_d<6, TO>(a, count, s);
  }
}

int launch_absorb(int count, const double* const* W, void* const* out, bool out_f32,
                  const double* const* A, const long (*legs)[4], long nR, int n2,
                  const long* ostr, int D, int d, hipStream_t s) {
  if (!absorb_corner_fits(D, d) || nR < 1 || n2 < 1 || count < 1 || count > kAbsMaxProb) {
    set_thread_error("single-layer absorption: D, d or the problem count outside its tiling");
    return 1;
  }
  AbsArgs a{};
  for (int i = 0; i < count; ++i) {
    a.W[i] = W[i];
    a.Ct[i] = out[i];
    a.A[i] = A[i];
    for (int j = 0; j < 4; ++j) a.sA[i][j] = legs[i][j];
  }
  a.nR = nR;
  a.n2 = n2;
  a.sR1 = ostr[0];
  a.sR2 = ostr[1];
  a.so1 = ostr[2];
  a.so2 = ostr[3];
  a.d = d;
  return out_f32 ? launch_absorb_t<float>(a, count, D, s) : launch_absorb_t<double>(a, count, D, s);
}

int launch_absorb_corners(const double* const* W, void* const* Ct, bool out_f32, const double* A,
                          const long (*legs)[4], int chi, int D, int d, hipStream_t s) {
  const long Dl = (long)D * D, N1 = (long)chi * Dl;
  const long ostr[4] = {Dl * N1, Dl, N1, 1};
  const double* As[4] = {A, A, A, A};
  return launch_absorb(4, W, Ct, out_f32, As, legs, (long)chi * chi, chi, ostr, D, d, s);
}

}  // namespace sictm
