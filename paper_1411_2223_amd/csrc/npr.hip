// npr.hip -- the one-colour four-fermion operator of the paper's NPR code
// (section "GTX Titan Black", Eq. (1)), in FP64 as the paper runs it.
//
// For every hypercube z (corners z_A = 2z + A, A a 4-bit mask) and operator
// I = (S1, F1, S2, F2):
//   V[a1][a2][a3][a4] = sum_{A,B,C,D} M1_AB M2_CD eps(z_A) eps(z_C)
//       (G1(z_A)^dag U_AD G4(z_D))_{a1 a4} (G3(z_C)^dag U_CB G2(z_B))_{a3 a2}
// M = (gamma_S (x) xi_F)bar, the spin-taste matrix (1/4) Tr[gamma_A^dag gamma_S
// gamma_B gamma_F^dag]; eps = (-1)^(x+y+z+t); U_AD the link product averaged
// over every shortest path from z_A to z_D; G_f the propagators (each chi by a
// propagator, each chibar by its staggered conjugate).  M has one nonzero per
// row, at B = A ^ S ^ F, so each operator is 16 x 16 terms (A, C).
//
// One workgroup per hypercube:
//   1. the 16 corners' propagators to LDS, and the 64 single steps of the
//      hypercube (from corner A along mu: the link U_mu(z_A) if bit mu of A is
//      clear, else the conjugate of the link arriving at z_A);
//   2. the 256 averages U_AD by the first step of each path, in rounds of
//      growing distance |A ^ D| (U_AD = (1/d) sum_mu step(A, mu) U_{A^mu, D});
//      the pairs are dealt to threads in order of distance, so the lanes of a
//      wave share a round;
//   3. X_AD = G1(A)^dag U_AD G4(D) and Y_AD = G3(A)^dag U_AD G2(D) to LDS;
//   4. the contraction (contract): operators that pair up share their products.
#include <math.h>
#include <string.h>

#include <string>

#include "asq_internal.h"

namespace asq {
namespace {

constexpr int kNprThreads = 256;
constexpr int kNprOpsPerLaunch = 32;
constexpr int kNprOpsPerPass = 16;    // 4 per wave, each over the 16 lanes of its corners A
constexpr int kNprPairsPerPass = 8;   // 2 per wave, each over 32 lanes: corners A and halves of D
// a matrix per pair (A, D) at A * kRow + 9 D complex entries: one spare entry per
// row A puts the 16 rows A that a wave reads at once in different LDS banks
constexpr int kRow = 16 * 9 + 1;
constexpr int kPairMats = 16 * kRow;

// the 256 pairs (A, D), 16 A + D, in order of distance |A ^ D| (then A, then D)
struct PairOrder {
  unsigned char p[256];
};
constexpr int popcount4(int m) { return (m & 1) + (m >> 1 & 1) + (m >> 2 & 1) + (m >> 3 & 1); }
constexpr PairOrder make_pair_order() {
  PairOrder t{};
  int n = 0;
  for (int d = 0; d <= 4; ++d)
    for (int a = 0; a < 16; ++a)
      for (int b = 0; b < 16; ++b)
        if (popcount4(a ^ b) == d) t.p[n++] = (unsigned char)(16 * a + b);
  return t;
}
__constant__ PairOrder kPairOrder = make_pair_order();

struct NprOp {
  unsigned char p1, p2;  // S1 ^ F1, S2 ^ F2: B = A ^ p1, D = C ^ p2
  unsigned short neg1;   // bit A: M1_{A, A^p1} eps(z_A) = -1 (else +1)
  unsigned short neg2;   // bit C: M2_{C, C^p2} eps(z_C) = -1
  unsigned char out;     // place of the operator in the launch's output
  // of a pair (see contract): the partner's place, and the signs lambda and kappa
  unsigned char out_b;
  unsigned char lambda_neg, kappa_neg;
};
constexpr unsigned char kNoPartner = 255;  // out_b of an operator summed by the pair form on its own

struct NprArgs {
  int X, Y, Z, T;
  int hx, hy, hz;  // hypercubes per direction (x, y, z)
  const double2* thin;
  const double2* g[4];
  double2* out;     // [nop_total][nz][81]
  long nz;
  int op0;          // index of this launch's first operator in the output
  int nsingle;      // operators on their own: ops[0 .. nsingle)
  int npair;        // pairs: ops[nsingle .. nsingle + npair)
  NprOp ops[kNprOpsPerLaunch];
};

typedef double2 c64;

__device__ __forceinline__ c64 cmul(c64 a, c64 b) {
  return make_double2(__builtin_fma(a.x, b.x, -a.y * b.y), __builtin_fma(a.x, b.y, a.y * b.x));
}
// acc + conj(a) b
__device__ __forceinline__ c64 cmac_cj(c64 acc, c64 a, c64 b) {
  acc.x = __builtin_fma(a.x, b.x, acc.x);
  acc.x = __builtin_fma(a.y, b.y, acc.x);
  acc.y = __builtin_fma(a.x, b.y, acc.y);
  acc.y = __builtin_fma(-a.y, b.x, acc.y);
  return acc;
}
__device__ __forceinline__ c64 cmac(c64 acc, c64 a, c64 b) {
  acc.x = __builtin_fma(a.x, b.x, acc.x);
  acc.x = __builtin_fma(-a.y, b.y, acc.x);
  acc.y = __builtin_fma(a.x, b.y, acc.y);
  acc.y = __builtin_fma(a.y, b.x, acc.y);
  return acc;
}

// c = a b (3 x 3, row-major)
__device__ __forceinline__ void m3mul(const c64* a, const c64* b, c64* c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      c64 s = cmul(a[3 * i], b[j]);
      s = cmac(s, a[3 * i + 1], b[3 + j]);
      s = cmac(s, a[3 * i + 2], b[6 + j]);
      c[3 * i + j] = s;
    }
}
// c = a^dag b
__device__ __forceinline__ void m3mul_dag(const c64* a, const c64* b, c64* c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      c64 s = make_double2(0.0, 0.0);
      s = cmac_cj(s, a[i], b[j]);
      s = cmac_cj(s, a[3 + i], b[3 + j]);
      s = cmac_cj(s, a[6 + i], b[6 + j]);
      c[3 * i + j] = s;
    }
}
// c = a b^dag
__device__ __forceinline__ void m3mul_bdag(const c64* a, const c64* b, c64* c) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      c64 s = make_double2(0.0, 0.0);
      s = cmac_cj(s, b[3 * j], a[3 * i]);
      s = cmac_cj(s, b[3 * j + 1], a[3 * i + 1]);
      s = cmac_cj(s, b[3 * j + 2], a[3 * i + 2]);
      c[3 * i + j] = s;
    }
}

// Contraction over the pairs (A, D) of one hypercube.  With C = D ^ p2 and B = A ^ p1,
//   V[a1][a2][a3][a4] = sum_{A,D} f(A, D) X_AD[a1][a4] Y_CB[a3][a2],  f = s1(A) s2(C).
// A lane owns one operator and one corner A, sums D one a3 at a time (27 outputs) and
// shares the sums with the other lanes of the operator by halving exchanges, after
// which each lane stores the outputs it ended with.  The 16 lanes of an operator read
// 16 rows A of X and 16 entries B of a row C of Y, each in its own LDS banks.
//
// PAIR: two operators a, b with p1_b = p1_a ^ 1, p2_b = p2_a ^ 1 and f_b = kappa f_a
// (a spin structure and its product with gamma_x on both bilinears), where
// f_a(A ^ 1, D ^ 1) = lambda f_a(A, D), are summed together over the reps (A even):
//   V_a = sum f (X Y + lambda X1 Y1),  kappa V_b = sum f (X Y1 + lambda X1 Y),
// X1, Y1 the entries at flipped x bits.  With X+- = X +- X1 (Y alike) and
//   S0 = sum f X+ Y(lambda),  S1 = sum f X- Y(-lambda),
// V_a = (S0 + S1) / 2 and kappa V_b = lambda (S0 - S1) / 2: two operators for the
// products of one.  X and Y hold the sums (even A, even B) and differences; lanes of
// even A form S0, of odd A S1; 32 lanes per pair, each with half of the D.  16
// operators of 20^3 x 64 (8 pairs) take 1.87 ms, 2.50 ms one by one (before the lane
// swaps of the exchanges, 1.98).
// DPP controls: the lane 8 on in its row of 16 (lane ^ 8), and lane ^ 2
constexpr int kRowRotate8 = 0x128, kQuadXor2 = 0x4e;
template <int CTRL>
__device__ __forceinline__ double from_lane(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
// One halving step over lane bit BIT (32 or 16): lo of this lane and its partner where
// the bit is clear, hi of both where it is set.  The swap exchanges the upper half
// (odd rows) of one register with the lower half (even rows) of the other.
template <int BIT>
__device__ __forceinline__ double add_swapped(double lo, double hi) {
  const unsigned long long a = (unsigned long long)__double_as_longlong(lo);
  const unsigned long long b = (unsigned long long)__double_as_longlong(hi);
  auto swap = [](unsigned x, unsigned y) {
    if constexpr (BIT == 32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
    else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
  };
  const auto l = swap((unsigned)a, (unsigned)b);
  const auto h = swap((unsigned)(a >> 32), (unsigned)(b >> 32));
  return __longlong_as_double((long long)((unsigned long long)h[0] << 32 | l[0])) +
         __longlong_as_double((long long)((unsigned long long)h[1] << 32 | l[1]));
}

template <bool PAIR>
__device__ __forceinline__ void contract(const NprArgs& P, long z, const c64* Xs, const c64* Ys) {
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  constexpr int kLanes = PAIR ? 32 : 16, kPass = PAIR ? kNprPairsPerPass : kNprOpsPerPass;
  constexpr int kSum = PAIR ? 8 : 16;  // D per lane
  const int n = PAIR ? P.npair : P.nsingle;
  // the lane bits that are summed over (of A, and of D in a pair) are the upper four,
  // for the exchanges below; then, in a pair, the lowest bit of A; then the operator
  const int Ak = PAIR ? lane >> 1 & 15 : lane >> 2, t = PAIR ? Ak & 1 : 0;
  const int d0 = PAIR ? (lane >> 5) * kSum : 0;
  const c64* xrow = Xs + Ak * kRow;
  for (int pass = 0; pass * kPass < n; ++pass) {
    const int opl = pass * kPass + (64 / kLanes) * wv + lane % (64 / kLanes);
    const bool act = opl < n;
    NprOp o = {};
    if (act) o = P.ops[(PAIR ? P.nsingle : 0) + opl];
    const int Ar = Ak ^ t;  // the rep's corner
    const double s1 = (o.neg1 >> Ar & 1) ? -1.0 : 1.0;
    int B = Ar ^ o.p1, p2 = o.p2;
    double sy = s1;
    if constexpr (PAIR) {
      // Y(+-) of the pair of (C, B): at the entry whose second index is even, or the
      // next one; a difference taken from its other end changes sign
      const int b0 = B & 1, ty = t ^ o.lambda_neg;
      p2 ^= b0;
      B = (B ^ b0) | ty;
      if (b0 & ty) sy = -sy;
    }
    const c64* ycol = Ys + 9 * B;
    double* const out =
        (double*)(P.out + ((size_t)(P.op0 + (act ? (t ? o.out_b : o.out) : 0)) * P.nz + z) * 81);
#pragma unroll 1
    for (int a3 = 0; a3 < 3; ++a3) {
      double v[54];  // [a1][a2][a4] as (re, im) pairs
#pragma unroll
      for (int k = 0; k < 54; ++k) v[k] = 0.0;
      if (act) {
        const c64* ybase = ycol + 3 * a3;
#pragma unroll 2
        for (int k = 0; k < kSum; ++k) {
          const int Dk = d0 + k;
          const double s = (o.neg2 >> (Dk ^ o.p2) & 1) ? -sy : sy;
          c64 xv[9], yv[3];
#pragma unroll
          for (int e = 0; e < 9; ++e) xv[e] = xrow[9 * Dk + e];  // X_AD[a1][a4]
#pragma unroll
          for (int e = 0; e < 3; ++e) {                           // Y_CB[a3][a2]
            const c64 y = ybase[(Dk ^ p2) * kRow + e];
            yv[e] = make_double2(s * y.x, s * y.y);
          }
#pragma unroll
          for (int a1 = 0; a1 < 3; ++a1)
#pragma unroll
            for (int a2 = 0; a2 < 3; ++a2)
#pragma unroll
              for (int a4 = 0; a4 < 3; ++a4) {
                const int q = 2 * (9 * a1 + 3 * a2 + a4);
                const c64 a = xv[3 * a1 + a4], b = yv[a2];
                v[q] = __builtin_fma(a.x, b.x, v[q]);
                v[q] = __builtin_fma(-a.y, b.y, v[q]);
                v[q + 1] = __builtin_fma(a.x, b.y, v[q + 1]);
                v[q + 1] = __builtin_fma(a.y, b.x, v[q + 1]);
              }
        }
      }
      // 16 lanes add their partial sums by halving: at each step a lane keeps the
      // lower or upper part of its current range (by one lane bit), adds the partner's
      // copy of that part and hands over the other part.  Ranges 54 -> 27 -> 14 -> 7 ->
      // 4 (odd lengths padded by a zero).  The long steps are lane swaps and a row
      // rotation, which leave the LDS pipe to the operands.
      const bool u3 = lane & 32, u2 = lane & 16, u1 = lane & 8, u0 = lane & 4;
#pragma unroll
      for (int k = 0; k < 27; ++k) v[k] = add_swapped<32>(v[k], v[k + 27]);
#pragma unroll
      for (int k = 0; k < 14; ++k) v[k] = add_swapped<16>(v[k], k + 14 < 27 ? v[k + 14] : 0.0);
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        const double lo = v[k], hi = k + 7 < 14 ? v[k + 7] : 0.0;
        v[k] = (u1 ? hi : lo) + from_lane<kRowRotate8>(u1 ? lo : hi);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double lo = v[k], hi = k + 4 < 7 ? v[k + 4] : 0.0;
        v[k] = (u0 ? hi : lo) + __shfl_xor(u0 ? lo : hi, 4, 64);
      }
      if constexpr (PAIR) {
        // lanes of even and odd A hold S0 and S1 of the same outputs
        const double h = t && (o.lambda_neg != o.kappa_neg) ? -0.5 : 0.5;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double w = from_lane<kQuadXor2>(v[k]);
          v[k] = h * (t ? w - v[k] : v[k] + w);
        }
      }
      if (act && !(t && o.out_b == kNoPartner)) {
        // this lane's 4 entries start at 27 u3 + 14 u2 + 7 u1 + 4 u0 of the 54;
        // an entry is real where it lies inside every range it was cut from
        const int o3 = 4 * u0, o2 = 7 * u1 + o3, o1 = 14 * u2 + o2, base = 27 * u3 + o1;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (o3 + k < 7 && o2 + k < 14 && o1 + k < 27) {
            const int q = base + k, jj = q >> 1;  // jj = 9 a1 + 3 a2 + a4
            const int a1 = jj / 9, a2 = jj / 3 % 3, a4 = jj % 3;
            out[2 * (27 * a1 + 9 * a2 + 3 * a3 + a4) + (q & 1)] = v[k];
          }
      }
    }
  }
}

__global__ void __launch_bounds__(kNprThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) npr_kernel(const NprArgs P) {
  // LDS: 74 240 bytes, reused between phases.
  //   phases 1-2: propagators [f][A][9] at 0, steps [A][mu][9] at 576, U (pair layout) at kPairMats
  //   phases 3-4: X (pair layout) at 0, Y (pair layout) at kPairMats
  __shared__ c64 lds[2 * kPairMats];
  c64* Gs = lds;
  c64* Ls = lds + 576;
  c64* Us = lds + kPairMats;
  c64* Xs = lds;
  c64* Ys = lds + kPairMats;

  const int tid = (int)threadIdx.x;
  const long z = (long)blockIdx.x;
  int zc[4];
  {
    long r = z;
    zc[0] = (int)(r % P.hx);
    r /= P.hx;
    zc[1] = (int)(r % P.hy);
    r /= P.hy;
    zc[2] = (int)(r % P.hz);
    zc[3] = (int)(r / P.hz);
  }
  auto lex = [&](int A) -> long {
    const long x = 2 * zc[0] + (A & 1), y = 2 * zc[1] + (A >> 1 & 1);
    const long zz = 2 * zc[2] + (A >> 2 & 1), t = 2 * zc[3] + (A >> 3 & 1);
    return x + P.X * (y + P.Y * (zz + P.Z * t));
  };
  // 1. propagators of the 16 corners (4 x 16 x 9 complex), and the 32 links inside
  //    the hypercube, each stored as the forward step from its lower corner and,
  //    conjugated, as the backward step from its upper corner
  for (int k = tid; k < 576; k += kNprThreads) {
    const int f = k / 144, A = (k / 9) % 16, e = k % 9;
    Gs[k] = P.g[f][lex(A) * 9 + e];
  }
  for (int k = tid; k < 288; k += kNprThreads) {
    const int j = k / 9, e = k % 9;
    const int mu = j >> 3, lo = j & 7;
    const int A = ((lo >> mu) << (mu + 1)) | (lo & ((1 << mu) - 1));  // bit mu clear
    const c64 v = P.thin[(lex(A) * 4 + mu) * 9 + e];
    Ls[(A * 4 + mu) * 9 + e] = v;
    Ls[((A | 1 << mu) * 4 + mu) * 9 + 3 * (e % 3) + e / 3] = make_double2(v.x, -v.y);
  }
  // 2. U_AD for the pair this thread owns, in rounds of growing distance
  const int pr = kPairOrder.p[tid];
  const int A = pr >> 4, D = pr & 15;
  const int d = __popc(A ^ D);
  c64* const umine = Us + A * kRow + 9 * D;
  c64 u[9];
  if (d == 0) {
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = make_double2(e % 4 == 0 ? 1.0 : 0.0, 0.0);
#pragma unroll
    for (int e = 0; e < 9; ++e) umine[e] = u[e];
  }
  __syncthreads();
  if (d == 1) {
    const c64* st = Ls + (A * 4 + (__ffs(A ^ D) - 1)) * 9;
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = st[e];
#pragma unroll
    for (int e = 0; e < 9; ++e) umine[e] = u[e];
  }
  for (int round = 2; round <= 4; ++round) {
    __syncthreads();
    if (d == round) {
      c64 acc[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) acc[e] = make_double2(0.0, 0.0);
      int m = A ^ D;
      for (int q = 0; q < round; ++q) {
        const int mu = __ffs(m) - 1;
        m &= m - 1;
        c64 t[9];
        m3mul(Ls + (A * 4 + mu) * 9, Us + (A ^ 1 << mu) * kRow + 9 * D, t);
#pragma unroll
        for (int e = 0; e < 9; ++e) {
          acc[e].x += t[e].x;
          acc[e].y += t[e].y;
        }
      }
      const double inv = 1.0 / (double)round;
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        u[e] = make_double2(acc[e].x * inv, acc[e].y * inv);
        umine[e] = u[e];
      }
    }
  }
  __syncthreads();
  // 3. the bilinears' colour matrices of the pair (A, D)
  {
    c64 xm[9], ym[9], t[9];
    m3mul_dag(Gs + (0 * 16 + A) * 9, u, t);  // G1(A)^dag U_AD
    m3mul(t, Gs + (3 * 16 + D) * 9, xm);    // ... G4(D)
    m3mul_dag(Gs + (2 * 16 + A) * 9, u, t);  // G3(A)^dag U_AD
    m3mul(t, Gs + (1 * 16 + D) * 9, ym);    // ... G2(D)
    __syncthreads();  // everyone is done with the propagators, steps and U in LDS
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      Xs[A * kRow + 9 * D + e] = xm[e];
      Ys[A * kRow + 9 * D + e] = ym[e];
    }
  }
  __syncthreads();
  // 4. contraction of the operators on their own, then of the pairs on the sums and
  //    differences
  contract<false>(P, z, Xs, Ys);
  if (P.npair > 0) {
    __syncthreads();  // everyone is done with X and Y
    {
      // X+ of the rep (A even, D) at (A, D), X- at (A + 1, D): the thread of (A, D) with
      // A odd belongs to the rep (A - 1, D ^ 1).  Y+ and Y- likewise, by the parity of
      // the second index.
      const int t = A & 1, s = D & 1;
      const int own = A * kRow + 9 * D, other = (A ^ 1) * kRow + 9 * (D ^ 1);
      const double ft = t ? -1.0 : 1.0, fs = s ? -1.0 : 1.0;
      c64 xm[9], ym[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        const c64 x = Xs[other + e], y = Ys[other + e], x0 = Xs[own + e], y0 = Ys[own + e];
        xm[e] = make_double2(x.x + ft * x0.x, x.y + ft * x0.y);
        ym[e] = make_double2(y.x + fs * y0.x, y.y + fs * y0.y);
      }
      __syncthreads();
      c64* xd = Xs + A * kRow + 9 * (D ^ t);
      c64* yd = Ys + (A ^ s) * kRow + 9 * D;
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        xd[e] = xm[e];
        yd[e] = ym[e];
      }
    }
    __syncthreads();
    contract<true>(P, z, Xs, Ys);
  }
}

// gamma_X gamma_Y = sigma(X, Y) gamma_{X ^ Y}: each gamma_nu of Y moves left past
// the gamma_mu of X with mu > nu, each exchange a sign (they anticommute).
int sigma(int X, int Y) {
  int n = 0;
  for (int mu = 0; mu < 4; ++mu)
    for (int nu = 0; nu < mu; ++nu) n += (X >> mu & 1) & (Y >> nu & 1);
  return (n & 1) ? -1 : 1;
}
// gamma_X^dag = reversed product = (-1)^(k(k-1)/2) gamma_X, k = |X|
int rev(int X) {
  const int k = __builtin_popcount(X);
  return ((k * (k - 1) / 2) & 1) ? -1 : 1;
}
int bit(unsigned short m, int k) { return m >> k & 1; }

// f_a(A ^ 1, D ^ 1) / f_a(A, D): sets lambda if it is constant, as the pair form needs.
bool set_lambda(NprOp& a) {
  const int l1 = bit(a.neg1, 0) ^ bit(a.neg1, 1), l2 = bit(a.neg2, a.p2) ^ bit(a.neg2, 1 ^ a.p2);
  for (int k = 0; k < 16; ++k)
    if ((bit(a.neg1, k) ^ bit(a.neg1, k ^ 1)) != l1 || (bit(a.neg2, k ^ a.p2) ^ bit(a.neg2, k ^ 1 ^ a.p2)) != l2)
      return false;
  a.lambda_neg = (unsigned char)(l1 ^ l2);
  return true;
}

// Whether b is the partner of a (see contract): f_b / f_a is constant.  Sets kappa.
bool set_partner(NprOp& a, const NprOp& b) {
  if (b.p1 != (a.p1 ^ 1) || b.p2 != (a.p2 ^ 1)) return false;
  const int k1 = bit(a.neg1, 0) ^ bit(b.neg1, 0), k2 = bit(a.neg2, a.p2) ^ bit(b.neg2, b.p2);
  for (int k = 0; k < 16; ++k)
    if ((bit(a.neg1, k) ^ bit(b.neg1, k)) != k1 || (bit(a.neg2, k ^ a.p2) ^ bit(b.neg2, k ^ b.p2)) != k2) return false;
  a.kappa_neg = (unsigned char)(k1 ^ k2);
  a.out_b = b.out;
  return true;
}

// (1/4) Tr[gamma_A^dag gamma_S gamma_B gamma_F^dag] for B = A ^ S ^ F (the only
// nonzero entry of row A): the product is r(A) r(F) gamma_A gamma_S gamma_B gamma_F,
// which reduces to a sign times gamma_0 = 1.
int spin_taste_sign(int A, int S, int F) {
  const int B = A ^ S ^ F;
  return rev(A) * rev(F) * sigma(A, S) * sigma(A ^ S, B) * sigma(A ^ S ^ B, F);
}

}  // namespace
}  // namespace asq

using namespace asq;

extern "C" int asqtad_npr_fourfermion(const int dims[4], const double* thin_dev, const double* g1_dev,
                                      const double* g2_dev, const double* g3_dev, const double* g4_dev, int nop,
                                      const int* ops_host, double* out_dev, void* hip_stream) {
  const char* who = "asqtad_npr_fourfermion";
  if (!dims || !thin_dev || !g1_dev || !g2_dev || !g3_dev || !g4_dev || !ops_host || !out_dev || nop <= 0) {
    set_last_error(std::string(who) + ": null pointer or nop <= 0");
    return ASQ_EINVAL;
  }
  for (int mu = 0; mu < 4; ++mu)
    if (dims[mu] < 2 || (dims[mu] & 1) || dims[mu] > (1 << 14)) {
      set_last_error(std::string(who) + ": extents must be even, 2 .. 16384");
      return ASQ_EINVAL;
    }
  for (int k = 0; k < 4 * nop; ++k)
    if (ops_host[k] < 0 || ops_host[k] > 15) {
      set_last_error(std::string(who) + ": spin and taste labels are 4-bit masks (0 .. 15)");
      return ASQ_EINVAL;
    }
  const uintptr_t al = (uintptr_t)thin_dev | (uintptr_t)g1_dev | (uintptr_t)g2_dev | (uintptr_t)g3_dev |
                       (uintptr_t)g4_dev | (uintptr_t)out_dev;
  if (al & 15) {
    set_last_error(std::string(who) + ": links, propagators and output must be 16-byte aligned");
    return ASQ_EINVAL;
  }
  const long V = (long)dims[0] * dims[1] * dims[2] * dims[3];
  const long nz = V / 16;
  if (nz >= (1L << 31)) {
    set_last_error(std::string(who) + ": lattice too large");
    return ASQ_EINVAL;
  }
  // the output may not overlap an input
  const size_t ob = (size_t)nop * nz * 81 * 16;
  const void* ins[5] = {thin_dev, g1_dev, g2_dev, g3_dev, g4_dev};
  const size_t ib[5] = {(size_t)V * 4 * 9 * 16, (size_t)V * 9 * 16, (size_t)V * 9 * 16, (size_t)V * 9 * 16,
                        (size_t)V * 9 * 16};
  for (int k = 0; k < 5; ++k) {
    const uintptr_t a = (uintptr_t)ins[k], o = (uintptr_t)out_dev;
    if (o < a + ib[k] && a < o + ob) {
      set_last_error(std::string(who) + ": the output must not overlap the links or propagators");
      return ASQ_EINVAL;
    }
  }
  NprArgs P;
  memset(&P, 0, sizeof(P));
  P.X = dims[0];
  P.Y = dims[1];
  P.Z = dims[2];
  P.T = dims[3];
  P.hx = dims[0] / 2;
  P.hy = dims[1] / 2;
  P.hz = dims[2] / 2;
  P.thin = (const double2*)thin_dev;
  P.g[0] = (const double2*)g1_dev;
  P.g[1] = (const double2*)g2_dev;
  P.g[2] = (const double2*)g3_dev;
  P.g[3] = (const double2*)g4_dev;
  P.out = (double2*)out_dev;
  P.nz = nz;
  hipStream_t s = (hipStream_t)hip_stream;
  for (int op0 = 0; op0 < nop; op0 += kNprOpsPerLaunch) {
    P.op0 = op0;
    const int n = nop - op0 < kNprOpsPerLaunch ? nop - op0 : kNprOpsPerLaunch;
    NprOp all[kNprOpsPerLaunch];
    for (int k = 0; k < n; ++k) {
      const int* o = ops_host + 4 * (op0 + k);
      NprOp& q = all[k];
      q = NprOp{};
      q.p1 = (unsigned char)(o[0] ^ o[1]);
      q.p2 = (unsigned char)(o[2] ^ o[3]);
      q.out = (unsigned char)k;
      for (int A = 0; A < 16; ++A) {
        // eps(z_A) = (-1)^|A|: the hypercube origin 2z has even coordinates
        const int eps = (__builtin_popcount(A) & 1) ? -1 : 1;
        if (spin_taste_sign(A, o[0], o[1]) * eps < 0) q.neg1 |= (unsigned short)(1u << A);
        if (spin_taste_sign(A, o[2], o[3]) * eps < 0) q.neg2 |= (unsigned short)(1u << A);
      }
    }
    // Each operator joins the first later one that is its partner.  The pair form
    // sums an operator without a partner in a slot of its own, for what it costs in
    // the single form plus half an exchange.
    NprOp slots[kNprOpsPerLaunch], rest[kNprOpsPerLaunch];
    bool used[kNprOpsPerLaunch] = {};
    int ns = 0, npair = 0, nrest = 0;
    for (int k = 0; k < n; ++k) {
      if (used[k]) continue;
      NprOp a = all[k];
      a.out_b = kNoPartner;
      if (!set_lambda(a)) {
        rest[nrest++] = a;
        continue;
      }
      for (int j = k + 1; j < n; ++j)
        if (!used[j] && set_partner(a, all[j])) {
          used[j] = true;
          ++npair;
          break;
        }
      slots[ns++] = a;
    }
    // a pass of 8 slots of the pair form takes 0.6 of one of 16 operators of the single
    // form (half the products, the same exchanges)
    const int by_slots = 6 * ((ns + kNprPairsPerPass - 1) / kNprPairsPerPass);
    const int by_ops = 10 * ((ns + npair + kNprOpsPerPass - 1) / kNprOpsPerPass);
    P.nsingle = P.npair = 0;
    if (by_slots < by_ops) {
      for (int k = 0; k < nrest; ++k) P.ops[P.nsingle++] = rest[k];
      for (int k = 0; k < ns; ++k) P.ops[P.nsingle + P.npair++] = slots[k];
    } else {
      for (int k = 0; k < n; ++k) P.ops[P.nsingle++] = all[k];
    }
    npr_kernel<<<(unsigned)nz, kNprThreads, 0, s>>>(P);
    ASQ_HIP_TRY(hipGetLastError());
  }
  return ASQ_OK;
}
