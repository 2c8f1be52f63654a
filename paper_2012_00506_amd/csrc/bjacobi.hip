// Parallel two-sided block Jacobi for the reduced Hermitian eigenproblems of
// the Rayleigh-Ritz step (Algorithm alg:FEAST: A_q W = W Lambda) and the
// Gram matrices of the eigen-decomposition orthonormalisation, for matrices
// too large for the one-workgroup Jacobi.
//
// The matrix is padded to mp = 64 h columns (the padding decoupled with a
// huge diagonal, so that it sorts last and is never rotated) and split into
// 2h blocks of 32 columns.  Blocks are kept in a physical order in which
// round r pairs positions (2k, 2k+1): one round
//  1. diagonalises every 64 x 64 principal block A[K, K] of pair K by a
//     cyclic Jacobi in LDS, giving a unitary U_K (k_bj_pairs);
//  2. forms A[K, L] <- U_K^H A[K, L] U_L for every pair of pairs and
//     V[:, L] <- V[:, L] U_L as two 64 x 64 x 64 complex products on FP64
//     MFMA per tile (k_bj_update), writing every 32-row/column block to its
//     position for the next round.
// Positions move between rounds as in the round-robin (circle) schedule:
// position 0 stays, the others advance one step around the ring
// 2, 4, ..., 2h-2, 2h-1, 2h-3, ..., 3, 1, so that over 2h - 1 rounds every
// two blocks share a pair once (one sweep).  Sweeps repeat until the
// off-diagonal part of A is below tol times its norm.
#include <math.h>

#include <algorithm>
#include <vector>

#include "prof.h"
#include "rr.h"

namespace fb {

static constexpr int kBs = 32;        // columns per block
static constexpr int kPb = 2 * kBs;   // columns per pair
static constexpr int kPL = kPb + 1;   // padded column length in LDS
static constexpr double kPad = 1e20;  // diagonal of the padding

struct BJDev {  // kBjDescBytes bytes
  c128* A[2];   // mp x mp, ld = mp (current / next)
  c128* V[2];   // mp x mp
  c128* U;      // h x 64 x 64, row-major per pair: U[K][k * 64 + j] = U_K(k, j)
  int32_t* skip;// h: U of the pair is the identity
  double* part; // 2 doubles per column of A: off^2 and total^2 partial sums
  int32_t m, mp, h, cplx;  // cplx: an imaginary part is set in A
};

typedef double bd4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bd4 bj_mfma(double a, double b, bd4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// position of a block's content in the next round
__device__ __forceinline__ int bj_next(int pos, int h) {
  if (h == 1 || pos == 0) return pos;
  if ((pos & 1) == 0) {                       // top row, k = pos / 2 >= 1
    const int k = pos >> 1;
    return k < h - 1 ? pos + 2 : pos + 1;     // last top goes to the last bottom
  }
  const int k = pos >> 1;                     // bottom row
  return k >= 1 ? pos - 2 : 2;                // first bottom goes to top 1
}

// -------------------------------------------------------------- pad / init
__global__ void k_bj_init(const JacobiJob* __restrict__ jobs, BJDev* __restrict__ dv) {
  const JacobiJob jb = jobs[blockIdx.y];
  const BJDev d = dv[blockIdx.y];
  const int64_t tot = (int64_t)d.mp * d.mp;
  bool imag = false;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(e / d.mp), i = (int)(e - (int64_t)j * d.mp);
    c128 a = mk(0.0, 0.0);
    if (i < d.m && j < d.m)
      a = gld(jb.A + (int64_t)j * jb.lda + i);
    else if (i == j)
      a = mk(kPad, 0.0);
    gst(d.A[0] + e, a);
    gst(d.V[0] + e, mk(i == j ? 1.0 : 0.0, 0.0));
    imag |= a.y != 0.0;
  }
  if (__syncthreads_or(imag) && threadIdx.x == 0) atomicOr(&dv[blockIdx.y].cplx, 1);
}

// -------------------------------------------------------------- off-norm
// padding columns and rows (diagonal kPad) are left out
__global__ void __launch_bounds__(256) k_bj_norms(BJDev* __restrict__ dv, int cur) {
  const BJDev d = dv[blockIdx.y];
  const int j = blockIdx.x;
  if (j >= d.mp) return;
  const c128* A = (cur ? d.A[1] : d.A[0]);
  __shared__ double r0[256], r1[256];
  double off = 0.0, all = 0.0;
  const bool padj = gld(A + (int64_t)j * d.mp + j).x > 0.5 * kPad;
  if (!padj) {
    for (int i = threadIdx.x; i < d.mp; i += blockDim.x) {
      if (gld(A + (int64_t)i * d.mp + i).x > 0.5 * kPad) continue;
      double a = cabs2(gld(A + (int64_t)j * d.mp + i));
      all += a;
      if (i != j) off += a;
    }
  }
  r0[threadIdx.x] = off;
  r1[threadIdx.x] = all;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      r0[threadIdx.x] += r0[threadIdx.x + s];
      r1[threadIdx.x] += r1[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    gst(d.part + 2 * j, r0[0]);
    gst(d.part + 2 * j + 1, r1[0]);
  }
}

// one workgroup per matrix: the columns' sums through LDS, added in order
__global__ void __launch_bounds__(256) k_bj_norms_final(BJDev* __restrict__ dv,
                                                        double* __restrict__ out) {
  __shared__ double part[2][256];
  const BJDev d = dv[blockIdx.x];
  const int t = threadIdx.x;
  double sum = 0.0;
  for (int j0 = 0; j0 < d.mp; j0 += 256) {
    const int nj = min(256, d.mp - j0);
    if (t < nj) {
      part[0][t] = gld(d.part + 2 * (j0 + t));
      part[1][t] = gld(d.part + 2 * (j0 + t) + 1);
    }
    __syncthreads();
    if (t < 2)
#pragma unroll 8
      for (int j = 0; j < nj; ++j) sum += part[t][j];
    __syncthreads();
  }
  if (t < 2) out[2 * blockIdx.x + t] = sum;
}

// -------------------------------------------------------------- pair solves
// One workgroup per (pair, matrix): one cyclic Jacobi sweep on the 64 x 64
// principal block (none once it is diagonal), accumulating U.  A second inner
// sweep makes U more exact but buys few outer sweeps: on the benchmark's
// reduced matrices (m = 1 346..1 551) one inner sweep took 43 outer sweeps
// against 40 in 1.9 s against 2.3 s.
static constexpr int kInner = 1;
static constexpr int kPairThreads = 1024;  // one 2 x 2 block update per thread per round

// Rotation of one pair: columns p, q are turned by J = [cs sn; -e sn  e cs].
struct alignas(16) BJRot {
  double cs, sn;
  c128 e;
};
// position's pair in the round: positions k and kPb - 1 - k play each other
__device__ __forceinline__ int bj_pair(int pos) { return pos < kBs ? pos : kPb - 1 - pos; }

// Elements of the pair problem: complex, or real where no imaginary part is
// set (a real matrix: the same operations without the terms that are zero).
template <bool CPLX>
struct BJElem;
template <>
struct BJElem<true> {
  using E = c128;
  static __device__ __forceinline__ E from(c128 v) { return v; }
  static __device__ __forceinline__ c128 to(E v) { return v; }
  static __device__ __forceinline__ double norm2(E v) { return cabs2(v); }
  static __device__ __forceinline__ double re(E v) { return v.x; }
  static __device__ __forceinline__ double im(E v) { return v.y; }
  // e v (in S and in U: the two round their imaginary parts in another
  // order), conj(e) v
  static __device__ __forceinline__ E mul(c128 e, E v) {
    return mk(fma(e.x, v.x, -(e.y * v.y)), fma(v.y, e.x, v.x * e.y));
  }
  static __device__ __forceinline__ E mulu(c128 e, E v) {
    return mk(fma(e.x, v.x, -(e.y * v.y)), fma(e.y, v.x, v.y * e.x));
  }
  static __device__ __forceinline__ E mulc(c128 e, E v) {
    return mk(fma(e.x, v.x, e.y * v.y), fma(e.x, v.y, -(e.y * v.x)));
  }
  // c a - s b, s a + c b
  static __device__ __forceinline__ E minus(double c, E a, double s, E b) {
    return mk(fma(c, a.x, -(s * b.x)), fma(c, a.y, -(s * b.y)));
  }
  static __device__ __forceinline__ E plus(double s, E a, double c, E b) {
    return mk(fma(s, a.x, c * b.x), fma(s, a.y, c * b.y));
  }
};
template <>
struct BJElem<false> {
  using E = double;
  static __device__ __forceinline__ E from(c128 v) { return v.x; }
  static __device__ __forceinline__ c128 to(E v) { return mk(v, 0.0); }
  static __device__ __forceinline__ double norm2(E v) { return v * v; }
  static __device__ __forceinline__ double re(E v) { return v; }
  static __device__ __forceinline__ double im(E) { return 0.0; }
  static __device__ __forceinline__ E mul(c128 e, E v) { return e.x * v; }
  static __device__ __forceinline__ E mulu(c128 e, E v) { return e.x * v; }
  static __device__ __forceinline__ E mulc(c128 e, E v) { return e.x * v; }
  static __device__ __forceinline__ E minus(double c, E a, double s, E b) {
    return fma(c, a, -(s * b));
  }
  static __device__ __forceinline__ E plus(double s, E a, double c, E b) {
    return fma(s, a, c * b);
  }
};

// A round has one barrier: wave 0 updates the 64 2 x 2 blocks of S that the
// next round's rotations are formed from (the diagonal ones and, for every
// next pair, the one that holds its off-diagonal element) and goes on to form
// them, while the other 15 waves update the 960 blocks left, one per thread,
// and turn U.
// What bounds it: the angles' chain of divisions and square roots on one
// wave, and in complex arithmetic the LDS traffic of S and U beside it.  With
// all waves waiting for the angles and two barriers a launch of 63 rounds took
// 147 us, real or complex; now, with U shared out over four workgroups, 95 us
// complex (20 pairs) and 72 us real (122 and 87 us in one workgroup).
template <bool CPLX, bool SPLIT>
__device__ __forceinline__ int bj_pair_sweeps(char* lds, BJRot (*rot)[kBs],
                                              double (*red)[kPairThreads],
                                              const c128* __restrict__ A, int64_t base, int mp,
                                              c128* __restrict__ U, int part, int rlog) {
  using X = BJElem<CPLX>;
  using E = typename X::E;
  E* S = reinterpret_cast<E*>(lds);  // column-major, ld kPL
  E* Us = S + kPb * kPL;             // column-major, ld kPL
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  for (int e = t; e < kPb * kPb; e += kPairThreads) {
    const int cj = e / kPb, ci = e % kPb;
    S[cj * kPL + ci] = X::from(gld(A + (base + cj) * mp + base + ci));
    Us[cj * kPL + ci] = X::from(mk(ci == cj ? 1.0 : 0.0, 0.0));
  }
  __syncthreads();
  // the player at position pos in round r, r <= kPb - 2
  auto player = [](int pos, int r) {
    int v = pos + r;
    v = v >= kPb ? v - (kPb - 1) : v;
    return pos == 0 ? 0 : v;
  };
  // rotations of round ro by one wave: lanes k and k + 32 take pair k, the
  // first its angle, the second its phase
  auto angles = [&](int ro, BJRot* o) {
    const int k = lane & 31;
    const bool second = lane >= 32;
    const int a = player(k, ro), b = player(kPb - 1 - k, ro);
    const int p = a < b ? a : b, q = a < b ? b : a;
    const E c = S[q * kPL + p];
    const double ac = sqrt(X::norm2(c));
    const double app = X::re(S[p * kPL + p]), aqq = X::re(S[q * kPL + q]);
    const bool turn = ac > 1e-300 && ac > 1e-18 * (fabs(app) + fabs(aqq));
    const double x = (second ? X::re(c) : aqq - app) / (second ? ac : 2.0 * ac);  // tau
    const double y = (second ? -X::im(c) : x >= 0.0 ? 1.0 : -1.0) /
                     (second ? ac : fabs(x) + hypot(1.0, x));                     // tan
    const double cs = 1.0 / sqrt(1.0 + y * y), sn = y * cs;
    BJRot* at = o + k;
    if (second)
      at->e = turn ? mk(x, y) : mk(1.0, 0.0);  // e^{-i arg c}
    else
      *reinterpret_cast<c128*>(at) = turn ? mk(cs, sn) : mk(1.0, 0.0);
  };
  // S <- J^H S J on one 2 x 2 block: rows of pair kk, columns of pair ll
  auto block = [&](const BJRot* o, int ro, int kk, int ll) {
    const int ak = player(kk, ro), bk = player(kPb - 1 - kk, ro);
    const int al = player(ll, ro), bl = player(kPb - 1 - ll, ro);
    const int pk = min(ak, bk), qk = max(ak, bk), pl = min(al, bl), ql = max(al, bl);
    const BJRot rk = o[kk], rl = o[ll];
    const E a00 = S[pl * kPL + pk], a10 = S[pl * kPL + qk];
    const E a01 = X::mul(rl.e, S[ql * kPL + pk]), a11 = X::mul(rl.e, S[ql * kPL + qk]);
    const E b00 = X::minus(rl.cs, a00, rl.sn, a01), b01 = X::plus(rl.sn, a00, rl.cs, a01);
    const E b10 = X::mulc(rk.e, X::minus(rl.cs, a10, rl.sn, a11));
    const E b11 = X::mulc(rk.e, X::plus(rl.sn, a10, rl.cs, a11));
    S[pl * kPL + pk] = X::minus(rk.cs, b00, rk.sn, b10);
    S[pl * kPL + qk] = X::plus(rk.sn, b00, rk.cs, b10);
    S[ql * kPL + pk] = X::minus(rk.cs, b01, rk.sn, b11);
    S[ql * kPL + qk] = X::plus(rk.sn, b01, rk.cs, b11);
  };
  // Pair j of the next round is made of the players at positions j + 1 and
  // kPb - j (0 and 1 for j = 0), which play in pairs xj and yj of this one:
  // every pair k meets two others, k - 2 and k + 2 (0 also 1, kBs - 1 also
  // kBs - 2).  Threads of wave 0 from 32 on take the block whose row holds the
  // lower player, the last 32 threads its mirror image; the other threads take
  // the remaining off-diagonal blocks, 29 to a pair ll.
  const int g = t - 64, j = w == 0 ? lane & 31 : g - 29 * kBs;
  const bool meet = w == 0 ? lane >= 32 : j >= 0;
  const int posx = j == 0 ? 0 : j + 1, posy = j == 0 ? 1 : kPb - j;
  int kk = lane & 31, ll = kk;
  if (w != 0 && !meet) {
    ll = g / 29;
    const int e0 = ll == 1 ? 0 : ll == 0 ? 0 : ll - 2;
    const int e1 = ll == 0 ? 1 : ll == 1 ? 1 : ll == kBs - 1 ? kBs - 2 : ll;
    const int e2 = ll == 0 ? 2 : ll == 1 ? 3 : ll >= kBs - 2 ? kBs - 1 : ll + 2;
    kk = g - 29 * ll;
    kk += kk >= e0 ? 1 : 0;
    kk += kk >= e1 ? 1 : 0;
    kk += kk >= e2 ? 1 : 0;
  }
  const int urow = SPLIT ? (part << rlog) + (lane & ((1 << rlog) - 1)) : lane;
  // wave 0 is the one that the others wait for
  if (w == 0) __builtin_amdgcn_s_setprio(3);
  int rotated = 0;
  for (int sw = 0; sw < kInner; ++sw) {
    // stop when the block is diagonal relative to its (non-padding) diagonal
    double off = 0.0, dg = 0.0;
    for (int e = t; e < kPb * kPb; e += kPairThreads) {
      const int cj = e / kPb, ci = e % kPb;
      const E v = S[cj * kPL + ci];
      if (ci != cj) off += X::norm2(v);
      else dg += fabs(X::re(v)) < 0.5 * kPad ? X::norm2(v) : 0.0;
    }
    red[0][t] = off;
    red[1][t] = dg;
    __syncthreads();
    for (int s = kPairThreads / 2; s > 0; s >>= 1) {
      if (t < s) {
        red[0][t] += red[0][t + s];
        red[1][t] += red[1][t + s];
      }
      __syncthreads();
    }
    const bool diag = !(red[0][0] > 1e-32 * red[1][0]);
    __syncthreads();
    if (diag) break;  // uniform: every thread read the same sums
    rotated = 1;
    if (w == 0) angles(0, rot[0]);
    __syncthreads();
    for (int ro = 0; ro < kPb - 1; ++ro) {
      const BJRot* o = rot[ro & 1];
      if (meet) {
        const int x = bj_pair(posx), y = bj_pair(posy);
        const bool low = (player(posx, ro) < player(posy, ro)) == (w == 0);
        kk = low ? x : y;
        ll = low ? y : x;
      }
      block(o, ro, kk, ll);
      if (w == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (ro + 2 < kPb) angles(ro + 1, rot[(ro & 1) ^ 1]);
      } else {
        // U <- U J (columns p, q), a lane per row of U and pair
        const int step = SPLIT ? 64 >> rlog : 1;  // pairs per wave
        for (int k = (w - 1) * step + (SPLIT ? lane >> rlog : 0); k < kBs;
             k += (kPairThreads / 64 - 1) * step) {
          const int a = player(k, ro), b = player(kPb - 1 - k, ro);
          const int p = min(a, b), q = max(a, b);
          const BJRot r = o[k];
          const E vp = Us[p * kPL + urow], vq = X::mulu(r.e, Us[q * kPL + urow]);
          Us[p * kPL + urow] = X::minus(r.cs, vp, r.sn, vq);
          Us[q * kPL + urow] = X::plus(r.sn, vp, r.cs, vq);
        }
      }
      __syncthreads();
    }
  }
  if (w == 0) __builtin_amdgcn_s_setprio(0);
  const int e1 = SPLIT ? kPb << rlog : kPb * kPb;
  for (int e = t; e < e1; e += kPairThreads) {
    const int k = (SPLIT ? part << rlog : 0) + e / kPb, jc = e % kPb;  // row-major
    gst(U + k * kPb + jc, X::to(Us[jc * kPL + k]));
  }
  return rotated;
}

// Workgroup (K 2^(6 - rlog) + part, matrix): pair K, and of its U the rows
// 2^rlog part .. 2^rlog (part + 1) - 1.  The workgroups of a pair repeat the
// same rotations of S, each for its own rows of U.
__global__ void __launch_bounds__(kPairThreads) k_bj_pairs(BJDev* __restrict__ dv, int cur,
                                                           int rlog) {
  extern __shared__ __align__(16) char lds_raw[];
  __shared__ BJRot rot[2][kBs];
  __shared__ double red[2][kPairThreads];
  const BJDev d = dv[blockIdx.y];
  const int K = blockIdx.x >> (6 - rlog), part = blockIdx.x & ((64 >> rlog) - 1);
  if (K >= d.h) return;
  const int t = threadIdx.x;
  const c128* A = (cur ? d.A[1] : d.A[0]);
  const int64_t base = (int64_t)K * kPb;
  bool imag = false;
  for (int e = t; d.cplx && e < kPb * kPb; e += kPairThreads)
    imag |= gld(A + (base + e / kPb) * d.mp + base + e % kPb).y != 0.0;
  c128* U = d.U + (size_t)K * kPb * kPb;
  const bool cplx = __syncthreads_or(imag);
  int rotated;
  if (rlog == 6)
    rotated = cplx ? bj_pair_sweeps<true, false>(lds_raw, rot, red, A, base, d.mp, U, 0, 6)
                   : bj_pair_sweeps<false, false>(lds_raw, rot, red, A, base, d.mp, U, 0, 6);
  else
    rotated = cplx ? bj_pair_sweeps<true, true>(lds_raw, rot, red, A, base, d.mp, U, part, rlog)
                   : bj_pair_sweeps<false, true>(lds_raw, rot, red, A, base, d.mp, U, part, rlog);
  if (t == 0 && part == 0) gst(d.skip + K, rotated ? 0 : 1);
}

// -------------------------------------------------------------- updates
// Workgroups 0 .. h(h+1)/2-1 of a matrix: the tiles (K, L), K <= L, of A,
// R = U_K^H A[K,L] U_L (R^H is the tile (L, K): A stays Hermitian);
// workgroups from h(h+1)/2 on: the tiles (I, L) of V, V[I, L] U_L.  Each
// 32-row and 32-column block of the result is written to its next-round
// position.  The columns of a tile are independent: CS workgroups take 64 /
// CS of them each.  Four waves share them, RT x CT MFMA tiles of 16 x 16 per
// wave (Gauss form; a real matrix takes the first of its three products, the
// second is zero and the third equal to the first); operand fragments are
// loaded one contraction step ahead.
// What bounds it: the latency of the two dependent products of an A tile, at
// the few tiles that a call has for 256 CUs.  Whole tiles took 35 us per launch
// for two complex matrices of 640 columns and 28 us for a real one of 320; now
// 20 (CS = 2) and 11 us (CS = 4); sixteen of 1500, whole tiles, 740 -> 620 us.
template <bool CONJA, bool CPLX, int RT, int CT, typename FA, typename FB>
__device__ __forceinline__ void bj_products(bd4 (&p1)[RT][CT], bd4 (&p2)[RT][CT],
                                            bd4 (&p3)[RT][CT], FA fa, FB fb, int lk) {
#pragma unroll
  for (int a = 0; a < RT; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) p1[a][b][r] = p2[a][b][r] = p3[a][b][r] = 0.0;
  c128 an[RT], bn[CT];
#pragma unroll
  for (int q = 0; q < RT; ++q) an[q] = fa(q, lk);
#pragma unroll
  for (int q = 0; q < CT; ++q) bn[q] = fb(q, lk);
#pragma unroll 2
  for (int kk = 0; kk < kPb; kk += 4) {
    double ar[RT], ai[RT], as[RT], br[CT], bi[CT], bs[CT];
#pragma unroll
    for (int q = 0; q < RT; ++q) {
      ar[q] = an[q].x;
      ai[q] = CONJA ? -an[q].y : an[q].y;
      as[q] = ar[q] + ai[q];
    }
#pragma unroll
    for (int q = 0; q < CT; ++q) {
      br[q] = bn[q].x;
      bi[q] = bn[q].y;
      bs[q] = bn[q].x + bn[q].y;
    }
    if (kk + 4 < kPb) {
#pragma unroll
      for (int q = 0; q < RT; ++q) an[q] = fa(q, kk + 4 + lk);
#pragma unroll
      for (int q = 0; q < CT; ++q) bn[q] = fb(q, kk + 4 + lk);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        p1[rt][ct] = bj_mfma(ar[rt], br[ct], p1[rt][ct]);
        if (CPLX) {
          p2[rt][ct] = bj_mfma(ai[rt], bi[ct], p2[rt][ct]);
          p3[rt][ct] = bj_mfma(as[rt], bs[ct], p3[rt][ct]);
        }
      }
  }
}

template <bool CPLX, int CS>
__device__ __forceinline__ void bj_update_part(const c128* As, c128* Ad, const c128* Vs, c128* Vd,
                                               const c128* U, const int32_t* skip, int mp, int h,
                                               c128* Ts, int wg, int part) {
  constexpr int RT = CS == 1 ? 2 : 1, CT = CS == 4 ? 1 : 2;
  constexpr int NCOL = kPb / CS;
  const int nA = h * (h + 1) / 2;
  const bool isA = wg < nA;
  int K, L;
  if (isA) {  // wg -> (K, L), K <= L, row by row
    K = 0;
    int off = 0;
    while (off + (h - K) <= wg) {
      off += h - K;
      ++K;
    }
    L = K + (wg - off);
  } else {
    K = (wg - nA) / h;  // row tile of V
    L = (wg - nA) % h;
  }
  const c128* Src = isA ? As : Vs;
  c128* Dst = isA ? Ad : Vd;
  const int64_t ld = mp;
  const int64_t r0 = (int64_t)K * kPb, c0 = (int64_t)L * kPb;
  const int skK = isA ? gld(skip + K) : 1, skL = gld(skip + L);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int j0 = NCOL * part;  // the workgroup's columns of the tile
  // the wave's rows and, within those columns, columns
  const int wr = 16 * RT * (CS == 1 ? w & 1 : w), wc = CS == 1 ? 32 * (w >> 1) : 0;
  const int li = lane & 15, lk = lane >> 4;
  const c128* UL = U + (size_t)L * kPb * kPb + j0;
  const c128* UK = U + (size_t)K * kPb * kPb;
  bd4 p1[RT][CT], p2[RT][CT], p3[RT][CT];
  auto to_lds = [&]() {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = wr + 16 * rt + lk + 4 * r, j = wc + 16 * ct + li;
          const double x1 = p1[rt][ct][r], x2 = p2[rt][ct][r], x3 = p3[rt][ct][r];
          Ts[j * kPL + i] = CPLX ? mk(x1 - x2, x3 - x1 - x2) : mk(x1, 0.0);
        }
  };

  if (skL) {  // no product on the right: the tile itself
    for (int e = t; e < kPb * NCOL; e += 256) {
      const int j = e / kPb, i = e % kPb;
      Ts[j * kPL + i] = gld(Src + (c0 + j0 + j) * ld + r0 + i);
    }
  } else {  // T = Src[K, L] U_L
    bj_products<false, CPLX, RT, CT>(
        p1, p2, p3, [&](int q, int k) { return gld(Src + (c0 + k) * ld + r0 + wr + 16 * q + li); },
        [&](int q, int k) { return gld(UL + k * kPb + wc + 16 * q + li); }, lk);
    to_lds();
  }
  __syncthreads();
  if (!skK) {  // R = U_K^H T
    bj_products<true, CPLX, RT, CT>(
        p1, p2, p3, [&](int q, int k) { return gld(UK + k * kPb + wr + 16 * q + li); },
        [&](int q, int k) {
          const c128* v = Ts + (wc + 16 * q + li) * kPL + k;
          return mk(v->x, v->y);
        },
        lk);
    __syncthreads();  // every wave has read T
    to_lds();
    __syncthreads();
  }
  // write out: rows of an A tile move with their blocks, V rows stay; an
  // off-diagonal A tile also gives its conjugate transpose
  for (int e = t; e < kPb * NCOL; e += 256) {
    const int j = e / kPb, i = e % kPb, jt = j0 + j;
    const int64_t gr = isA ? (int64_t)bj_next(2 * K + i / kBs, h) * kBs + i % kBs : r0 + i;
    const int64_t gc = (int64_t)bj_next(2 * L + jt / kBs, h) * kBs + jt % kBs;
    gst(Dst + gc * ld + gr, Ts[j * kPL + i]);
  }
  if (isA && K != L) {
    for (int e = t; e < kPb * NCOL; e += 256) {
      const int i = e / NCOL, j = e % NCOL, jt = j0 + j;  // conj(R(i, jt)) to (row of jt, column of i)
      const int64_t gr = (int64_t)bj_next(2 * L + jt / kBs, h) * kBs + jt % kBs;
      const int64_t gc = (int64_t)bj_next(2 * K + i / kBs, h) * kBs + i % kBs;
      gst(Dst + gc * ld + gr, cconj(Ts[j * kPL + i]));
    }
  }
}

template <int CS>
__global__ void __launch_bounds__(256, 2) k_bj_update(BJDev* __restrict__ dv, int cur) {
  extern __shared__ __align__(16) char lds_raw[];
  c128* Ts = reinterpret_cast<c128*>(lds_raw);  // 64 x (64 / CS), column-major, ld kPL
  const BJDev* d = dv + blockIdx.y;
  const int wg = blockIdx.x / CS, part = blockIdx.x % CS;
  const int h = d->h, mp = d->mp;
  if (wg >= h * (h + 1) / 2 + h * (mp / kPb)) return;
  // (by constant members: an indexed member array would live in scratch)
  c128 *A0 = d->A[0], *A1 = d->A[1], *V0 = d->V[0], *V1 = d->V[1];
  const c128 *As = cur ? A1 : A0, *Vs = cur ? V1 : V0;
  c128 *Ad = cur ? A0 : A1, *Vd = cur ? V0 : V1;
  if (d->cplx)
    bj_update_part<true, CS>(As, Ad, Vs, Vd, d->U, d->skip, mp, h, Ts, wg, part);
  else
    bj_update_part<false, CS>(As, Ad, Vs, Vd, d->U, d->skip, mp, h, Ts, wg, part);
}

// -------------------------------------------------------------- results
// eigenvalues ascending (rank by value, ties by position; the padding ranks
// last) and the matching columns of V (first m rows) into the job's outputs
__global__ void k_bj_rank(const JacobiJob* __restrict__ jobs, BJDev* __restrict__ dv, int cur) {
  const JacobiJob jb = jobs[blockIdx.y];
  const BJDev d = dv[blockIdx.y];
  const c128* A = (cur ? d.A[1] : d.A[0]);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.mp) return;
  const double wi = gld(A + (int64_t)i * d.mp + i).x, ki = rank_key(wi);
  int rank = 0;
  for (int j = 0; j < d.mp; ++j) {
    const double wj = rank_key(gld(A + (int64_t)j * d.mp + j).x);
    rank += (wj < ki || (wj == ki && j < i)) ? 1 : 0;
  }
  if (rank < d.m) {
    gst(jb.w + rank, wi);
    gst(jb.order + rank, i);
  }
}

__global__ void k_bj_vectors(const JacobiJob* __restrict__ jobs, BJDev* __restrict__ dv,
                             int cur) {
  const JacobiJob jb = jobs[blockIdx.y];
  const BJDev d = dv[blockIdx.y];
  const c128* V = (cur ? d.V[1] : d.V[0]);
  const int64_t tot = (int64_t)d.m * d.m;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(e / d.m), i = (int)(e - (int64_t)k * d.m);
    const int src = gld(jb.order + k);
    gst(jb.W + (int64_t)k * jb.ldw + i, gld(V + (int64_t)src * d.mp + i));
  }
}

// -------------------------------------------------------------- medium sizes
// The cyclic Jacobi of k_jacobi, the same rotations and arithmetic, with a
// launch per round: a workgroup takes 16 x 16 of the round's 2 x 2 blocks, or
// 16 pairs of 64 rows of V, and forms the rotations of its own pairs from the
// last round's matrix.  Rounds go from A to W and back (W is written last).
// What bounds it: the launches' latency, about 5 us per round, where one
// workgroup moved A and V through one CU.  A Rayleigh-Ritz step with m = 128
// 15.8 -> 6.4 ms, m = 250 99 -> 12.8 ms, eight of m = 200 54 -> 16 ms.
// JacobiJob.pad_: 2 * sweeps made, + 1 when converged.
static constexpr int kJrPairs = 16;   // pairs of a workgroup's tile
static constexpr int kJrRows = 64;    // rows of V per workgroup

__device__ __forceinline__ int jr_player(int pos, int r, int mp) {
  int v = pos + r;
  v = v >= mp ? v - (mp - 1) : v;
  return pos == 0 ? 0 : v;
}

__global__ void __launch_bounds__(1024) k_jr_norms(JacobiJob* __restrict__ jobs, int sweep,
                                                   double tol) {
  __shared__ double red[2][1024];
  const JacobiJob jb = jobs[blockIdx.x];
  const int m = jb.m, t = threadIdx.x;
  if (m <= 0 || (jb.pad_ & 1)) return;
  const int mp = m + (m & 1);
  const bool odd = (sweep * (mp - 1)) & 1;
  const c128* A = odd ? jb.W : jb.A;
  const int64_t lda = odd ? jb.ldw : jb.lda;
  if (sweep == 0)
    for (int64_t e = t; e < (int64_t)m * m; e += 1024) {
      const int j = (int)(e / m), i = (int)(e - (int64_t)j * m);
      gst(jb.V + (int64_t)j * jb.ldv + i, mk(i == j ? 1.0 : 0.0, 0.0));
    }
  double f = 0.0, o = 0.0;
  for (int64_t e = t; e < (int64_t)m * m; e += 1024) {
    const int j = (int)(e / m), i = (int)(e - (int64_t)j * m);
    const double a = cabs2(gld(A + (int64_t)j * lda + i));
    f += a;
    if (i != j) o += a;
  }
  red[0][t] = f;
  red[1][t] = o;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (t < s) {
      red[0][t] += red[0][t + s];
      red[1][t] += red[1][t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    const bool done = red[1][0] <= tol * tol * red[0][0] || m == 1;
    jobs[blockIdx.x].pad_ = done ? 2 * sweep + 1 : 2 * (sweep + 1);
  }
}

__global__ void __launch_bounds__(256) k_jr_round(const JacobiJob* __restrict__ jobs, int sweep,
                                                  int r) {
  __shared__ BJRot rot[2 * kJrPairs];
  __shared__ int2 pq[2 * kJrPairs];
  const JacobiJob jb = jobs[blockIdx.y];
  const int m = jb.m, mp = m + (m & 1), np = mp / 2;
  if (m <= 0 || (jb.pad_ & 1) || r >= mp - 1) return;
  const int nt = (np + kJrPairs - 1) / kJrPairs;
  const int wg = blockIdx.x;
  const bool isA = wg < nt * nt;
  const int x = isA ? wg % nt : (wg - nt * nt) % nt, y = isA ? wg / nt : (wg - nt * nt) / nt;
  if (!isA && y * kJrRows >= m) return;
  const bool odd = (sweep * (mp - 1) + r) & 1;
  const c128* A = odd ? jb.W : jb.A;
  c128* An = odd ? jb.A : jb.W;
  const int64_t lda = odd ? jb.ldw : jb.lda, ldn = odd ? jb.lda : jb.ldw;
  const int t = threadIdx.x;
  if (t < 2 * kJrPairs) {
    // pairs of x (the rows' or V's), then of y
    const int k = (t < kJrPairs ? x : y) * kJrPairs + t % kJrPairs;
    BJRot o;
    o.cs = 1.0;
    o.sn = 0.0;
    o.e = mk(1.0, 0.0);
    int p = m, q = m;
    if (k < np && (isA || t < kJrPairs)) {
      const int a = jr_player(k, r, mp), b = jr_player(mp - 1 - k, r, mp);
      p = min(a, b);
      q = max(a, b);
      if (q < m) {
        const c128 c = gld(A + (int64_t)q * lda + p);
        const double ac = sqrt(cabs2(c));
        if (ac > 1e-300) {
          const double app = gld(&A[(int64_t)p * lda + p].x), aqq = gld(&A[(int64_t)q * lda + q].x);
          const double tau = (aqq - app) / (2.0 * ac);
          const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + hypot(1.0, tau));
          o.cs = 1.0 / sqrt(1.0 + tt * tt);
          o.sn = tt * o.cs;
          o.e = mk(c.x / ac, -c.y / ac);
        }
      }
    }
    rot[t] = o;
    pq[t] = make_int2(p, q);
  }
  __syncthreads();
  using X = BJElem<true>;
  if (isA) {
    const int kk = t % kJrPairs, ll = kJrPairs + t / kJrPairs;
    const int pk = pq[kk].x, qk = pq[kk].y, pl = pq[ll].x, ql = pq[ll].y;
    if (pk >= m || pl >= m) return;  // beyond the last pair
    const bool qkv = qk < m, qlv = ql < m;
    // a dummy player's elements are zero: read in place of them, then cleared
    const int qks = qkv ? qk : pk, qls = qlv ? ql : pl;
    const c128 a00 = gld(A + (int64_t)pl * lda + pk);
    c128 a10 = gld(A + (int64_t)pl * lda + qks);
    c128 a01 = gld(A + (int64_t)qls * lda + pk);
    c128 a11 = gld(A + (int64_t)qls * lda + qks);
    a10 = mk(qkv ? a10.x : 0.0, qkv ? a10.y : 0.0);
    a01 = mk(qlv ? a01.x : 0.0, qlv ? a01.y : 0.0);
    a11 = mk(qkv && qlv ? a11.x : 0.0, qkv && qlv ? a11.y : 0.0);
    const BJRot rk = rot[kk], rl = rot[ll];
    a01 = X::mul(rl.e, a01);
    a11 = X::mul(rl.e, a11);
    const c128 b00 = X::minus(rl.cs, a00, rl.sn, a01), b01 = X::plus(rl.sn, a00, rl.cs, a01);
    const c128 b10 = X::mulc(rk.e, X::minus(rl.cs, a10, rl.sn, a11));
    const c128 b11 = X::mulc(rk.e, X::plus(rl.sn, a10, rl.cs, a11));
    gst(An + (int64_t)pl * ldn + pk, X::minus(rk.cs, b00, rk.sn, b10));
    if (qkv) gst(An + (int64_t)pl * ldn + qk, X::plus(rk.sn, b00, rk.cs, b10));
    if (qlv) gst(An + (int64_t)ql * ldn + pk, X::minus(rk.cs, b01, rk.sn, b11));
    if (qkv && qlv) gst(An + (int64_t)ql * ldn + qk, X::plus(rk.sn, b01, rk.cs, b11));
  } else {
#pragma unroll
    for (int g = 0; g < kJrPairs * kJrRows / 256; ++g) {
      const int k = t / kJrRows + g * (256 / kJrRows), i = y * kJrRows + t % kJrRows;
      const int p = pq[k].x, q = pq[k].y;
      if (q >= m || i >= m) continue;
      const BJRot o = rot[k];
      const c128 vp = gld(jb.V + (int64_t)p * jb.ldv + i);
      const c128 vq = X::mulu(o.e, gld(jb.V + (int64_t)q * jb.ldv + i));
      gst(jb.V + (int64_t)p * jb.ldv + i, X::minus(o.cs, vp, o.sn, vq));
      gst(jb.V + (int64_t)q * jb.ldv + i, X::plus(o.sn, vp, o.cs, vq));
    }
  }
}

// eigenvalues ascending (rank by value, ties by index), vectors follow
__global__ void __launch_bounds__(1024) k_jr_final(const JacobiJob* __restrict__ jobs) {
  __shared__ double d[kSmallJacobi];
  const JacobiJob jb = jobs[blockIdx.x];
  const int m = jb.m, mp = m + (m & 1), t = threadIdx.x, sweeps = jb.pad_ >> 1;
  if (m <= 0) return;
  const bool odd = (sweeps * (mp - 1)) & 1;
  const c128* A = odd ? jb.W : jb.A;
  const int64_t lda = odd ? jb.ldw : jb.lda;
  for (int i = t; i < m; i += 1024) d[i] = gld(&A[(int64_t)i * lda + i].x);
  __syncthreads();
  for (int i = t; i < m; i += 1024) {
    const double wi = d[i], ki = rank_key(wi);
    int rank = 0;
    for (int j = 0; j < m; ++j) {
      const double kj = rank_key(d[j]);
      rank += (kj < ki || (kj == ki && j < i)) ? 1 : 0;
    }
    gst(jb.w + rank, wi);
    gst(jb.order + rank, i);
  }
  if (t == 0 && jb.sweeps) gst(jb.sweeps, sweeps);
  __syncthreads();
  for (int64_t e = t; e < (int64_t)m * m; e += 1024) {
    const int k = (int)(e / m), i = (int)(e - (int64_t)k * m);
    gst(jb.W + (int64_t)k * jb.ldw + i, gld(jb.V + (int64_t)gld(jb.order + k) * jb.ldv + i));
  }
}

static int round_jacobi(std::vector<JacobiJob> jobs, JacobiJob* jobs_dev, int max_sweeps,
                        double tol, hipStream_t st) {
  const int nj = (int)jobs.size();
  int maxm = 0;
  for (const JacobiJob& j : jobs) maxm = std::max(maxm, j.m);
  const int mp = maxm + (maxm & 1), nt = (mp / 2 + kJrPairs - 1) / kJrPairs;
  const int wgs = nt * nt + nt * ((maxm + kJrRows - 1) / kJrRows);
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    k_jr_norms<<<nj, 1024, 0, st>>>(jobs_dev, sweep, tol);
    FB_HIP(hipGetLastError());
    FB_HIP(hipMemcpyAsync(jobs.data(), jobs_dev, sizeof(JacobiJob) * nj, hipMemcpyDeviceToHost, st));
    FB_HIP(hipStreamSynchronize(st));
    int rounds = 0;
    for (const JacobiJob& j : jobs)
      if (j.m > 0 && !(j.pad_ & 1)) rounds = std::max(rounds, j.m + (j.m & 1) - 1);
    if (rounds == 0) break;
    for (int r = 0; r < rounds; ++r) {
      k_jr_round<<<dim3(wgs, nj), 256, 0, st>>>(jobs_dev, sweep, r);
      FB_HIP(hipGetLastError());
    }
  }
  k_jr_final<<<nj, 1024, 0, st>>>(jobs_dev);
  FB_HIP(hipGetLastError());
  return 0;
}

// -------------------------------------------------------------- driver
static int bj_h(int m) { return (m + kPb - 1) / kPb; }

size_t block_jacobi_bytes(int m) {
  const int h = bj_h(m), mp = kPb * h;
  const size_t sq = ((size_t)mp * mp * sizeof(c128) + 255) & ~(size_t)255;
  return 4 * sq + (size_t)h * kPb * kPb * sizeof(c128) + 256 + (size_t)h * sizeof(int32_t) +
         256 + 2 * (size_t)mp * sizeof(double) + 4 * 256;
}

int block_jacobi(const std::vector<JacobiJob>& jobs, const JacobiJob* jobs_dev, char* work,
                 void* dv_dev, double* norms_dev, int max_sweeps, double tol, hipStream_t st) {
  const int nj = (int)jobs.size();
  if (nj == 0) return 0;
  std::vector<BJDev> dv(nj);
  int max_h = 0, max_mp = 0, max_rounds = 1;
  size_t off = 0;
  for (int q = 0; q < nj; ++q) {
    BJDev& d = dv[q];
    d.m = jobs[q].m;
    d.h = bj_h(d.m);
    d.mp = kPb * d.h;
    d.cplx = 0;  // set by k_bj_init
    auto take = [&](size_t bytes) {
      char* p = work + off;
      off += (bytes + 255) & ~(size_t)255;
      return p;
    };
    const size_t sq = (size_t)d.mp * d.mp * sizeof(c128);
    d.A[0] = (c128*)take(sq);
    d.A[1] = (c128*)take(sq);
    d.V[0] = (c128*)take(sq);
    d.V[1] = (c128*)take(sq);
    d.U = (c128*)take((size_t)d.h * kPb * kPb * sizeof(c128));
    d.skip = (int32_t*)take((size_t)d.h * sizeof(int32_t));
    d.part = (double*)take(2 * (size_t)d.mp * sizeof(double));
    max_h = std::max(max_h, d.h);
    max_mp = std::max(max_mp, d.mp);
    max_rounds = std::max(max_rounds, 2 * d.h - 1);
  }
  static bool attr = false;
  const size_t lds_pairs = 2 * (size_t)kPb * kPL * sizeof(c128);
  const size_t lds_upd = (size_t)kPb * kPL * sizeof(c128);
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)k_bj_pairs, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds_pairs);
    (void)hipFuncSetAttribute((const void*)k_bj_update<1>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_upd);
    (void)hipGetLastError();
    attr = true;
  }
  BJDev* dvd = (BJDev*)dv_dev;
  FB_HIP(hipMemcpyAsync(dvd, dv.data(), sizeof(BJDev) * nj, hipMemcpyHostToDevice, st));
  k_bj_init<<<dim3(1024, nj), 256, 0, st>>>(jobs_dev, dvd);
  FB_HIP(hipGetLastError());
  std::vector<double> nrm(2 * nj);
  int sweeps = 0, cur = 0;  // cur: which copy of A and V a round reads
  // few pairs leave most of the chip idle: their U is then shared out over 2
  // or 4 workgroups each, as long as every workgroup has a CU of its own (a
  // second round of workgroups would cost more than the 18 % that it saves)
  const int cus = rule_cus();
  const int rlog = 4 * max_h * nj <= cus ? 4 : 2 * max_h * nj <= cus ? 5 : 6;
  const int upd_wgs = max_h * (max_h + 1) / 2 + max_h * (max_mp / kPb);
  // and tiles are split until there are four workgroups per CU
  const int64_t tiles = (int64_t)upd_wgs * nj;
  const int csplit = 4 * tiles <= 4 * cus ? 4 : 2 * tiles <= 4 * cus ? 2 : 1;
  for (int sw = 0; sw <= max_sweeps; ++sw) {
    k_bj_norms<<<dim3(max_mp, nj), 256, 0, st>>>(dvd, cur);
    FB_HIP(hipGetLastError());
    k_bj_norms_final<<<nj, 256, 0, st>>>(dvd, norms_dev);
    FB_HIP(hipGetLastError());
    FB_HIP(hipMemcpyAsync(nrm.data(), norms_dev, sizeof(double) * 2 * nj, hipMemcpyDeviceToHost, st));
    FB_HIP(hipStreamSynchronize(st));
    bool done = true;
    for (int q = 0; q < nj; ++q)
      if (!(nrm[2 * q] <= tol * tol * nrm[2 * q + 1])) done = false;
    if (done || sw == max_sweeps) break;
    ++sweeps;
    // every matrix takes max_rounds rounds (a smaller one completes further
    // sweeps of its own schedule, which keeps it converging)
    for (int r = 0; r < max_rounds; ++r) {
      k_bj_pairs<<<dim3(max_h << (6 - rlog), nj), kPairThreads, lds_pairs, st>>>(dvd, cur, rlog);
      FB_HIP(hipGetLastError());
      if (csplit == 4)
        k_bj_update<4><<<dim3(4 * upd_wgs, nj), 256, lds_upd / 4, st>>>(dvd, cur);
      else if (csplit == 2)
        k_bj_update<2><<<dim3(2 * upd_wgs, nj), 256, lds_upd / 2, st>>>(dvd, cur);
      else
        k_bj_update<1><<<dim3(upd_wgs, nj), 256, lds_upd, st>>>(dvd, cur);
      FB_HIP(hipGetLastError());
      cur ^= 1;
    }
  }
  k_bj_rank<<<dim3((max_mp + 255) / 256, nj), 256, 0, st>>>(jobs_dev, dvd, cur);
  FB_HIP(hipGetLastError());
  k_bj_vectors<<<dim3(1024, nj), 256, 0, st>>>(jobs_dev, dvd, cur);
  FB_HIP(hipGetLastError());
  for (int q = 0; q < nj; ++q)
    if (jobs[q].sweeps) FB_HIP(hipMemcpyAsync(jobs[q].sweeps, &sweeps, sizeof(int32_t),
                                              hipMemcpyHostToDevice, st));
  FB_HIP(hipStreamSynchronize(st));
  return 0;
}

static_assert(sizeof(BJDev) <= kBjDescBytes, "descriptor size");

size_t eig_work_bytes(const std::vector<int>& ms) {
  size_t b = 0;
  int n = 0;
  for (int m : ms)
    if (m > kSmallJacobi) {
      b += (block_jacobi_bytes(m) + 255) & ~(size_t)255;
      ++n;
    }
  return b + (size_t)n * kBjDescBytes + 2 * (size_t)n * sizeof(double) + 1024;
}

void carve_eig_work(Arena& ar, const std::vector<int>& ms, EigWork& w) {
  size_t b = 0;
  int n = 0;
  for (int m : ms)
    if (m > kSmallJacobi) {
      b += (block_jacobi_bytes(m) + 255) & ~(size_t)255;
      ++n;
    }
  w.bj = n ? ar.take<char>(b + 256 * (size_t)n) : nullptr;
  w.dv = n ? (void*)ar.take<char>((size_t)n * kBjDescBytes) : nullptr;
  w.norms = n ? ar.take<double>(2 * (size_t)n) : nullptr;
}

bool rounds_pay(int maxm, int64_t sum2, int cus) {
  const int64_t room = 80 * (int64_t)maxm * maxm - 450000;  // of 256 CUs
  return maxm >= kRoundJacobi && 256 * sum2 <= room * cus;
}

int reduced_eig(std::vector<JacobiJob> jobs, JacobiJob* jobs_dev, const EigWork& w,
                int max_sweeps, double tol, hipStream_t st) {
  std::vector<JacobiJob> small, large;
  for (const JacobiJob& j : jobs) (j.m > kSmallJacobi ? large : small).push_back(j);
  std::vector<JacobiJob> all(small);
  all.insert(all.end(), large.begin(), large.end());
  if (all.empty()) return 0;
  FB_HIP(hipMemcpyAsync(jobs_dev, all.data(), sizeof(JacobiJob) * all.size(),
                        hipMemcpyHostToDevice, st));
  if (!small.empty()) {
    int maxm = 0;
    int64_t sum2 = 0;
    for (const JacobiJob& j : small) {
      maxm = std::max(maxm, j.m);
      sum2 += (int64_t)j.m * j.m;
    }
    if (rounds_pay(maxm, sum2, rule_cus())) {
      ProfScope ps(FB_PROF_JACOBI, st, 0.0);
      FB_TRY(round_jacobi(small, jobs_dev, max_sweeps, tol, st));
    } else {
      FB_TRY(launch_jacobi((int)small.size(), jobs_dev, max_sweeps, tol, st));
    }
  }
  if (!large.empty()) {
    if (!w.bj) return FB_ERR_INTERNAL;
    ProfScope ps(FB_PROF_JACOBI, st, 0.0);
    FB_TRY(block_jacobi(large, jobs_dev + small.size(), w.bj, w.dv, w.norms, max_sweeps, tol, st));
  }
  return 0;
}

}  // namespace fb
