// Band LU with partial pivoting of the shifted systems A = zI - B
// (one factorisation per integration node, Section 2.2, eq:feast_L2),
// producing the block form consumed by the block solves.
//
// One workgroup per system.  The active part of the elimination of columns
// j .. j+7 is rows j .. j+b+7 and columns j .. j+2b+7 (U widens to bandwidth
// 2b under row interchanges).
//
// Output per block k of b columns (the window rows kb .. kb+2b-1):
//   perm  the net row permutation of the block's interchanges,
//   Lh11  unit lower multipliers of the top b rows (row-swapped as later
//         interchanges of the block move them, so that P A_panel = Lh U),
//   Lh21  multipliers of the bottom b rows,
//   U(k,k), U(k,k+1), U(k,k+2).
// A second kernel replaces Lh11 and U(k,k) by their inverses, a third Lh21
// by M = Lh21 Lh11^{-1}, and a fourth Lh11^{-1}, U(k,k+1) and U(k,k+2) by
// Q = U(k,k)^{-1} Lh11^{-1}, G1 = U(k,k)^{-1} U(k,k+1) and
// G2 = U(k,k)^{-1} U(k,k+2), so that each step of every solve sweep is one
// set of independent dense b x b products (see solve.hip).
//
// Within a block the multipliers are written to a per-system scratch under
// their row's position at the block's start (or entry), and gathered into row
// order once after the end of the block.
#include "mfma.h"
#include "prof.h"
#include "solve_job.h"

namespace fb {

static const int kLuThreads = 512;
static const size_t kLdsBudget = 160 * 1024;

// ---- wave-wide reductions of wave 0 for the pivot search, by DPP lane moves
// within rows of 16 lanes (xor 1, xor 2, half mirror, mirror) and reads of
// lanes 0, 16, 32 and 48; every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ uint64_t rdlane64(uint64_t v, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}
template <bool MAX>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v) {
  auto pick = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
  v = pick(v, dpp32<0xB1>(v));   // quad_perm [1,0,3,2]
  v = pick(v, dpp32<0x4E>(v));   // quad_perm [2,3,0,1]
  v = pick(v, dpp32<0x141>(v));  // row_half_mirror
  v = pick(v, dpp32<0x140>(v));  // row_mirror
  auto rd = [&](int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
  return pick(pick(rd(0), rd(16)), pick(rd(32), rd(48)));
}
// leading and remaining 32 bits of the bit pattern of a non-negative float or
// double, whose order is the values'
__device__ __forceinline__ uint32_t high_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t high_bits(double v) {
  return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32);
}
__device__ __forceinline__ uint32_t low_bits(float) { return 0; }
__device__ __forceinline__ uint32_t low_bits(double v) {
  return (uint32_t)__double_as_longlong(v);
}

// ---------------------------------------------------------------- fragments
// A fragments of one wave for one block product: register s holds
// A[16 w + lane % 16][4 s + lane / 16] (complex).
template <typename R, int NB>
struct Frag {
  cx<R> a[NB / 4];
};

// k ranges [k0, k1) are multiples of 16 and the same for the whole wave
// (readfirstlane makes that visible to the compiler, so that the range test
// is one scalar branch per 16-row chunk and a chunk's LDS reads issue
// together).
template <typename R, int NB>
__device__ __forceinline__ void frag_load(Frag<R, NB>& f, const cx<R>* A, int w, int lane, int k0,
                                          int k1) {
  const int i = 16 * w + (lane & 15), kq = lane >> 4;
  const int c0 = __builtin_amdgcn_readfirstlane(k0) >> 4;
  const int c1 = __builtin_amdgcn_readfirstlane(k1) >> 4;
#pragma unroll
  for (int ch = 0; ch < NB / 16; ++ch) {
    if (ch < c0 || ch >= c1) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * ch + 4 * q + kq;
      f.a[4 * ch + q] = A[(size_t)k * NB + i];
    }
  }
}

// acc += A * B over k in [k0, k1) from prefetched fragments; NEG subtracts.
// B row k is LDS row k, row stride ldb elements.
template <typename R, int NB, int NC, bool NEG>
__device__ __forceinline__ void frag_mma(Acc<R, NC>& acc, const Frag<R, NB>& f, const cx<R>* Bl,
                                         int ldb, int lane, int k0, int k1) {
  const int kq = lane >> 4;
  const int j = lane & 15;
  const int c0 = __builtin_amdgcn_readfirstlane(k0) >> 4;
  const int c1 = __builtin_amdgcn_readfirstlane(k1) >> 4;
#pragma unroll
  for (int ch = 0; ch < NB / 16; ++ch) {
    if (ch < c0 || ch >= c1) continue;
    cx<R> bv[4][NC];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * ch + 4 * q + kq;
      const cx<R>* bp = Bl + (size_t)k * ldb + j;
#pragma unroll
      for (int c = 0; c < NC; ++c) bv[q][c] = bp[16 * c];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      cx<R> a = f.a[4 * ch + q];
      R ar = a.x, ai = a.y;
      if (NEG) {
        ar = -ar;
        ai = -ai;
      }
      const R as = ar + ai;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        acc.p1[c] = MF<R>::mma(ar, bv[q][c].x, acc.p1[c]);
        acc.p2[c] = MF<R>::mma(ai, bv[q][c].y, acc.p2[c]);
        acc.p3[c] = MF<R>::mma(as, bv[q][c].x + bv[q][c].y, acc.p3[c]);
      }
    }
  }
}

// accumulator -> LDS (rows 16 w + MF<R>::row(lane, r), columns 16 c + lane%16)
template <typename R, int NC>
__device__ __forceinline__ void acc_to_lds(const Acc<R, NC>& acc, cx<R>* L, int ldb, int w,
                                           int lane) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * w + MF<R>::row(lane, r);
      L[(size_t)row * ldb + 16 * c + (lane & 15)] = acc.get(c, r);
    }
}

// ---------------------------------------------------------------- elimination
// Panels of kP columns of the band padded to bandwidth NB.  The window holds
// MT x 16 physical rows (the NB + kP logical rows a panel can touch, in no
// order) by NCB x 16 columns (block column c / 16 mod NCB).  A row stays in
// its physical slot until it becomes a pivot row; the slot then takes an
// entering row, so that interchanges move nothing and every update is a
// product over all physical rows.
//
// Step s applies panel s to the right and factors panel s + 1:
//   1. the block column that holds panel s + 1, a row tile per wave (its
//      pivot rows solved with the panel's unit lower triangle, the rest
//      updated on MFMA, the entering rows put into the freed slots),
//   2. wave 0 factors panel s + 1 in registers (lane = row, up to NR rows
//      per lane); the other waves take the remaining block columns one by
//      one from a counter in LDS, with the panel's rows of U, its
//      multipliers and the previous block's gather.
// The row tiles that do not fit LDS live in the system's global scratch.
//
// What bounds it: up to b = 64 the panel chain of wave 0 (pivot search,
// reciprocal, broadcast and update of one column after the other, about 1 000
// cycles a column) and the block column that it waits for, above that the
// updates of one CU and, in complex128, the row tiles in global memory.  Eight
// columns per panel: the chain's own update work grows with the panel, the
// window's traffic falls with it.  Before, one column and one rank-one update
// per two barriers.  LU per column, before -> now: complex64 b = 64 3.3 -> 0.75
// us, b = 128 10.7 -> 1.7 us; complex128 b = 30 2.8 -> 0.9 us, b = 64 3.9 ->
// 1.1 us (one launch of 4 to 32 systems).
constexpr int kP = 8;
constexpr int kNoRow = 0x40000000;  // logical row of an empty slot

template <typename R>
struct LuArgs {
  const c128* Bblk;
  int64_t n;
  int K;
  const c128* zs;
  cx<R>* mats;     // nsys * K * 5 * NB * NB
  int16_t* perm;   // nsys * K * 2 NB
  int32_t* info;   // nsys
  cx<R>* lscr;     // nsys * 2 * 2 NB * NB: multipliers by window row, by block parity
  cx<R>* gwin;     // nsys * (MT - LT) * 16 * LD
};

// Geometry of the elimination window.  A 16 x 16 tile is stored in the
// accumulator layout of the MFMA that updates it: the 64 lanes' four real
// parts, then their four imaginary parts, in 16-byte pieces.
template <typename R, int NB>
struct LuShape {
  static constexpr int MT = NB / 16 + 1;      // row tiles: NB + kP rows
  static constexpr int NCB = NB / 8 + 1;      // block columns: 2 NB + 16
  static constexpr int ROWS = 16 * MT;
  static constexpr int NR = (NB + kP + 63) / 64;
  static constexpr int UC = 16 * NCB + 2;     // row of the panel's rows of U
  static constexpr int INTS = 4 + 2 * kP + 4 * NB + 2 * ROWS;
  // counter, pivots, positions, rows; the panels (two), their pivot rows, U
  static constexpr size_t HEAD =
      ((INTS * sizeof(int) + 15) & ~(size_t)15) +
      (2 * kP * ROWS + 2 * kP * kP + kP * UC) * sizeof(cx<R>);
  static constexpr size_t TILE = 256 * sizeof(cx<R>) * (size_t)NCB;  // a row of tiles
  static constexpr int FIT = (int)((kLdsBudget - HEAD) / TILE);
  static constexpr int LT = FIT < MT ? FIT : MT;  // row tiles in LDS
  static constexpr size_t LDS = HEAD + LT * TILE;
  static constexpr size_t SCRATCH = (size_t)(MT - LT) * TILE;
};
// place of element (row, col) of a tile, in R; the imaginary part 256 further on
template <typename R>
__device__ __forceinline__ int tile_at(int row, int col) {
  if constexpr (sizeof(R) == 4)
    return (((row >> 2) & 3) * 16 + col) * 4 + (row & 3);
  else
    return ((row >> 3) & 1) * 128 + ((row & 3) * 16 + col) * 2 + ((row >> 2) & 1);
}
// a lane's part of a tile: real and imaginary accumulators
template <typename R>
struct LuTile {
  typename MF<R>::V re, im;
};
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
// 16 bytes per lane and access; GL: global memory
template <bool GL>
__device__ __forceinline__ void tile_load(LuTile<float>& c, const float* t, int lane) {
  const f32x4* p = reinterpret_cast<const f32x4*>(t) + lane;
  c.re = GL ? gld(p) : p[0];
  c.im = GL ? gld(p + 64) : p[64];
}
template <bool GL>
__device__ __forceinline__ void tile_store(float* t, const LuTile<float>& c, int lane) {
  f32x4* p = reinterpret_cast<f32x4*>(t) + lane;
  if (GL) {
    gst(p, (f32x4)c.re);
    gst(p + 64, (f32x4)c.im);
  } else {
    p[0] = c.re;
    p[64] = c.im;
  }
}
template <bool GL>
__device__ __forceinline__ void tile_load(LuTile<double>& c, const double* t, int lane) {
  const f64x2* p = reinterpret_cast<const f64x2*>(t) + lane;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f64x2 x = GL ? gld(p + 64 * h) : p[64 * h];
    const f64x2 y = GL ? gld(p + 128 + 64 * h) : p[128 + 64 * h];
    c.re[2 * h] = x[0];
    c.re[2 * h + 1] = x[1];
    c.im[2 * h] = y[0];
    c.im[2 * h + 1] = y[1];
  }
}
template <bool GL>
__device__ __forceinline__ void tile_store(double* t, const LuTile<double>& c, int lane) {
  f64x2* p = reinterpret_cast<f64x2*>(t) + lane;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const f64x2 x = {c.re[2 * h], c.re[2 * h + 1]}, y = {c.im[2 * h], c.im[2 * h + 1]};
    if (GL) {
      gst(p + 64 * h, x);
      gst(p + 128 + 64 * h, y);
    } else {
      p[64 * h] = x;
      p[128 + 64 * h] = y;
    }
  }
}
// Barrier for what waves hand each other through LDS: outstanding global
// stores are not waited for.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <typename R>
__device__ __forceinline__ R lane_value(R v, int l);
template <>
__device__ __forceinline__ float lane_value(float v, int l) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
}
template <>
__device__ __forceinline__ double lane_value(double v, int l) {
  return __longlong_as_double((long long)rdlane64((uint64_t)__double_as_longlong(v), l));
}

// c ? a : b by parts (a choice between whole elements would go through memory)
template <typename R>
__device__ __forceinline__ cx<R> pick(bool c, cx<R> a, cx<R> b) {
  return mk(c ? a.x : b.x, c ? a.y : b.y);
}
// x - l u, the product rounded before it is subtracted: one rounding of the
// size of x
template <typename R>
__device__ __forceinline__ cx<R> csub(cx<R> x, cx<R> l, cx<R> u) {
  return mk(x.x - fma(l.x, u.x, -(l.y * u.y)), x.y - fma(l.y, u.x, l.x * u.y));
}
// 1 / u from |u|^2 = d: the hardware's estimate of 1 / d and Newton steps, the
// last of which rounds; where d leaves the range in which they hold, the
// general division
__device__ __forceinline__ float recip_of(float d) {
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  return fmaf(fmaf(-d, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip_of(double d) {
  double r = __builtin_amdgcn_rcp(d);
#pragma unroll
  for (int i = 0; i < 3; ++i) r = fma(fma(-d, r, 1.0), r, r);
  return r;
}
template <typename R>
__device__ __forceinline__ cx<R> inverse_of(cx<R> u, R d) {
  constexpr R big = sizeof(R) == 4 ? (R)1e30f : (R)1e290;
  if (__builtin_expect(d > 1 / big && d < big, 1)) {
    // quotients with a last correction, which rounds them as a division does
    const R r = recip_of(d), x = u.x * r, y = -u.y * r;
    return mk<R>(fma(fma(-d, x, u.x), r, x), fma(fma(-d, y, -u.y), r, y));
  }
  return d > (R)0 ? cinv(u) : mk<R>(0, 0);
}

template <typename R, int NB>
__global__ void __launch_bounds__(kLuThreads) k_band_lu(LuArgs<R> a) {
  using C = cx<R>;
  using G = LuShape<R, NB>;
  constexpr int MT = G::MT, NCB = G::NCB, ROWS = G::ROWS, NR = G::NR, LT = G::LT, UC = G::UC;
  constexpr int LROWS = 16 * LT, RPB = NB / 16, BB = NB * NB;
  // Small blocks: every element takes its updates one after another in pivot
  // order, each product rounded, as in an unblocked elimination.  The panels
  // bound the kernel there, so that the matrix cores would gain nothing (and
  // the FP64 matrix rate is that of the vector unit).
  constexpr bool ORD = NB <= 48;
  constexpr int NW = kLuThreads / 64;
  extern __shared__ __align__(16) char lds_raw[];
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int sys = blockIdx.x;
  const int n = (int)a.n, K = a.K;
  const int npad = K * NB, steps = npad / kP;
  const c128 z = a.zs[sys];

  int* cnt = reinterpret_cast<int*>(lds_raw);  // next unit of the step
  int* ps = cnt + 4;                           // [2][kP] pivot slots of a panel
  int* idx = ps + 2 * kP;                      // [2][2 NB] window row at each position of a block
  int* meta = idx + 4 * NB;                    // [2][ROWS] window row | pivot step << 16, -1 empty
  C* Lp = reinterpret_cast<C*>(lds_raw + ((G::INTS * sizeof(int) + 15) & ~(size_t)15));
  C* Lt = Lp + 2 * kP * ROWS;                  // [2][kP][kP] the pivot rows of a panel
  C* Ub = Lt + 2 * kP * kP;                    // [kP][UC] the panel's rows of U, from block column J
  R* W = reinterpret_cast<R*>(Ub + kP * UC);   // [LT][NCB] tiles
  R* gw = reinterpret_cast<R*>(a.gwin) + (size_t)sys * (MT - LT) * NCB * 512;
  C* mats = a.mats + (size_t)sys * K * 5 * BB;
  int16_t* permg = a.perm + (size_t)sys * K * 2 * NB;
  C* lscr = a.lscr + (size_t)sys * 4 * BB;

  const int c16 = lane & 15, g4 = lane >> 4;

  // element (row, col) of the tile in block column p of the window
  auto wput = [&](int row, int p, int col, C v) {
    if (LT == MT || row < LROWS) {
      R* at = W + (((row >> 4) * NCB + p) * 512 + tile_at<R>(row, col));
      at[0] = v.x;
      at[256] = v.y;
    } else {
      R* at = gw + ((((row - LROWS) >> 4) * NCB + p) * 512 + tile_at<R>(row, col));
      gst(at, v.x);
      gst(at + 256, v.y);
    }
  };
  // rows r .. of block row kb, block column cb (in units of NB): element
  // (kb NB + r, cb NB + cc) of z I - B, identity beyond n, zero beyond K blocks
  auto a_load = [&](int kb, int r, int cb, int cc) -> c128 {
    const int s = cb - kb + 1;
    const bool ok = kb < K && s >= 0 && s < 3;
    return gld(a.Bblk + (size_t)(ok ? kb * 3 + s : 0) * BB + (cc * NB + r));
  };
  auto a_value = [&](c128 v, int kb, int r, int cb, int cc) -> C {
    const int s = cb - kb + 1;
    const bool ok = kb < K && s >= 0 && s < 3;
    C x = pick(ok, mk<R>((R)-v.x, (R)-v.y), mk<R>(0, 0));
    const bool in = kb * NB + r < n;
    x = pick(ok && s == 1 && r == cc, mk<R>(in ? (R)(z.x - v.x) : (R)1, in ? (R)z.y : (R)0), x);
    return x;
  };

  // ---- the first window: rows 0 .. NB + kP - 1 in their own slots
  for (int e = t; e < ROWS * 16 * NCB; e += kLuThreads) {
    const int row = e / (16 * NCB), c = e % (16 * NCB);
    C v = mk<R>(0, 0);
    if (row < NB + kP)
      v = a_value(a_load(row / NB, row % NB, c / NB, c % NB), row / NB, row % NB, c / NB, c % NB);
    wput(row, c >> 4, c & 15, v);
    if (c < kP) Lp[c * ROWS + row] = v;
  }
  for (int e = t; e < 2 * BB; e += kLuThreads) gst(lscr + e, mk<R>(0, 0));
  __syncthreads();
  if (w == 0) {
    // ---- wave 0: the panels.  Panel s1 = s + 1 is factored while the other
    // waves apply panel s; its columns were put into its place in Lp.
    __builtin_amdgcn_s_setprio(3);
    int lp[NR], wr[NR], first_zero = 0;  // logical and window row of the lane's slots
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int row = lane + 64 * r;
      lp[r] = row < NB + kP && row < npad ? row : kNoRow;
      wr[r] = lp[r];
    }
    int kb1 = 0, jj1 = 0;
    for (int s1 = 0; s1 < steps; ++s1) {
      const int j1 = kP * s1, kb0 = NB * kb1, parn = s1 & 1;
      int* idxk = idx + (kb1 & 1) * 2 * NB;
      C* Ln = Lp + parn * kP * ROWS;
      C x[NR][kP];
      int step[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int row = lane + 64 * r;
        step[r] = lp[r] == kNoRow ? -1 : kP;
        const int rr = row < ROWS ? row : 0;
#pragma unroll
        for (int c = 0; c < kP; ++c) x[r][c] = Ln[c * ROWS + rr];
      }
      if (jj1 == 0) {
        for (int e = lane; e < 2 * NB; e += 64) idxk[e] = e;
#pragma unroll
        for (int r = 0; r < NR; ++r) wr[r] = lp[r] - kb0;
      }
#pragma unroll
      for (int k = 0; k < kP; ++k) {
        // largest |x|^2 of the rows not yet pivots (a NaN counts as 0), ties
        // to the lowest logical row: by the leading 32 bits, which nearly
        // always decide
        R v[NR];
        uint32_t key[NR], best = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          v[r] = fmax(fma(x[r][k].x, x[r][k].x, x[r][k].y * x[r][k].y), (R)0);
          key[r] = step[r] == kP ? high_bits(v[r]) : 0;
          best = max(best, key[r]);
        }
        best = wave_reduce<true>(best);
        uint64_t m[NR];
        int total = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          m[r] = __builtin_amdgcn_ballot_w64(key[r] == best);
          total += __builtin_popcountll(m[r]);
        }
        if (__builtin_expect(total > 1 || best == 0, 0)) {
          uint32_t lo = 0, low = kNoRow;
          bool top[NR];
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            top[r] = step[r] == kP && key[r] == best;
            lo = max(lo, top[r] ? low_bits(v[r]) : 0u);
          }
          lo = wave_reduce<true>(lo);
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            top[r] = top[r] && low_bits(v[r]) == lo;
            low = min(low, top[r] ? (uint32_t)lp[r] : (uint32_t)kNoRow);
          }
          low = wave_reduce<false>(low);
#pragma unroll
          for (int r = 0; r < NR; ++r)
            m[r] = __builtin_amdgcn_ballot_w64(top[r] && (uint32_t)lp[r] == low);
        }
        // the pivot row's slot (wave-uniform) and its entries from column k on
        int pr = 0, plp = 0;
        R d = 0;
        C u[kP];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          if (NR > 1 && m[r] == 0) continue;
          const int pl = __builtin_ctzll(m[r]);
          pr = pl + 64 * r;
          d = lane_value(v[r], pl);
          plp = __builtin_amdgcn_readlane(lp[r], pl);
#pragma unroll
          for (int c = k; c < kP; ++c)
            u[c] = mk<R>(lane_value(x[r][c].x, pl), lane_value(x[r][c].y, pl));
        }
        if (!(d > (R)0) && first_zero == 0) first_zero = j1 + k + 1;
        const C rp = inverse_of(u[k], d);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          // the interchange: the row at position j1 + k takes the pivot's place
          const bool piv = pr == lane + 64 * r;
          lp[r] = piv ? j1 + k : lp[r] == j1 + k ? plp : lp[r];
          step[r] = piv ? k : step[r];
          const bool live = step[r] == kP;
          const C xk = x[r][k];
          C l = mk(fma(xk.x, rp.x, -(xk.y * rp.y)), fma(xk.x, rp.y, xk.y * rp.x));
          x[r][k] = pick(live, l, x[r][k]);
          l = pick(live, l, mk<R>(0, 0));
#pragma unroll
          for (int c = k + 1; c < kP; ++c) x[r][c] = csub(x[r][c], l, u[c]);
        }
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int row = lane + 64 * r;
        if (row < ROWS) {
#pragma unroll
          for (int c = 0; c < kP; ++c) Ln[c * ROWS + row] = x[r][c];
          meta[parn * ROWS + row] = step[r] < 0 ? -1 : wr[r] | (step[r] << 16);
        }
        if (step[r] == kP && jj1 + kP == NB) idxk[lp[r] - kb0] = wr[r];
        if (step[r] >= 0 && step[r] < kP) {
          ps[parn * kP + step[r]] = row;
          idxk[jj1 + step[r]] = wr[r];
#pragma unroll
          for (int c = 0; c < kP; ++c) Lt[(parn * kP + step[r]) * kP + c] = x[r][c];
          // the freed slot's entering row
          const int in = j1 + kP + NB + step[r];
          lp[r] = in < npad ? in : kNoRow;
          wr[r] = lp[r] - kb0;
        }
      }
      jj1 += kP;
      if (jj1 == NB) {
        jj1 = 0;
        ++kb1;
      }
      lds_barrier();    // panel s1 is factored and panel s1 - 1 applied
      lds_barrier();    // the panel's rows of U are formed
      lds_barrier();    // the columns of panel s1 + 1 are updated
    }
    if (lane == 0) gst(a.info + sys, first_zero);
    __syncthreads();
    return;
  }

  // ---- the other waves
  __syncthreads();  // panel 0
  // wave-uniform state of a step: column j0 = NB kblk + jj; block column J =
  // j0 / 16, its place jp = J mod NCB in the window and tj = J mod RPB
  int kblk = 0, jj = 0, jp = 0, tj = 0;
  for (int s = 0; s < steps; ++s) {
    const int par = s & 1, o = jj & 15;
    const C* Lk = Lp + par * kP * ROWS;
    const int* psk = ps + par * kP;
    // entering rows j0 + kP + NB + k, k = 0 .. 7: block row kbe, rows re + k
    const bool up = jj + kP == NB;
    const int kbe = kblk + (up ? 2 : 1), re = up ? 0 : jj + kP;
    // block column J + d: its place in the window; block and column in it
    auto place = [&](int d) {
      const int p = jp + d;
      return p >= NCB ? p - NCB : p;
    };
    auto ent_load = [&](c128* e, int d) {
      const int cb = kblk + (tj + d) / RPB, cc = ((tj + d) % RPB) * 16 + c16;
#pragma unroll
      for (int q = 0; q < 2; ++q) e[q] = a_load(kbe, re + g4 + 4 * q, cb, cc);
    };
    auto ent_value = [&](const c128* e, int q, int d) {
      const int cb = kblk + (tj + d) / RPB, cc = ((tj + d) % RPB) * 16 + c16;
      return a_value(e[q], kbe, re + g4 + 4 * q, cb, cc);
    };
    auto ent_store = [&](const c128* e, int d) {
#pragma unroll
      for (int q = 0; q < 2; ++q) wput(psk[g4 + 4 * q], place(d), c16, ent_value(e, q, d));
    };
    // this lane's entries of the panel's rows of U in block column J + d as
    // MFMA operands: rows g4 and g4 + 4
    struct Bop {
      R x[2], y[2], ny[2];
    };
    auto b_load = [&](Bop& o2, int d) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const C u = Ub[(g4 + 4 * q) * UC + 16 * d + c16];
        o2.x[q] = u.x;
        o2.y[q] = u.y;
        o2.ny[q] = -u.y;
      }
    };
    // the panel's rows of U in block column J + d to the factors
    auto u_out = [&](int d) {
      const int te = tj + d, k = lane & 7;  // te: within the three blocks of this row block
      if (te >= 3 * RPB) return;
      C* at = mats + (size_t)(kblk * 5 + 2 + te / RPB) * BB + ((te % RPB) * 16 * NB + jj + k);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int c = (lane >> 3) + 8 * q;
        if (d == 0 && c < kP) continue;  // the panel's own columns
        gst(at + c * NB, Ub[k * UC + 16 * d + c]);
      }
    };
    // c -= L U for row tile rt
    auto update = [&](LuTile<R>& c, int rt, const Bop& o2, int d) {
      if constexpr (ORD) {
#pragma unroll
        for (int k = 0; k < kP; ++k) {
          const C u = Ub[k * UC + 16 * d + c16];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const C f = Lk[k * ROWS + 16 * rt + MF<R>::row(lane, r)];
            const C x = csub(mk<R>(c.re[r], c.im[r]), f, u);
            c.re[r] = x.x;
            c.im[r] = x.y;
          }
        }
        return;
      }
      // the products are summed first and subtracted once: one rounding of
      // the size of c per panel (complex64, n = 16384, b = 64: the
      // solutions' residuals are 5.5e-7, and 6.2e-7 with c as the accumulator)
      LuTile<R> m;
      m.re = m.im = typename MF<R>::V{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const C f = Lk[(g4 + 4 * q) * ROWS + 16 * rt + c16];
        m.re = MF<R>::mma(f.x, o2.x[q], m.re);
        m.im = MF<R>::mma(f.x, o2.y[q], m.im);
        m.re = MF<R>::mma(f.y, o2.ny[q], m.re);
        m.im = MF<R>::mma(f.y, o2.x[q], m.im);
      }
      c.re -= m.re;
      c.im -= m.im;
    };
    auto w_tile = [&](int rt, int p) { return W + (rt * NCB + p) * 512; };
    auto g_tile = [&](int rt, int p) { return gw + ((rt - LT) * NCB + p) * 512; };

    const int d1 = o == 0 ? 0 : 1;  // block column of panel s + 1
    constexpr int NO = NW - 1, Q1 = (MT + NO - 1) / NO;
    // unit u of the step: block column J + unit_col(u), the last of the steps
    // that finish block column J its successor in that place
    const int ntile = NCB - 1;
    auto unit_col = [&](int u) { return o != 0 && u == ntile - 1 ? NCB : d1 + 1 + u; };
    // ---- 1. the panel's rows of U, 64 columns per wave: the pivot rows
    // solved with the panel's unit lower triangle
    for (int ch = NW - 1 - w; 4 * ch + d1 < NCB; ch += NO) {
      const int d = d1 + 4 * ch + g4;
      const bool in = d < NCB;
      const int p = in ? place(d) : 0;
      const C* L = Lt + par * kP * kP;
      C x[kP];
#pragma unroll
      for (int k = 0; k < kP; ++k) {
        // without branches, so that the rows in global memory are read together
        const int row = __builtin_amdgcn_readfirstlane(psk[k]);
        const int at = ((row >> 4) * NCB + p) * 512 + tile_at<R>(row, c16);
        if constexpr (LT == MT) {
          x[k] = mk(W[at], W[at + 256]);
        } else {
          const bool l = row < LROWS;
          const int al = l ? at : 0, ag = l ? 0 : at - LT * NCB * 512;
          x[k] = pick(l, mk(W[al], W[al + 256]), mk(gld(gw + ag), gld(gw + (ag + 256))));
        }
      }
#pragma unroll
      for (int k = 1; k < kP; ++k)
#pragma unroll
        for (int i = 0; i < k; ++i) x[k] = csub(x[k], L[k * kP + i], x[i]);
      if (in) {
#pragma unroll
        for (int k = 0; k < kP; ++k) Ub[k * UC + 16 * d + c16] = x[k];
      }
    }
    // what the next parts need from memory
    c128 e1[2], e0[2];
    LuTile<R> v1[Q1];
    ent_load(e1, d1);
    ent_load(e0, unit_col(w - 1));
    if (w - 1 < MT) {
#pragma unroll
      for (int q = 0; q < Q1; ++q) {
        const int rt = w - 1 + NO * q;
        if (rt < LT)
          tile_load<false>(v1[q], w_tile(rt, place(d1)), lane);
        else if (rt < MT)
          tile_load<true>(v1[q], g_tile(rt, place(d1)), lane);
      }
    }
    lds_barrier();

    // ---- 2. the block column of panel s + 1, a row tile per wave: that
    // panel's columns go to its place in Lp
    if (w - 1 < MT) {
      const int po = o ^ kP;  // the panel's columns: po .. po + 7
      C* Ln = Lp + (par ^ 1) * kP * ROWS + (c16 & 7) * ROWS;
      const bool isp = (c16 & kP) == po;
      Bop o2;
      b_load(o2, d1);
#pragma unroll
      for (int q = 0; q < Q1; ++q) {
        const int rt = w - 1 + NO * q;
        if (rt >= MT) break;
        update(v1[q], rt, o2, d1);
        if (isp) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            Ln[16 * rt + MF<R>::row(lane, r)] = mk<R>(v1[q].re[r], v1[q].im[r]);
        }
        // the other half of a finished block column is not read again
        if (o != 0) {
          if (rt < LT)
            tile_store<false>(w_tile(rt, place(d1)), v1[q], lane);
          else
            tile_store<true>(g_tile(rt, place(d1)), v1[q], lane);
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int row = psk[g4 + 4 * q];
        const C x1 = ent_value(e1, q, d1);
        if ((row >> 4) % NO != w - 1) continue;
        if (isp) Ln[row] = x1;
        if (o != 0) wput(row, place(d1), c16, x1);
      }
    }
    if (t == 64) cnt[0] = NO;  // the first units are dealt out
    lds_barrier();

    // ---- 3. the rest of the panel, while wave 0 factors the next one
    const int ngather = jj == 0 && kblk > 0 ? NB / 4 : 0;
    const int nzero = jj == kP ? NB / 8 : 0;
    const int nunit = ntile + 2 + ngather + nzero;
    auto grab = [&]() {
      int u = 0;
      if (lane == 0) u = atomicAdd(cnt, 1);
      return __builtin_amdgcn_readfirstlane(u);
    };
    int unext = w - 1;
    for (;;) {
      int u = unext;
      if (u >= nunit) break;
      // the entering elements of this unit are on their way; the next unit's
      // are asked for before this one's work
      const c128 e[2] = {e0[0], e0[1]};
      unext = grab();
      if (unext < ntile) ent_load(e0, unit_col(unext));
      if (u < ntile) {
        if (o != 0 && u == ntile - 1) {
          // block column J is finished: it becomes block column J + NCB
          LuTile<R> c;
          c.re = c.im = typename MF<R>::V{0, 0, 0, 0};
          for (int rt = 0; rt < LT; ++rt) tile_store<false>(w_tile(rt, jp), c, lane);
          for (int rt = LT; rt < MT; ++rt) tile_store<true>(g_tile(rt, jp), c, lane);
#pragma unroll
          for (int q = 0; q < 2; ++q) wput(psk[g4 + 4 * q], jp, c16, ent_value(e, q, NCB));
          continue;
        }
        const int d = d1 + 1 + u, p = place(d);
        // row tiles in global memory, four at a time, their loads in flight
        // over the tiles in LDS
        constexpr int GT = MT - LT < 4 ? (MT - LT > 0 ? MT - LT : 1) : 4;
        LuTile<R> v[GT];
        if constexpr (LT < MT) {
#pragma unroll
          for (int q = 0; q < GT; ++q) tile_load<true>(v[q], g_tile(LT + q, p), lane);
        }
        Bop o2;
        b_load(o2, d);
#pragma unroll
        for (int rt = 0; rt < LT; ++rt) {
          LuTile<R> c;
          tile_load<false>(c, w_tile(rt, p), lane);
          update(c, rt, o2, d);
          tile_store<false>(w_tile(rt, p), c, lane);
        }
        if constexpr (LT < MT) {
#pragma unroll
          for (int rt = LT; rt < MT; rt += GT) {
#pragma unroll
            for (int q = 0; q < GT; ++q)
              if (rt + q < MT) {
                update(v[q], rt + q, o2, d);
                tile_store<true>(g_tile(rt + q, p), v[q], lane);
                if (rt + GT + q < MT) tile_load<true>(v[q], g_tile(rt + GT + q, p), lane);
              }
          }
        }
        ent_store(e, d);
        u_out(d);
        continue;
      }
      u -= ntile;
      if (u == 0) {
        // multipliers by window row
        C* scr = lscr + ((kblk & 1) * 2 * BB + jj * 2 * NB);
        for (int row = lane; row < ROWS; row += 64) {
          const int md = meta[par * ROWS + row];
          if (md < 0) continue;
          const int st = md >> 16, wrow = md & 0xffff;
#pragma unroll
          for (int i = 0; i < kP; ++i)
            if (i < st) gst(scr + (i * 2 * NB + wrow), Lk[i * ROWS + row]);
        }
        continue;
      }
      if (u == 1) {
        // the panel's rows of U outside the window's block columns: zeros,
        // and the panel's own upper triangle
        const int k = lane & 7;
        u_out(d1);
        for (int te = 0; te < 3 * RPB; ++te) {
          if (te > tj && te < tj + NCB) continue;
          C* at = mats + (size_t)(kblk * 5 + 2 + te / RPB) * BB + (te % RPB) * 16 * NB + jj + k;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int c = (lane >> 3) + 8 * q, cp = c - o;
            if (te == tj && cp >= kP) continue;
            C v = mk<R>(0, 0);
            if (te == tj && cp >= k) v = Lt[(par * kP + k) * kP + cp];
            gst(at + c * NB, v);
          }
        }
        continue;
      }
      u -= 2;
      if (u < ngather) {
        // the previous block's multipliers into row order (P A_panel = Lh U)
        // and its permutation
        const int kp = kblk - 1, pp = kp & 1;
        const C* scr = lscr + pp * 2 * BB;
        for (int e = lane; e < 2 * NB; e += 64) {
          const int src = idx[pp * 2 * NB + e];
          if (u == 0) gst(permg + (size_t)kp * 2 * NB + e, (int16_t)src);
          C* at = mats + (size_t)(kp * 5 + (e < NB ? 0 : 1)) * BB + (e < NB ? e : e - NB);
          C v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = gld(scr + ((4 * u + q) * 2 * NB + src));
#pragma unroll
          for (int q = 0; q < 4; ++q) gst(at + (4 * u + q) * NB, v[q]);
        }
        continue;
      }
      u -= ngather;
      // the other parity's multipliers: zeros, for block k + 1
      C* scr = lscr + (((kblk + 1) & 1) * 2 * BB + u * 16 * NB);
      for (int e = lane; e < 16 * NB; e += 64) gst(scr + e, mk<R>(0, 0));
    }
    // what the waves wrote to global memory is read by others in later steps
    // of the block where the window is partly there, else not before the next
    // block
    if (LT < MT || up)
      __syncthreads();
    else
      lds_barrier();
    // ---- the next step's state
    jj += kP;
    if (o != 0) {
      if (++jp == NCB) jp = 0;
      if (++tj == RPB) tj = 0;
    }
    if (jj == NB) {
      jj = 0;
      ++kblk;
    }
  }
  // the last block's multipliers and permutation
  {
    const int kp = K - 1, pp = kp & 1;
    const C* scr = lscr + pp * 2 * BB;
    for (int c = w - 1; c < NB; c += NW - 1)
      for (int e = lane; e < 2 * NB; e += 64) {
        const int src = idx[pp * 2 * NB + e];
        if (c == 0) gst(permg + (size_t)kp * 2 * NB + e, (int16_t)src);
        gst(mats + (size_t)(kp * 5 + (e < NB ? 0 : 1)) * BB + c * NB + (e < NB ? e : e - NB),
            gld(scr + (c * 2 * NB + src)));
      }
  }
}

// In-place inverses of the unit lower Lh11 and the upper U(k,k) of every
// block by 16 x 16 tiles on MFMA: one workgroup per (system,
// block, which) and one wave per 16-column tile j of the inverse X, held in
// LDS (rows padded to 17 elements) by its rows that can be nonzero only:
// rows 16 j .. NB-1 of an L tile column, rows 0 .. 16 j + 15 of a U one,
// T (T + 1) / 2 tiles in all (T = NB / 16).  Each wave first inverts its diagonal
// tile by column recurrences on the already inverted part (16 lanes):
//   L = [1 0; l L22]:      L^{-1} column c below the diagonal = -L22^{-1} l
//   U = [U11 u; 0 ucc]:    U^{-1} column c above the diagonal = -U11^{-1} u / ucc
// then, after a barrier,
// runs the substitution down (L) or up (U) its tile column:
//   L: X(i,j) = -D(i)^{-1} sum_{k=j}^{i-1} L(i,k) X(k,j),   i = j+1 .. T-1
//   U: X(i,j) = -D(i)^{-1} sum_{k=i+1}^{j} U(i,k) X(k,j),   i = j-1 .. 0
// with D(i)^{-1} read from the diagonal tile of wave i's column; the sums
// are products of L or U tiles (fragments read from global memory) with the
// wave's own column (LDS), in Gauss form.  A wave hands values between its
// lanes through LDS under a wavefront fence.  All waves finish reading the
// block before the inverse is written over it.
template <typename R, int NB>
__global__ void __launch_bounds__(NB * 4)
k_block_invert_mfma(cx<R>* __restrict__ mats, int nblk) {
  constexpr int T = NB / 16;
  constexpr int LDT = 17;
  extern __shared__ __align__(16) char lds_raw[];
  cx<R>* Xs = reinterpret_cast<cx<R>*>(lds_raw);  // T (T + 1) / 2 tiles of 16 x LDT
  const int g = blockIdx.x;
  const int blk = g >> 1, which = g & 1;  // 0: Lh11 (slot 0), 1: U(k,k) (slot 2)
  if (blk >= nblk) return;
  cx<R>* M = mats + ((size_t)blk * 5 + (which ? 2 : 0)) * NB * NB;
  const int t = threadIdx.x, lane = t & 63;
  const int j = __builtin_amdgcn_readfirstlane(t >> 6);  // this wave's tile column
  // tile column i: X(r, c) at r LDT + c for its stored rows (16 i .. NB - 1 for
  // L, 0 .. 16 i + 15 for U); the tiles stored before it number
  // i T - i (i - 1) / 2 for L and i (i + 1) / 2 for U
  auto col = [&](int i) -> cx<R>* {
    const int before = which == 0 ? i * T - i * (i - 1) / 2 : i * (i + 1) / 2;
    const int r0 = which == 0 ? 16 * i : 0;
    return Xs + (size_t)(16 * before - r0) * LDT;
  };
  cx<R>* X = col(j);
  const int r0 = which == 0 ? 16 * j : 0;
  const int nrows = which == 0 ? NB - 16 * j : 16 * j + 16;
  auto wfence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // the column tile's stored rows: zero, with the diagonal tile of M at rows 16 j ..
  for (int e = lane; e < nrows * 16; e += 64) {
    const int r = r0 + e % nrows, c = e / nrows;
    cx<R> v = mk<R>(0, 0);
    if (r >= 16 * j && r < 16 * j + 16) v = M[(size_t)(16 * j + c) * NB + r];
    X[r * LDT + c] = v;
  }
  wfence();
  cx<R>* D = X + 16 * j * LDT;  // D(r, c) at r LDT + c
  const int r = lane;
  if (which == 0) {
    // unit lower: column c below the diagonal = -Dinv22 l (trailing part done)
    for (int c = 14; c >= 0; --c) {
      cx<R> acc = mk<R>(0, 0);
      if (r > c && r < 16) {
        acc = D[r * LDT + c];
        for (int q = c + 1; q < r; ++q) cmac(acc, D[r * LDT + q], D[q * LDT + c]);
      }
      wfence();
      if (r > c && r < 16) D[r * LDT + c] = mk<R>(-acc.x, -acc.y);
      wfence();
    }
    if (r < 16) {
      D[r * LDT + r] = mk<R>((R)1, (R)0);
      for (int c = r + 1; c < 16; ++c) D[r * LDT + c] = mk<R>(0, 0);
    }
  } else {
    // upper: column c above the diagonal = -Dinv11 u / d_cc (leading part done)
    for (int c = 0; c < 16; ++c) {
      const cx<R> d = cinv(D[c * LDT + c]);
      cx<R> acc = mk<R>(0, 0);
      if (r < c) {
        for (int q = r; q < c; ++q) cmac(acc, D[r * LDT + q], D[q * LDT + c]);
        acc = acc * d;
      }
      wfence();
      if (r < c) D[r * LDT + c] = mk<R>(-acc.x, -acc.y);
      if (r == c) D[r * LDT + r] = d;
      wfence();
    }
    if (r < 16)
      for (int c = 0; c < r; ++c) D[r * LDT + c] = mk<R>(0, 0);
  }
  __syncthreads();
  // substitution along the tile column; fragments of the D(i)^{-1} tile:
  // register s holds D(i)^{-1}(lane % 16, 4 s + lane / 16)
  auto dinv_frag = [&](Frag<R, 16>& f, int i) {
    const cx<R>* Di = col(i) + 16 * i * LDT;
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) f.a[s2] = Di[(lane & 15) * LDT + 4 * s2 + (lane >> 4)];
  };
  const int lo = which == 0 ? j + 1 : 0, hi = which == 0 ? T : j;
  for (int step = 0; step < hi - lo; ++step) {
    const int i = which == 0 ? lo + step : hi - 1 - step;
    const int k0 = which == 0 ? 16 * j : 16 * (i + 1);
    const int k1 = which == 0 ? 16 * i : 16 * (j + 1);
    Frag<R, NB> f;
    frag_load<R, NB>(f, M, i, lane, k0, k1);
    Acc<R, 1> acc;
    acc.zero();
    frag_mma<R, NB, 1, false>(acc, f, X, LDT, lane, k0, k1);
    acc_to_lds(acc, X, LDT, i, lane);  // the sum, at rows 16 i ..
    wfence();
    Frag<R, 16> fd;
    dinv_frag(fd, i);
    Acc<R, 1> acc2;
    acc2.zero();
    frag_mma<R, 16, 1, true>(acc2, fd, X + 16 * i * LDT, LDT, lane, 0, 16);
    wfence();
    acc_to_lds(acc2, X, LDT, i, lane);
    wfence();
  }
  __syncthreads();  // every wave has read M
  for (int e = lane; e < NB * 16; e += 64) {
    const int rr = e % NB, c = e / NB;
    const bool stored = rr >= r0 && rr < r0 + nrows;
    gst(M + (size_t)(16 * j + c) * NB + rr, stored ? X[rr * LDT + c] : mk<R>(0, 0));
  }
}

template <typename R>
static size_t invert_mfma_lds_bytes(int nb) {
  const size_t t = (size_t)nb / 16;
  return sizeof(cx<R>) * (t * (t + 1) / 2) * 16 * 17;
}

template <typename R, int NB>
static int launch_invert_mfma_nb(cx<R>* mats, int nblk, hipStream_t st) {
  const size_t smem = invert_mfma_lds_bytes<R>(NB);
  if (smem > kLdsBudget) return FB_ERR_INTERNAL;
  (void)hipFuncSetAttribute((const void*)k_block_invert_mfma<R, NB>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
  (void)hipGetLastError();
  k_block_invert_mfma<R, NB><<<2 * nblk, NB * 4, smem, st>>>(mats, nblk);
  FB_HIP(hipGetLastError());
  return 0;
}

// every block size up to 128 fits LDS in both precisions
template <typename R>
static int launch_invert_mfma(cx<R>* mats, int nb, int nblk, hipStream_t st) {
  if (invert_mfma_lds_bytes<R>(nb) > kLdsBudget) return FB_ERR_INTERNAL;
  int rc = 0;
  switch (nb) {
    case 16: rc = launch_invert_mfma_nb<R, 16>(mats, nblk, st); break;
    case 32: rc = launch_invert_mfma_nb<R, 32>(mats, nblk, st); break;
    case 48: rc = launch_invert_mfma_nb<R, 48>(mats, nblk, st); break;
    case 64: rc = launch_invert_mfma_nb<R, 64>(mats, nblk, st); break;
    case 80: rc = launch_invert_mfma_nb<R, 80>(mats, nblk, st); break;
    case 96: rc = launch_invert_mfma_nb<R, 96>(mats, nblk, st); break;
    case 112: rc = launch_invert_mfma_nb<R, 112>(mats, nblk, st); break;
    case 128: rc = launch_invert_mfma_nb<R, 128>(mats, nblk, st); break;
    default: return FB_ERR_INTERNAL;
  }
  return rc;
}

// M = Lh21 Lh11^{-1} in place of Lh21 (slot 1), one workgroup per block and
// one wave per 16 rows: a wave holds its rows of Lh21 as MFMA fragments and
// multiplies them by panels of PW columns of the lower triangular inverse
// staged in LDS (rows below the panel's first column only).  A wave reads and
// writes only its own rows of the slot.
template <typename R, int NB>
__global__ void __launch_bounds__(NB * 4)
k_form_m(cx<R>* __restrict__ mats, int nblk) {
  constexpr int PW = NB < 64 ? NB : 64;
  constexpr int NC = PW / 16;
  constexpr int LD = PW + 1;
  extern __shared__ __align__(16) char lds_raw[];
  cx<R>* Lp = reinterpret_cast<cx<R>*>(lds_raw);  // NB x LD: Lh11^{-1}(k, p0 + c) at k LD + c
  const int blk = blockIdx.x;
  if (blk >= nblk) return;
  const cx<R>* Li = mats + ((size_t)blk * 5 + 0) * NB * NB;
  cx<R>* L21 = mats + ((size_t)blk * 5 + 1) * NB * NB;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  Frag<R, NB> f;
  frag_load<R, NB>(f, L21, w, lane, 0, NB);
  for (int p0 = 0; p0 < NB; p0 += PW) {
    __syncthreads();
    // the last panel of a block that PW does not divide is partial: its
    // columns beyond the block are zeros and are not written
    for (int e = t; e < NB * PW; e += NB * 4) {
      const int k = e % NB, c = e / NB;
      Lp[k * LD + c] = p0 + c < NB ? Li[(size_t)(p0 + c) * NB + k] : mk<R>(0, 0);
    }
    __syncthreads();
    Acc<R, NC> acc;
    acc.zero();
    frag_mma<R, NB, NC, false>(acc, f, Lp, LD, lane, p0, NB);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + MF<R>::row(lane, r);
        const int col = p0 + 16 * c + (lane & 15);
        if (col < NB) gst(L21 + (size_t)col * NB + row, acc.get(c, r));
      }
  }
}

template <typename R, int NB>
static int launch_form_m_nb(cx<R>* mats, int nblk, hipStream_t st) {
  constexpr int PW = NB < 64 ? NB : 64;
  const size_t smem = sizeof(cx<R>) * (size_t)NB * (PW + 1);
  (void)hipFuncSetAttribute((const void*)k_form_m<R, NB>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
  (void)hipGetLastError();
  k_form_m<R, NB><<<nblk, NB * 4, smem, st>>>(mats, nblk);
  FB_HIP(hipGetLastError());
  return 0;
}

template <typename R>
static int launch_form_m(cx<R>* mats, int nb, int nblk, hipStream_t st) {
  switch (nb) {
    case 16: return launch_form_m_nb<R, 16>(mats, nblk, st);
    case 32: return launch_form_m_nb<R, 32>(mats, nblk, st);
    case 48: return launch_form_m_nb<R, 48>(mats, nblk, st);
    case 64: return launch_form_m_nb<R, 64>(mats, nblk, st);
    case 80: return launch_form_m_nb<R, 80>(mats, nblk, st);
    case 96: return launch_form_m_nb<R, 96>(mats, nblk, st);
    case 112: return launch_form_m_nb<R, 112>(mats, nblk, st);
    case 128: return launch_form_m_nb<R, 128>(mats, nblk, st);
    default: return FB_ERR_INTERNAL;
  }
}

// The blocks that let every solve sweep take one product phase per block
// row, from the inverses (slot 2: U(k,k)^{-1}, slot 0: Lh11^{-1}) and U's
// off-diagonal blocks:
//   Q  = U(k,k)^{-1} Lh11^{-1}  in place of Lh11^{-1} (slot 0),
//   G1 = U(k,k)^{-1} U(k,k+1)   in place of U(k,k+1)  (slot 3),
//   G2 = U(k,k)^{-1} U(k,k+2)   in place of U(k,k+2)  (slot 4).
// One workgroup per block and one wave per 16 rows: a wave holds its rows of
// the upper triangular inverse as MFMA fragments and multiplies them by
// panels of PW columns of each right operand staged in LDS, with the
// triangles that vanish in exact arithmetic (below the diagonal of U(k,k)^{-1},
// above it in Lh11^{-1} and U(k,k+2)) taken as zeros.  A panel is staged
// before any wave overwrites its columns.  Runs after k_form_m, which reads
// Lh11^{-1}.
template <typename R, int NB>
__global__ void __launch_bounds__(NB * 4)
k_form_qg(cx<R>* __restrict__ mats, int nblk) {
  constexpr int PW = NB < 64 ? NB : 64;
  constexpr int NC = PW / 16;
  constexpr int LD = PW + 1;
  extern __shared__ __align__(16) char lds_raw[];
  cx<R>* Bp = reinterpret_cast<cx<R>*>(lds_raw);  // NB x LD: operand(k, p0 + c) at k LD + c
  const int blk = blockIdx.x;
  if (blk >= nblk) return;
  cx<R>* base = mats + (size_t)blk * 5 * NB * NB;
  const cx<R>* Ui = base + (size_t)2 * NB * NB;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  Frag<R, NB> f;
  frag_load<R, NB>(f, Ui, w, lane, 16 * w, NB);
  {
    // fragment s holds row 16 w + lane % 16, column 4 s + lane / 16
    const int i = 16 * w + (lane & 15);
#pragma unroll
    for (int s = 0; s < NB / 4; ++s)
      if (4 * s + (lane >> 4) < i) f.a[s] = mk<R>(0, 0);
  }
  for (int which = 0; which < 3; ++which) {
    cx<R>* O = base + (size_t)(which == 0 ? 0 : which + 2) * NB * NB;
    const bool lower = which != 1;  // Lh11^{-1} and U(k,k+2)
    for (int p0 = 0; p0 < NB; p0 += PW) {
      __syncthreads();
      for (int e = t; e < NB * PW; e += NB * 4) {
        const int k = e % NB, c = e / NB;
        // a partial last panel (PW does not divide NB): zeros beyond the block
        cx<R> v = p0 + c < NB ? O[(size_t)(p0 + c) * NB + k] : mk<R>(0, 0);
        if (lower && k < p0 + c) v = mk<R>(0, 0);
        Bp[k * LD + c] = v;
      }
      __syncthreads();
      Acc<R, NC> acc;
      acc.zero();
      frag_mma<R, NB, NC, false>(acc, f, Bp, LD, lane, 16 * w, NB);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * w + MF<R>::row(lane, r);
          const int col = p0 + 16 * c + (lane & 15);
          if (col < NB) gst(O + (size_t)col * NB + row, acc.get(c, r));
        }
    }
  }
}

template <typename R, int NB>
static int launch_form_qg_nb(cx<R>* mats, int nblk, hipStream_t st) {
  constexpr int PW = NB < 64 ? NB : 64;
  const size_t smem = sizeof(cx<R>) * (size_t)NB * (PW + 1);
  (void)hipFuncSetAttribute((const void*)k_form_qg<R, NB>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
  (void)hipGetLastError();
  k_form_qg<R, NB><<<nblk, NB * 4, smem, st>>>(mats, nblk);
  FB_HIP(hipGetLastError());
  return 0;
}

template <typename R>
static int launch_form_qg(cx<R>* mats, int nb, int nblk, hipStream_t st) {
  switch (nb) {
    case 16: return launch_form_qg_nb<R, 16>(mats, nblk, st);
    case 32: return launch_form_qg_nb<R, 32>(mats, nblk, st);
    case 48: return launch_form_qg_nb<R, 48>(mats, nblk, st);
    case 64: return launch_form_qg_nb<R, 64>(mats, nblk, st);
    case 80: return launch_form_qg_nb<R, 80>(mats, nblk, st);
    case 96: return launch_form_qg_nb<R, 96>(mats, nblk, st);
    case 112: return launch_form_qg_nb<R, 112>(mats, nblk, st);
    case 128: return launch_form_qg_nb<R, 128>(mats, nblk, st);
    default: return FB_ERR_INTERNAL;
  }
}

template <typename R>
size_t lu_window_scratch(int b, int nsys) {
  size_t per = 0;
  switch (block_size(b)) {
    case 16: per = LuShape<R, 16>::SCRATCH; break;
    case 32: per = LuShape<R, 32>::SCRATCH; break;
    case 48: per = LuShape<R, 48>::SCRATCH; break;
    case 64: per = LuShape<R, 64>::SCRATCH; break;
    case 80: per = LuShape<R, 80>::SCRATCH; break;
    case 96: per = LuShape<R, 96>::SCRATCH; break;
    case 112: per = LuShape<R, 112>::SCRATCH; break;
    case 128: per = LuShape<R, 128>::SCRATCH; break;
  }
  return (size_t)nsys * per;
}

template <typename R, int NB>
static int launch_band_lu_nb(const LuArgs<R>& a, int nsys, hipStream_t st) {
  (void)hipFuncSetAttribute((const void*)k_band_lu<R, NB>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
  (void)hipGetLastError();
  k_band_lu<R, NB><<<nsys, kLuThreads, LuShape<R, NB>::LDS, st>>>(a);
  FB_HIP(hipGetLastError());
  return 0;
}

template <typename R>
static int launch_band_lu(const LuArgs<R>& a, int nb, int nsys, hipStream_t st) {
  switch (nb) {
    case 16: return launch_band_lu_nb<R, 16>(a, nsys, st);
    case 32: return launch_band_lu_nb<R, 32>(a, nsys, st);
    case 48: return launch_band_lu_nb<R, 48>(a, nsys, st);
    case 64: return launch_band_lu_nb<R, 64>(a, nsys, st);
    case 80: return launch_band_lu_nb<R, 80>(a, nsys, st);
    case 96: return launch_band_lu_nb<R, 96>(a, nsys, st);
    case 112: return launch_band_lu_nb<R, 112>(a, nsys, st);
    case 128: return launch_band_lu_nb<R, 128>(a, nsys, st);
    default: return FB_ERR_INTERNAL;
  }
}

// Transposed copy of every nb x nb factor block (32 x 32 tiles through LDS),
// read by the conjugate-transposed solves so that a wave's factor fragment
// loads are contiguous along the block's rows.
template <typename R>
__global__ void __launch_bounds__(256)
k_transpose_blocks(const cx<R>* __restrict__ src, cx<R>* __restrict__ dst, int nb) {
  __shared__ cx<R> tile[32][33];
  const size_t bb = (size_t)nb * nb;
  const cx<R>* S = src + (size_t)blockIdx.x * bb;
  cx<R>* D = dst + (size_t)blockIdx.x * bb;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int i0 = 0; i0 < nb; i0 += 32)
    for (int j0 = 0; j0 < nb; j0 += 32) {
      // tile of S at rows i0.., columns j0.. (element (i, j) at j * nb + i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = j0 + ty + 8 * q, i = i0 + tx;
        if (i < nb && j < nb) tile[ty + 8 * q][tx] = gld(S + (size_t)j * nb + i);
      }
      __syncthreads();
      // D(j, i) = S(i, j): D element (j, i) at i * nb + j
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + ty + 8 * q, j = j0 + tx;
        if (i < nb && j < nb) gst(D + (size_t)i * nb + j, tile[tx][ty + 8 * q]);
      }
      __syncthreads();
    }
}

template <typename R>
int launch_lu_impl(const Band& bd, int nsys, const c128* z_dev, cx<R>* mats, cx<R>* matsT,
                   int16_t* perm, int32_t* info, cx<R>* scratch, cx<R>* lscr, hipStream_t st) {
  const int b = bd.b;
  const int nb = block_size(b);
  const int K = (int)((bd.n + nb - 1) / nb);
  if (bd.Bblk == nullptr || bd.nb != nb) return FB_ERR_INTERNAL;
  const LuArgs<R> a{bd.Bblk, bd.n, K, z_dev, mats, perm, info, lscr, scratch};
  {
    ProfScope ps(FB_PROF_LU, st, 16.0 * (double)bd.n * b * b * nsys);
    FB_TRY(launch_band_lu<R>(a, nb, nsys, st));
  }
  int nblk = nsys * K;
  // inverses (2 nb^3 / 3 complex multiply-adds per block), M (nb^3 / 2) and
  // Q, G1, G2 (nb^3 / 3 + nb^3 / 2 + nb^3 / 3)
  ProfScope ps(FB_PROF_INVERT, st,
               8.0 * nblk * (double)nb * nb * nb * (2.0 / 3.0 + 0.5 + 7.0 / 6.0));
  FB_TRY(launch_invert_mfma<R>(mats, nb, nblk, st));
  FB_TRY(launch_form_m<R>(mats, nb, nblk, st));
  FB_TRY(launch_form_qg<R>(mats, nb, nblk, st));
  if (matsT) {
    k_transpose_blocks<R><<<5 * nblk, 256, 0, st>>>(mats, matsT, nb);
    FB_HIP(hipGetLastError());
  }
  return 0;
}

template int launch_lu_impl<float>(const Band&, int, const c128*, c64*, c64*, int16_t*,
                                   int32_t*, c64*, c64*, hipStream_t);
template int launch_lu_impl<double>(const Band&, int, const c128*, c128*, c128*, int16_t*,
                                    int32_t*, c128*, c128*, hipStream_t);
template size_t lu_window_scratch<float>(int, int);
template size_t lu_window_scratch<double>(int, int);

}  // namespace fb
