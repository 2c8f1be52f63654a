// Sylvester inertia of B - sigma I by band LDL^H without pivoting (FP64), in
// panels of four columns with the trailing window held in registers.
//
// One workgroup of four waves (one per SIMD) eliminates one shift.  The live
// window is T x T tiles of 16 x 16 (T = ceil((b + 16) / 16)), its lower half
// held in the accumulator layout of the FP64 MFMA; each diagonal of tiles
// belongs to one wave and moves down within that wave's registers when the
// window does.  A panel of four columns takes
//   publish  the owners of the pivot block's column copy the panel's raw
//            columns W (16 T x 4) to LDS,
//   pivots   every wave factors the panel's 4 x 4 diagonal block A11 pivot by
//            pivot, and thread j solves for column j of V = A11^{-1} W^H,
//   update   A22 -= W V: four real 16x16x4 MFMAs per complex tile, one per
//            real tile,
// with two barriers.  After four panels the entering 16 rows of the band,
// fetched to LDS meanwhile, take the places at the diagonals' ends.
//
// What bounds it: the serial chain of a panel (two LDS round trips, four
// pivots with their reciprocals, the solve), about 0.4 us, and the FP64 matrix
// rate of one CU (from T = 5 complex, T = 9 real about as long again).  Four
// columns per panel are one MFMA depth: wider panels need a longer serial
// factorisation of their diagonal block, narrower ones waste the instruction.
// Measured, one unblocked rank-one update per barrier before -> this kernel
// with the split below: complex n = 16384, b = 64, 17 shifts 29.3 -> 3.5 ms;
// real n = 12288, b = 113, 64 shifts 54.9 -> 2.0 ms; real n = 512, b = 8,
// 2 shifts 0.40 -> 0.095 ms.
//
// With few shifts the chain is also cut in two: one workgroup eliminates the
// leading rows downwards, another the trailing rows upwards (the same code on
// the reversed, conjugated band), and a third launch adds the two Schur
// complements on the 16-aligned separator between them and finishes it.
// In exact arithmetic every elimination order gives the same inertia as long
// as no pivot is zero, but without pivoting the digits that an order keeps
// depend on its smallest pivots.  A shift that meets a zero pivot, or one below
// 2^-34 ||B||_1 on the way up or in the separator, is redone in the plain order,
// leading rows first, whose counts are the documented ones.
#include <type_traits>

#include "fb_internal.h"
#include "prof.h"
#include "solve_kernel.h"

namespace fb {

namespace {

constexpr int kWaves = 4;
constexpr int kInertiaThreads = 64 * kWaves;
constexpr size_t kLdsBudget = 160 * 1024;
// shifts that a launch splits in two halves: their workgroups fill the chip
constexpr int kSplitShifts = 128;
// A pivot below kZero ||B||_1 is a zero one.  In the orders that only the split
// has, one below kSmall ||B||_1, which lets the elements grow until two thirds of
// their digits are lost, is reported as such, so that the plain order is taken.
// (Ordinary matrices have such pivots too, one in 1e9 or so; with 2^-26, one in 6
// million, every second launch of 128 shifts at n = 65536, b = 128 would meet
// one and be redone.)
constexpr double kZero = 0x1p-104;
constexpr double kSmall = 0x1p-34;

// ---- element types: complex Hermitian or real symmetric
__device__ __forceinline__ double re_of(double a) { return a; }
__device__ __forceinline__ double re_of(c128 a) { return a.x; }
__device__ __forceinline__ double im_of(double) { return 0.0; }
__device__ __forceinline__ double im_of(c128 a) { return a.y; }
__device__ __forceinline__ double scale(double a, double s) { return a * s; }
__device__ __forceinline__ c128 scale(c128 a, double s) { return mk(a.x * s, a.y * s); }
__device__ __forceinline__ double conj_of(double a) { return a; }
__device__ __forceinline__ c128 conj_of(c128 a) { return mk(a.x, -a.y); }
// v - a u
__device__ __forceinline__ double sub_prod(double v, double a, double u) { return fma(-a, u, v); }
__device__ __forceinline__ c128 sub_prod(c128 v, c128 a, c128 u) {
  return mk(fma(a.y, u.y, fma(-a.x, u.x, v.x)), fma(-a.y, u.x, fma(-a.x, u.y, v.y)));
}
// 1 / d: the hardware estimate, two Newton steps and a last one that rounds
// (50 cycles where the general division takes 77), in the range in which they
// hold
__device__ __forceinline__ double recip(double d) {
  if (__builtin_expect(!(fabs(d) > 1e-290 && fabs(d) < 1e290), 0)) return 1.0 / d;
  double r = __builtin_amdgcn_rcp(d);
#pragma unroll
  for (int i = 0; i < 3; ++i) r = fma(fma(-d, r, 1.0), r, r);
  return r;
}
template <bool CPLX>
struct Elem;
template <>
struct Elem<true> {
  using E = c128;
  static __device__ __forceinline__ E load(const c128* p) { return gld(p); }
  static __device__ __forceinline__ E real(double x) { return mk(x, 0.0); }
  static __device__ __forceinline__ E make(double x, double y) { return mk(x, y); }
};
template <>
struct Elem<false> {
  using E = double;
  static __device__ __forceinline__ E load(const c128* p) { return gld((const double*)p); }
  static __device__ __forceinline__ E real(double x) { return x; }
  static __device__ __forceinline__ E make(double x, double) { return x; }
};

// The tiles of each wave.  A tile keeps its distance from the diagonal as the
// window moves down a block, (hi, lo) -> (hi - 1, lo - 1), so that a whole
// diagonal of tiles belongs to one wave (the longest first, each to the wave
// with the fewest tiles so far) and moves within its registers.  The first
// slots of a wave are its tiles of block column 0, the ones it publishes.
template <int T>
struct Slots {
  int diags[kWaves];         // diagonals of a wave
  int tiles[kWaves];         // tiles of a wave
  int slots, pub;            // most tiles and most diagonals of a wave
  int hi[kWaves][2 * T], lo[kWaves][2 * T];
  int at[T][T];              // slot of tile (hi, lo) within its wave
  int owner[T];              // wave of diagonal hi - lo
  constexpr Slots()
      : diags{}, tiles{}, slots(0), pub(0), hi{}, lo{}, at{}, owner{} {
    for (int d = 0; d < T; ++d) {
      int best = 0;
      for (int w = 1; w < kWaves; ++w)
        if (tiles[w] < tiles[best]) best = w;
      owner[d] = best;
      tiles[best] += T - d;
    }
    for (int w = 0; w < kWaves; ++w) {
      int n = 0;
      for (int l = 0; l < T; ++l)
        for (int d = 0; d + l < T; ++d)
          if (owner[d] == w) {
            hi[w][n] = d + l;
            lo[w][n] = l;
            at[d + l][l] = n++;
            if (l == 0) ++diags[w];
          }
      for (; n < 2 * T; ++n) {  // empty slots: never published
        hi[w][n] = 0;
        lo[w][n] = 1;
      }
      slots = tiles[w] > slots ? tiles[w] : slots;
      pub = diags[w] > pub ? diags[w] : pub;
    }
  }
};

enum Mode : int { kFull = 0, kHalves = 1, kMiddle = 2 };

struct InertiaArgs {
  const c128* Bd;
  int64_t n;
  int b;
  const double* shifts;
  const double* stats;
  int32_t* counts;  // 3 per shift
  int mode;
  int gated;        // kFull: only shifts whose counts hold a zero or small pivot
  double tiny[2];   // relative limit of a zero pivot, downwards and upwards
  int h0, h1;       // blocks of 16 rows eliminated from the top and the bottom
  int32_t* part;    // 4 per shift: (neg, zero) of the two halves
  c128* dump;       // 2 per shift: the window left by a half, tile by tile
};

// entering entries: diagonals -15 .. 16 (T - 1) + 15 of 16 rows padded to 17
template <int T>
constexpr int kEnter = (16 * (T - 1) + 31) * 17;

// A column of a panel in LDS: 16 T rows, row 16 X + r at 16 X + 4 (r % 4) +
// r / 4, so that the four accumulator registers of a lane (rows l / 16 + 4 r)
// are one run; the stride puts the panel's four columns on different banks.
template <int T>
constexpr int kCol = 16 * T + (T % 2 ? 24 : 8);

template <int T, bool CPLX>
constexpr size_t inertia_lds_bytes() {
  // W double-buffered and V, four columns each, and the entering rows with a
  // place for what lies outside the band; real and imaginary parts apart, so
  // that an MFMA operand is read without register moves
  return sizeof(double) * (CPLX ? 2 : 1) * (size_t)(3 * 4 * kCol<T> + kEnter<T> + 1);
}

template <int T, bool CPLX>
__global__ void __launch_bounds__(kInertiaThreads, 1) k_band_inertia(InertiaArgs a) {
  using E = typename Elem<CPLX>::E;
  using Ld = Elem<CPLX>;
  constexpr int R = 16 * T;
  constexpr Slots<T> tab{};
  constexpr int NS = tab.slots;
  extern __shared__ __align__(16) char lds_raw[];
  // real parts, then (CPLX) imaginary parts PL doubles further on
  constexpr int RS = kCol<T>;
  constexpr int PL = 3 * 4 * RS + kEnter<T> + 1;
  double* Wl = reinterpret_cast<double*>(lds_raw);  // [2][4][RS]
  double* Vl = Wl + 2 * 4 * RS;                     // [4][RS]
  double* El = Vl + 4 * RS;  // A(16 X + r, 16 X + r - d) at 17 (d + 15) + r
  auto rowpos = [](int r) { return (r & ~15) + 4 * (r & 3) + ((r >> 2) & 3); };
  auto lget = [&](const double* p) -> E { return Ld::make(p[0], CPLX ? p[PL] : 0.0); };
  auto lput = [&](double* p, E v) {
    p[0] = re_of(v);
    if constexpr (CPLX) p[PL] = im_of(v);
  };

  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int half = a.mode == kHalves ? (blockIdx.x & 1) : 0;
  const int s = a.mode == kHalves ? blockIdx.x >> 1 : blockIdx.x;
  if (a.gated && a.counts[3 * s + 1] == 0) return;
  const int64_t n = a.n;
  const int b = a.b;
  const c128* Bd = a.Bd;
  const double sigma = a.shifts[s];
  const double pivmin = a.tiny[half] * a.stats[0];
  const double pad = 1.0 + 2.0 * pivmin;  // a pivot that is never tiny
  // rows of this elimination and of them the ones it eliminates
  const int64_t sep0 = (int64_t)16 * a.h0;                       // first separator row
  const int64_t S = n - (int64_t)16 * (a.h0 + a.h1);             // separator rows
  const int64_t nv = a.mode == kMiddle ? S : n;
  const int64_t ncols = a.mode == kHalves ? (int64_t)16 * (half ? a.h1 : a.h0) : nv;
  const c128* dump0 = nullptr;
  const c128* dump1 = nullptr;
  constexpr size_t kDump = (size_t)T * (T + 1) / 2 * 256;
  if (a.mode == kMiddle) {
    dump0 = a.dump + (size_t)(2 * s) * kDump;
    dump1 = dump0 + kDump;
  }

  // A(i, i - d) of the shifted band in this elimination's row order (the
  // reversed half reads the conjugate, which has the same inertia); pad on the
  // diagonal beyond the last row.  Out-of-range elements read element 0 and are
  // replaced, so that the loads stay branch-free.
  auto band_off = [&](int64_t i, int d) -> int64_t {
    const bool ok = d >= 0 && d <= b && i < n && i - d >= 0;
    return ok ? (int64_t)d * n + (half ? n - 1 - i : i - d) : 0;
  };
  auto band_val = [&](E v, int64_t i, int d) -> E {
    if (i >= n) return Ld::real(d == 0 ? pad : 0.0);
    if (d < 0 || d > b) return Ld::real(0.0);
    if (d == 0) return Ld::real(re_of(v) - sigma);
    return v;
  };
  auto dump_at = [&](const c128* D, int i, int j) -> E {  // i >= j
    const int X = i >> 4, J = j >> 4;
    return Ld::load(D + (size_t)(X * (X + 1) / 2 + J) * 256 + (i & 15) * 16 + (j & 15));
  };

  // ---- tiles of this wave: slot e holds the tile at block row hi[e], block
  // column lo[e] of the window, counted from the pivot block
  mf_d4 tr[NS], ti[CPLX ? NS : 1];
  int hi[NS], lo[NS];
#pragma unroll
  for (int e = 0; e < NS; ++e) {
    hi[e] = w == 0 ? tab.hi[0][e] : w == 1 ? tab.hi[1][e] : w == 2 ? tab.hi[2][e] : tab.hi[3][e];
    lo[e] = w == 0 ? tab.lo[0][e] : w == 1 ? tab.lo[1][e] : w == 2 ? tab.lo[2][e] : tab.lo[3][e];
  }
  const int c16 = lane & 15, r4 = lane >> 4;
#pragma unroll
  for (int e = 0; e < NS; ++e) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * hi[e] + r4 + 4 * r, j = 16 * lo[e] + c16, d = i - j;
      E v;
      if (a.mode == kMiddle) {
        if (i >= S || j >= S) {
          v = Ld::real(d == 0 ? pad : 0.0);
        } else if (d < 0) {
          v = Ld::real(0.0);
        } else {
          // top's Schur complement + bottom's (reversed) - the matrix itself
          const E x = dump_at(dump0, i, j);
          const E y = dump_at(dump1, (int)S - 1 - j, (int)S - 1 - i);
          E z = Ld::real(0.0);
          if (d <= b) z = band_val(Ld::load(Bd + band_off(sep0 + i, d)), sep0 + i, d);
          if constexpr (CPLX)
            v = mk(x.x + (y.x - z.x), x.y + (y.y - z.y));
          else
            v = x + (y - z);
        }
      } else {
        v = band_val(Ld::load(Bd + band_off(i, d)), i, d);
      }
      if constexpr (CPLX) {
        tr[e][r] = v.x;
        ti[e][r] = v.y;
      } else {
        tr[e][r] = v;
      }
    }
  }

  // diagonals outside the band stay zero
  for (int e = t; e < kEnter<T>; e += kInertiaThreads) lput(El + e, Ld::real(0.0));

  int neg = 0, zero = 0, par = 0;
  // whole blocks: the columns past the last are the padding's, whose pivots
  // count as positive
  const int nblk = (int)((ncols + 15) / 16);
  constexpr int NPF = T;  // (16 (T - 1) + 1) 16 entries over 256 threads
  E pf[NPF];
  const c128* pfp[NPF];  // this thread's entries of the next block row to enter
  int pfl[NPF];          // and their places in LDS
#pragma unroll
  for (int q = 0; q < NPF; ++q) {
    const int e = t + q * kInertiaThreads, d = e >> 4, r = e & 15;
    const int64_t i = 16 * T + r;
    pfp[q] = Bd + (int64_t)min(d, b) * n + (half ? n - 1 - i : i - min(d, b));
    pfl[q] = d <= b ? 3 * 4 * RS + (d + 15) * 17 + r : 3 * 4 * RS + kEnter<T>;
  }
#pragma unroll 1
  for (int blk = 0; blk < nblk; ++blk) {
    // entering block row, fetched over the block's four panels
    const bool last = a.mode != kHalves && blk + 1 == nblk;
    const int64_t X16 = 16 * ((int64_t)blk + T);
    if (!last) {
      if (X16 + 16 <= n) {
#pragma unroll
        for (int q = 0; q < NPF; ++q) pf[q] = Ld::load(pfp[q]);
      } else {
        // rows past the last: a diagonal of at least pad once sigma is off it
#pragma unroll
        for (int q = 0; q < NPF; ++q) {
          const int e = t + q * kInertiaThreads;
          const bool in = X16 + (e & 15) < n;
          pf[q] = Ld::load(in ? pfp[q] : Bd);
          if (!in) pf[q] = Ld::real(e < 16 ? pad + 2.0 * fabs(sigma) : 0.0);
        }
      }
#pragma unroll
      for (int q = 0; q < NPF; ++q) pfp[q] += half ? -16 : 16;
    }
#pragma unroll
    for (int pan = 0; pan < 4; ++pan) {
      const int o = 4 * pan;
      const int wcur = par * 4 * RS;
      const double* W = Wl + wcur;
      par ^= 1;
      // ---- publish the panel's columns (the tiles of the pivot block's column)
#pragma unroll
      for (int e = 0; e < tab.pub; ++e) {
        // (one comparison per lane: column c16 - o of the panel, block column 0)
        const unsigned kk = (unsigned)(c16 - o) | ((unsigned)lo[e] << 4);
        if (__builtin_expect(kk < 4, 1)) {
          const int at = wcur + 16 * hi[e] + (int)kk * RS + 4 * r4;
          *reinterpret_cast<mf_d4*>(Wl + at) = tr[e];
          if constexpr (CPLX) *reinterpret_cast<mf_d4*>(Wl + at + PL) = ti[e];
        }
      }
      __syncthreads();
      // ---- pivots of the 4 x 4 diagonal block: l(c, k) = a(c, k) / d_k
      E a11[4][4], l[4][4], v[4];
      double rd[4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = c; r < 4; ++r) a11[r][c] = lget(W + c * RS + 4 * r + pan);
      // thread j takes row j of the panel (a thread past the last repeats it)
      const int j = rowpos(min(t, R - 1));
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = conj_of(lget(W + q * RS + j));
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double dk = re_of(a11[k][k]);
        const bool tiny = fabs(dk) < pivmin;
        zero += tiny ? 1 : 0;
        neg += !tiny && dk < 0.0 ? 1 : 0;
        dk = tiny ? -pivmin : dk;
        rd[k] = recip(dk);
#pragma unroll
        for (int c = k + 1; c < 4; ++c) {
          l[c][k] = scale(a11[c][k], rd[k]);
#pragma unroll
          for (int r = c; r < 4; ++r)
            a11[r][c] = sub_prod(a11[r][c], a11[r][k], conj_of(l[c][k]));
        }
      }
      // column j of V = A11^{-1} W^H: L z = w, x = z / d, L^H v = x
#pragma unroll
      for (int k = 1; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < k; ++c) v[k] = sub_prod(v[k], l[k][c], v[c]);
#pragma unroll
      for (int k = 3; k >= 0; --k) {
        v[k] = scale(v[k], rd[k]);
#pragma unroll
        for (int c = k + 1; c < 4; ++c) v[k] = sub_prod(v[k], conj_of(l[c][k]), v[c]);
      }
      if (__builtin_expect(t < R, 1)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) lput(Vl + q * RS + j, v[q]);
      }
      if (pan == 3 && !last) {
#pragma unroll
        for (int q = 0; q < NPF; ++q) {
          E x = pf[q];
          // (keeps the wait for the loads here)
          if constexpr (CPLX)
            asm volatile("" : "+v"(x.x), "+v"(x.y));
          else
            asm volatile("" : "+v"(x));
          if (q == 0 && t < 16) x = Ld::real(re_of(x) - sigma);
          lput(Wl + pfl[q], x);
        }
      }
      __syncthreads();
      // ---- update of every tile: a tile that the panel does not reach
      // subtracts zeros, one whose columns it has just finished is not read
      // again, and both cost less than a branch per tile
      const double* Wr = W + r4 * RS + rowpos(c16);
      const double* Vr = Vl + r4 * RS + rowpos(c16);
#pragma unroll
      for (int e = 0; e < NS; ++e) {
        const E x = lget(Wr + 16 * hi[e]), y = lget(Vr + 16 * lo[e]);
        if constexpr (CPLX) {
          tr[e] = MF<double>::mma(-x.x, y.x, tr[e]);
          ti[e] = MF<double>::mma(-x.x, y.y, ti[e]);
          tr[e] = MF<double>::mma(x.y, y.y, tr[e]);
          ti[e] = MF<double>::mma(-x.y, y.x, ti[e]);
        } else {
          tr[e] = MF<double>::mma(-x, y, tr[e]);
        }
      }
    }
    // ---- the window moves down a block: tile (i, j) becomes (i - 1, j - 1),
    // and each diagonal's last tile is the entering block row's
    if (!last) {
      auto move = [&](auto wave) {
        constexpr int w2 = decltype(wave)::value;
#pragma unroll
        for (int d = 0; d < T; ++d) {
          if (tab.owner[d] != w2) continue;
#pragma unroll
          for (int l = 0; l + 1 < T - d; ++l) {
            tr[tab.at[d + l][l]] = tr[tab.at[d + l + 1][l + 1]];
            if constexpr (CPLX) ti[tab.at[d + l][l]] = ti[tab.at[d + l + 1][l + 1]];
          }
          const int e = tab.at[T - 1][T - 1 - d];
          const double* Ep = El + (16 * d + r4 - c16 + 15) * 17 + r4;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const E x = lget(Ep + 4 * r * 18);
            tr[e][r] = re_of(x);
            if constexpr (CPLX) ti[e][r] = im_of(x);
          }
        }
      };
      if (w == 0)
        move(std::integral_constant<int, 0>{});
      else if (w == 1)
        move(std::integral_constant<int, 1>{});
      else if (w == 2)
        move(std::integral_constant<int, 2>{});
      else
        move(std::integral_constant<int, 3>{});
    }
  }

  if (a.mode == kHalves) {
    c128* D = a.dump + (size_t)(2 * s + half) * kDump;
#pragma unroll
    for (int e = 0; e < NS; ++e) {
      if (lo[e] > hi[e]) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        c128* at = D + (size_t)(hi[e] * (hi[e] + 1) / 2 + lo[e]) * 256 + (r4 + 4 * r) * 16 + c16;
        if constexpr (CPLX)
          gst(at, mk(tr[e][r], ti[e][r]));
        else
          gst((double*)at, tr[e][r]);
      }
    }
    if (t == 0) {
      a.part[4 * s + 2 * half] = neg;
      a.part[4 * s + 2 * half + 1] = zero;
    }
    return;
  }
  if (t == 0) {
    if (a.mode == kMiddle) {
      neg += a.part[4 * s] + a.part[4 * s + 2];
      zero += a.part[4 * s + 1] + a.part[4 * s + 3];
    }
    a.counts[3 * s + 0] = neg;
    a.counts[3 * s + 1] = zero;
    a.counts[3 * s + 2] = (int32_t)(n - neg - zero);
  }
}

template <int T, bool CPLX>
int launch_t(const InertiaArgs& a, int grid, hipStream_t st) {
  const size_t smem = inertia_lds_bytes<T, CPLX>();
  static_assert(inertia_lds_bytes<9, true>() <= kLdsBudget, "LDS");
  (void)hipFuncSetAttribute((const void*)k_band_inertia<T, CPLX>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBudget);
  (void)hipGetLastError();
  k_band_inertia<T, CPLX><<<grid, kInertiaThreads, smem, st>>>(a);
  FB_HIP(hipGetLastError());
  return 0;
}

template <bool CPLX>
int launch_any(const InertiaArgs& a, int tiles, int grid, hipStream_t st) {
  switch (tiles) {
    case 2: return launch_t<2, CPLX>(a, grid, st);
    case 3: return launch_t<3, CPLX>(a, grid, st);
    case 4: return launch_t<4, CPLX>(a, grid, st);
    case 5: return launch_t<5, CPLX>(a, grid, st);
    case 6: return launch_t<6, CPLX>(a, grid, st);
    case 7: return launch_t<7, CPLX>(a, grid, st);
    case 8: return launch_t<8, CPLX>(a, grid, st);
    case 9: return launch_t<9, CPLX>(a, grid, st);
    default: return FB_ERR_INTERNAL;
  }
}

int window_tiles(int b) { return (b + 31) / 16; }

// The halves pay for two more launches and the separator's b columns: taken
// when the rows they share out are well more than that.
bool splits(const Band& bd, int nshift) {
  return nshift <= kSplitShifts && bd.n >= 2 * (int64_t)bd.b + 512;
}

}  // namespace

size_t inertia_scratch_bytes(const Band& bd, int nshift) {
  const int k = nshift < kSplitShifts ? nshift : kSplitShifts;
  if (k <= 0 || !splits(bd, k)) return 0;
  const size_t t = (size_t)window_tiles(bd.b);
  return (size_t)k * (2 * (t * (t + 1) / 2) * 256 * sizeof(c128) + 4 * sizeof(int32_t));
}

// scratch: inertia_scratch_bytes for at least nshift shifts, or nullptr (every
// shift is then eliminated by one workgroup)
int launch_inertia(const Band& bd, int nshift, const double* shifts_dev, int32_t* cnt_dev,
                   void* scratch, hipStream_t st) {
  if (nshift <= 0) return 0;
  const int tiles = window_tiles(bd.b);
  InertiaArgs a{};
  a.Bd = bd.Bd;
  a.n = bd.n;
  a.b = bd.b;
  a.shifts = shifts_dev;
  a.stats = bd.stats;
  a.counts = cnt_dev;
  a.tiny[0] = kZero;
  auto go = [&](int grid) {
    return bd.cplx ? launch_any<true>(a, tiles, grid, st) : launch_any<false>(a, tiles, grid, st);
  };
  ProfScope ps(FB_PROF_INERTIA, st, 4.0 * (double)bd.n * bd.b * bd.b * nshift);
  if (scratch == nullptr || !splits(bd, nshift)) {
    a.mode = kFull;
    return go(nshift);
  }
  const size_t t = (size_t)tiles;
  a.dump = (c128*)scratch;
  a.part = (int32_t*)((char*)scratch +
                      (size_t)nshift * 2 * (t * (t + 1) / 2) * 256 * sizeof(c128));
  const int64_t blocks = (bd.n - bd.b) / 16;  // the separator keeps b .. b + 15 rows
  a.h0 = (int)((blocks + 1) / 2);
  a.h1 = (int)(blocks / 2);
  a.tiny[1] = kSmall;
  a.mode = kHalves;
  FB_TRY(go(2 * nshift));
  a.tiny[0] = kSmall;
  a.mode = kMiddle;
  FB_TRY(go(nshift));
  a.tiny[0] = kZero;
  a.mode = kFull;
  a.gated = 1;
  return go(nshift);
}

}  // namespace fb
