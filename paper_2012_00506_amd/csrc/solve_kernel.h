// MFMA block-solve kernel templates (instantiated per precision in
// solve_f32.hip and solve_f64.hip).
#pragma once
#include <type_traits>

#include "fb_internal.h"
#include "mfma.h"
#include "prof.h"
#include "solve_job.h"
#include "tune.h"

namespace fb {

static __device__ __forceinline__ int remap_job(int bid, int njobs) {
  // consecutive jobs (one system's tiles) on one XCD: workgroups are dealt
  // to the 8 XCDs round-robin, so XCD x runs the x-th contiguous range
  const int per = (njobs + 7) / 8;
  return (bid % 8) * per + bid / 8;
}


// Chunk of op(A): columns 16 ch .. 16 ch + 15 for the wave's 16 rows, element
// (16 w + lane % 16, 16 ch + 4 q + lane / 16) in a[q].
template <typename R>
struct Ck {
  cx<R> a[4];
};

// ---------------------------------------------------------------- MFMA block solve
// NB / 16 waves per job, wave w computing rows 16 w .. 16 w + 15 of every
// product for the tile's 16 NC columns.  Tiles are computed transposed (the
// right-hand sides are the first MFMA operand), so that a lane's
// accumulators belong to one block row, lane % 16, and four columns: 16 lanes
// cover 16 consecutive rows of a column, and right-hand sides, intermediates
// and solutions move between global memory and the accumulators in runs of
// 128 or 256 bytes, without a detour through LDS.  LDS holds three slots of
// NB x 16 NC (panels of 16 columns; within a row the columns are permuted by
// the row, which keeps the accumulators' writes off each other's banks) and
// the block's permutation.  Factor fragments stream from L2 RD chunks ahead
// of the MFMAs that use them, across products, barriers and steps.
//
// What bounds it: the MFMAs (4 NB complex multiply-adds per element of x) and,
// not fully overlapped, the right-hand sides, intermediates and solutions in
// HBM (48 bytes per element of x, 64 for a correction).  Sweeps are chains of
// steps, so that several workgroups have to share a CU: three slots instead of
// staging buffers for every transfer, loads and stores without branches in
// full tiles, and registers for two waves per SIMD or more.  At n = 16384,
// complex64, b = 64, 64 system-directions of 1400 columns: 23.4 ms (MFMA
// alone 15, HBM alone 14.6) against 40.4 in a form that staged every tile
// through LDS; b = 128, 64 of 576: 19.5 against 34.8 (12.3); complex128, b =
// 64, 48 of 1056: 27.7 against 37.6 (17.6).
template <typename R, int NB, int NC>
__global__ void __launch_bounds__(NB * 4, 2)
k_band_solve(const cx<R>* __restrict__ mats, const cx<R>* __restrict__ matsT,
             const int16_t* __restrict__ permg, int64_t n, int K,
             const SolveJob* __restrict__ jobs, int njobs, const int32_t* __restrict__ gate) {
  constexpr bool TS = sizeof(R) == 4;  // H solves read the transposed copy
  constexpr int NCH = NB / 16;
  constexpr int L = 2 * NCH;
  constexpr int RD = NCH < 2 ? NCH : 2;  // chunks in flight
  constexpr int T = 16 * NC;
  constexpr int SL = NB * T;                   // elements of a slot
  constexpr int RB = 16 * (int)sizeof(cx<R>);  // bytes of a panel row
  using E = cx<R>;
  using Acc1 = Acc<R, NC>;
  extern __shared__ __align__(16) char lds_raw[];
  E* S = reinterpret_cast<E*>(lds_raw);
  uint16_t* spt = reinterpret_cast<uint16_t*>(lds_raw + 3 * SL * sizeof(E));  // gather offsets
  uint16_t* spo = spt + NB;                                                    // window row offsets
  const int job = remap_job(blockIdx.x, njobs);
  if (job >= njobs) return;
  const SolveJob jb = jobs[job];
  if (gate && !gate[jb.grp]) return;  // a correction its group no longer needs
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const int row = 16 * w + li;  // the lane's block row
  const size_t bb = (size_t)NB * NB;
  const E* F = mats + (size_t)jb.sys * K * 5 * bb;
  const E* FT = TS ? matsT + (size_t)jb.sys * K * 5 * bb : F;
  const int16_t* P = permg + (size_t)jb.sys * K * 2 * NB;
  const int ncol = jb.ncol;
  auto blk = [&](int k, int slot) { return F + ((size_t)k * 5 + slot) * bb; };
  auto blkh = [&](int k, int slot) { return FT + ((size_t)k * 5 + slot) * bb; };

  // ---- global tiles in accumulator order.  Columns beyond ncol read the
  // first one (never stored); rows beyond n are zeroed by the user.
  const int colg = MF<R>::row(lane, 0), colr = MF<R>::row(0, 1);
  auto col_of = [&](int c, int r) { return 16 * c + colg + colr * r; };
  auto gtile = [&](auto (&v)[NC][4], auto base, int64_t ld, int k) {
    const int64_t i = (int64_t)k * NB + row;
    const auto p0 = base + (i < n ? i : n - 1);
    const auto pl = p0 + colg * ld;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        v[c][r] = gld(col_of(c, r) < ncol ? pl + (16 * c + colr * r) * ld : p0);
  };
  auto rowok = [&](int k) { return (int64_t)k * NB + row < n; };
  auto gput = [&](const auto (&v)[NC][4], auto base, int64_t ld, int k) {
    auto pl = base + ((int64_t)k * NB + row) + colg * ld;
    if (ncol == T && (int64_t)(k + 1) * NB <= n) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) gst(pl + (16 * c + colr * r) * ld, v[c][r]);
    } else if (rowok(k)) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (col_of(c, r) < ncol) gst(pl + (16 * c + colr * r) * ld, v[c][r]);
    }
  };
  E* mid = reinterpret_cast<E*>(jb.mid) + (int64_t)jb.col0 * jb.ldmid;
  c128* out = jb.out + (int64_t)jb.col0 * jb.ldout;

  // ---- LDS tiles.  Element (row i, column c) of a slot: panel c / 16, row
  // i, place (c % 16) ^ 4 (i % 4).
  auto lput = [&](E* panel, int sw, const E (&v)[4]) {
    if constexpr (sizeof(R) == 4) {
      float4* p = reinterpret_cast<float4*>(panel + ((4 * kq) ^ (sw << 2)));
      p[0] = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
      p[1] = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) panel[kq + 4 * (r ^ sw)] = v[r];
    }
  };
  auto lget = [&](const E* panel, int sw, E (&v)[4]) {
    if constexpr (sizeof(R) == 4) {
      const float4* p = reinterpret_cast<const float4*>(panel + ((4 * kq) ^ (sw << 2)));
      const float4 a = p[0], b = p[1];
      v[0] = mk<R>(a.x, a.y);
      v[1] = mk<R>(a.z, a.w);
      v[2] = mk<R>(b.x, b.y);
      v[3] = mk<R>(b.z, b.w);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const E* p = panel + kq + 4 * (r ^ sw);
        v[r] = mk<R>(p->x, p->y);
      }
    }
  };
  auto put_own = [&](int slot, const E (&v)[NC][4]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) lput(S + slot * SL + (c * NB + row) * 16, li & 3, v[c]);
  };
  auto get_own = [&](int slot, E (&v)[NC][4]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) lget(S + slot * SL + (c * NB + row) * 16, li & 3, v[c]);
  };
  // window row d of slots 0 (rows 0 .. NB - 1) and 1 (NB .. 2 NB - 1): byte
  // offset of its row in panel 0, and 4 (d % 4) elements in the low bits
  auto woff = [&](int d) {
    return (d < NB ? d : d + NB * (NC - 1)) * RB + (d & 3) * 4 * (int)sizeof(E);
  };
  auto win = [&](int off, int c) {
    return reinterpret_cast<E*>(lds_raw + (off & ~(RB - 1)) + c * NB * RB);
  };
  auto win_sw = [&](int off) { return (off & (RB - 1)) / (4 * (int)sizeof(E)); };
  // row d of a tile in registers, in the factors' type
  auto conv = [&](const auto (&v)[NC][4], bool ok, E (&x)[NC][4]) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[c][r] = mk<R>(ok ? (R)v[c][r].x : (R)0, ok ? (R)v[c][r].y : (R)0);
  };
  auto acc_set = [&](Acc1& acc, const E (&v)[NC][4]) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc.set(c, r, v[c][r]);
  };
  auto acc_get = [&](const Acc1& acc, E (&v)[NC][4]) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[c][r] = acc.get(c, r);
  };
  // the solution's rows of block k (added to the old values for a correction)
  auto emit = [&](const E (&x)[NC][4], const c128 (&old)[NC][4], int k) {
    c128 o[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o[c][r] = mk((double)x[c][r].x, (double)x[c][r].y);
        if (jb.add) o[c][r] = old[c][r] + o[c][r];
      }
    gput(o, out, jb.ldout, k);
  };
  // permutation of block k: one entry per thread (again from the first
  // beyond 2 NB)
  const int pe = t % (2 * NB);
  auto perm_get = [&](int k) { return gld(P + (size_t)k * 2 * NB + pe); };
  auto perm_put = [&](int v) {
    const uint16_t o = (uint16_t)woff(v);
    spo[pe] = o;
    // gather order of the top rows: entry 16 ch + 4 q + kq at [ch][kq][q]
    if (pe < NB) spt[(pe & ~15) + 4 * (pe & 3) + ((pe >> 2) & 3)] = o;
  };

  // ---- products
  auto ck_load = [&](Ck<R>& c, const E* A, bool tr, int ch) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * ch + 4 * q;
      c.a[q] = tr ? gld(A + k + (row * NB + kq)) : gld(A + k * NB + (kq * NB + row));
    }
  };
  // rows 16 ch + 4 q + kq of a slot, column li of every panel
  auto b_slot = [&](int slot) {
    return [=](int ch, E (&bv)[4][NC]) {
      const E* p = S + slot * SL + kq * 16 + (li ^ (kq << 2));
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < NC; ++c) bv[q][c] = p[(c * NB + 16 * ch + 4 * q) * 16];
    };
  };
  Ck<R> carry[RD];
  auto mma = [&](Acc1& acc, const Ck<R>& ck, const E (&bv)[4][NC], bool conj, bool neg) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      R ar = ck.a[q].x, ai = conj ? -ck.a[q].y : ck.a[q].y;
      if (neg) {
        ar = -ar;
        ai = -ai;
      }
      const R as = ar + ai;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        acc.p1[c] = MF<R>::mma(bv[q][c].x, ar, acc.p1[c]);
        acc.p2[c] = MF<R>::mma(bv[q][c].y, ai, acc.p2[c]);
        acc.p3[c] = MF<R>::mma(bv[q][c].x + bv[q][c].y, as, acc.p3[c]);
      }
    }
  };
  // acc += op(A0) B0, mid(), acc -= op(A1) B1 (neg0: acc -= op(A0) B0); carry
  // holds the first chunks of A0 on entry and of An (the next step's A0) on exit
  auto step = [&](Acc1& acc, const E* A0, const E* A1, const E* An, auto B0, auto B1, bool conj,
                  bool neg0, auto midf) {
    const bool tr = conj && !TS;
    Ck<R> buf[L + RD];
#pragma unroll
    for (int i = 0; i < RD; ++i) buf[i] = carry[i];
    E bv[2][4][NC];
    B0(0, bv[0]);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int ip = i + RD;
      ck_load(buf[ip], ip < NCH ? A0 : (ip < L ? A1 : An), tr, ip % NCH);
      if (i + 1 < L) {
        if (i + 1 < NCH)
          B0(i + 1, bv[(i + 1) & 1]);
        else
          B1(i + 1 - NCH, bv[(i + 1) & 1]);
      }
      if (i == NCH) midf();
      mma(acc, buf[i], bv[i & 1], conj, i < NCH ? neg0 : true);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < RD; ++i) carry[i] = buf[L + i];
  };
  auto start = [&](const E* A, bool conj) {
#pragma unroll
    for (int i = 0; i < RD; ++i) ck_load(carry[i], A, conj && !TS, i);
  };
  auto none = [] {};

  Acc1 acc;
  E x[NC][4];
  c128 old[NC][4];
  E zero[NC][4];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) zero[c][r] = mk<R>(0, 0);
  // ---------------------------------------------------------- N forward
  // window = slots 0 (carry) and 1 (the block's new rows): v_k = Q z_top and
  // the next carry z_bot - M z_top, z = P y_win
  auto n_forward = [&](auto in) {
    using I = std::remove_cv_t<std::remove_pointer_t<decltype(in)>>;
    I fr[NC][4];
    gtile(fr, in, jb.ldin, 0);
    int pv = perm_get(0);
    start(blk(0, 0), false);
    conv(fr, rowok(0), x);
    put_own(0, x);
    gtile(fr, in, jb.ldin, 1);
    perm_put(pv);
    conv(fr, rowok(1), x);
    put_own(1, x);
    gtile(fr, in, jb.ldin, 2);
    pv = perm_get(K > 1 ? 1 : 0);
    __syncthreads();
    for (int k = 0; k < K; ++k) {
      uint2 off[NCH];  // gather offsets of the rows 16 ch + 4 q + kq
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        off[ch] = *reinterpret_cast<const uint2*>(spt + 16 * ch + 4 * kq);
      auto b_win = [&](int ch, E (&bv)[4][NC]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned h = q < 2 ? off[ch].x : off[ch].y;
          const unsigned o = ((q & 1) ? h >> 16 : h & 0xffffu) ^ (li * (unsigned)sizeof(E));
#pragma unroll
          for (int c = 0; c < NC; ++c)
            bv[q][c] = *reinterpret_cast<const E*>(lds_raw + o + c * NB * RB);
        }
      };
      const int zo = spo[NB + row];
      acc.zero();
      step(acc, blk(k, 0), blk(k, 1), blk(k + 1 < K ? k + 1 : k, 0), b_win, b_win, false, false,
           [&] {
             acc_get(acc, x);
             E z[NC][4];
#pragma unroll
             for (int c = 0; c < NC; ++c) lget(win(zo, c), win_sw(zo), z[c]);
             acc_set(acc, z);
             gput(x, mid, jb.ldmid, k);
           });
      __syncthreads();
      acc_get(acc, x);
      put_own(0, x);
      conv(fr, rowok(k + 2), x);
      put_own(1, x);
      perm_put(pv);
      gtile(fr, in, jb.ldin, k + 3 <= K ? k + 3 : K);
      pv = perm_get(k + 2 < K ? k + 2 : K - 1);
      __syncthreads();
    }
  };
  // ---------------------------------------------------------- H forward (U^H)
  // u_k = y_k - G1(k-1)^H u_{k-1} - G2(k-2)^H u_{k-2}; block 0 stands in for
  // the missing ones, which meet zero slots
  auto h_forward = [&](auto in) {
    int s1 = 0, s2 = 1, sv = 2;
    put_own(0, zero);
    put_own(1, zero);
    using I = std::remove_cv_t<std::remove_pointer_t<decltype(in)>>;
    I fr[NC][4];
    gtile(fr, in, jb.ldin, 0);
    start(blkh(0, 3), true);
    conv(fr, rowok(0), x);
    acc_set(acc, x);
    __syncthreads();
    for (int k = 0; k < K; ++k) {
      gtile(fr, in, jb.ldin, k + 1 < K ? k + 1 : k);
      step(acc, blkh(k >= 1 ? k - 1 : 0, 3), blkh(k >= 2 ? k - 2 : 0, 4), blkh(k, 3), b_slot(s1),
           b_slot(s2), true, true, none);
      acc_get(acc, x);
      put_own(sv, x);
      E y[NC][4];
      conv(fr, rowok(k + 1), y);
      acc_set(acc, y);
      gput(x, mid, jb.ldmid, k);
      __syncthreads();
      const int s = s2;
      s2 = s1;
      s1 = sv;
      sv = s;
    }
  };
  // the right-hand sides of a correction are in the factors' type
  auto with_rhs = [&](auto f) {
    if (jb.add)
      f((const E*)jb.in + (int64_t)jb.col0 * jb.ldin);
    else
      f((const c128*)jb.in + (int64_t)jb.col0 * jb.ldin);
  };
  if (jb.dir == 0) {
    with_rhs(n_forward);
    // ---------------------------------------------------------- N backward
    // x_k = v_k - G1 x_{k+1} - G2 x_{k+2}; the blocks beyond the last are
    // zero, as are the slots of x_K and x_{K+1}
    int s1 = 0, s2 = 1, sv = 2;
    put_own(0, zero);
    put_own(1, zero);
    E pm[NC][4];
    gtile(pm, mid, jb.ldmid, K - 1);
    start(blk(K - 1, 3), false);
    conv(pm, rowok(K - 1), x);
    acc_set(acc, x);
    __syncthreads();
    for (int k = K - 1; k >= 0; --k) {
      if (jb.add) gtile(old, out, jb.ldout, k);
      gtile(pm, mid, jb.ldmid, k > 0 ? k - 1 : 0);
      step(acc, blk(k, 3), blk(k, 4), blk(k > 0 ? k - 1 : k, 3), b_slot(s1), b_slot(s2), false,
           true, none);
      acc_get(acc, x);
      put_own(sv, x);
      E y[NC][4];
      conv(pm, true, y);  // rows below n for k > 0
      acc_set(acc, y);
      emit(x, old, k);
      __syncthreads();
      const int s = s2;
      s2 = s1;
      s1 = sv;
      sv = s;
    }
  } else {
    with_rhs(h_forward);
    // ---------------------------------------------------------- H backward (L^H)
    // top = Q^H u_k - M^H carry; x_win = P^T [top ; carry]: rows below NB are
    // the next carry (slot 0), the others leave (slot 1); u_k in slot 2
    put_own(0, zero);
    E pm[NC][4];
    gtile(pm, mid, jb.ldmid, K - 1);
    int pv = perm_get(K - 1);
    start(blkh(K - 1, 0), true);
    conv(pm, rowok(K - 1), x);
    put_own(2, x);
    perm_put(pv);
    __syncthreads();
    for (int k = K - 1; k >= 0; --k) {
      const bool leaves = k + 1 < K;
      if (jb.add && leaves) gtile(old, out, jb.ldout, k + 1);
      gtile(pm, mid, jb.ldmid, k > 0 ? k - 1 : 0);
      pv = perm_get(k > 0 ? k - 1 : 0);
      acc.zero();
      step(acc, blkh(k, 0), blkh(k, 1), blkh(k > 0 ? k - 1 : k, 0), b_slot(2), b_slot(0), true,
           false, none);
      E cr[NC][4];
      get_own(0, cr);
      const int to = spo[row], co = spo[NB + row];
      __syncthreads();
      acc_get(acc, x);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        lput(win(to, c), win_sw(to), x[c]);
        lput(win(co, c), win_sw(co), cr[c]);
      }
      conv(pm, true, x);
      put_own(2, x);
      perm_put(pv);
      __syncthreads();
      if (leaves) {
        get_own(1, x);
        emit(x, old, k + 1);
      }
    }
    if (jb.add) gtile(old, out, jb.ldout, 0);
    get_own(0, x);
    emit(x, old, 0);
  }
}

template <typename R, int NB, int NC>
int launch_nb(const cx<R>* mats, const cx<R>* matsT, const int16_t* perm, int64_t n, int njobs,
              const SolveJob* jobs_dev, hipStream_t st, const int32_t* gate) {
  const int K = (int)((n + NB - 1) / NB);
  const size_t smem = solve_lds_bytes(NB, 16 * NC, sizeof(cx<R>));
  (void)hipFuncSetAttribute((const void*)k_band_solve<R, NB, NC>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)hipGetLastError();
  for (int j0 = 0; j0 < njobs; j0 += 1 << 20) {
    int nj = njobs - j0 < (1 << 20) ? njobs - j0 : (1 << 20);
    int grid = 8 * ((nj + 7) / 8);
    k_band_solve<R, NB, NC><<<grid, NB * 4, smem, st>>>(mats, matsT, perm, n, K, jobs_dev + j0,
                                                        nj, gate);
    FB_HIP(hipGetLastError());
  }
  return 0;
}

template <typename R, int NC>
int launch_t(const cx<R>* mats, const cx<R>* matsT, const int16_t* perm, int64_t n, int nb,
             int njobs, const SolveJob* jobs_dev, hipStream_t st, const int32_t* gate) {
  switch (nb) {
    case 16: return launch_nb<R, 16, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
    case 32: return launch_nb<R, 32, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
    case 48: return launch_nb<R, 48, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
    case 64: return launch_nb<R, 64, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
    default: break;
  }
  if constexpr (NC == 1) {  // wider blocks take 16 columns (residual groups)
    switch (nb) {
      case 80: return launch_nb<R, 80, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
      case 96: return launch_nb<R, 96, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
      case 112: return launch_nb<R, 112, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
      case 128: return launch_nb<R, 128, NC>(mats, matsT, perm, n, njobs, jobs_dev, st, gate);
      default: break;
    }
  }
  return FB_ERR_INTERNAL;
}

// tile: columns per job
template <typename R>
int launch_tiles(int tile, const cx<R>* mats, const cx<R>* matsT, const int16_t* perm, int64_t n,
                 int nb, int njobs, const SolveJob* jobs_dev, hipStream_t st,
                 const int32_t* gate) {
  if (tile == 16)
    return launch_t<R, 1>(mats, matsT, perm, n, nb, njobs, jobs_dev, st, gate);
  if (tile == 32)
    return launch_t<R, 2>(mats, matsT, perm, n, nb, njobs, jobs_dev, st, gate);
  return FB_ERR_INTERNAL;
}

}  // namespace fb
