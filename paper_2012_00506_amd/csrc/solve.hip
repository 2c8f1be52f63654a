// Multi-right-hand-side solves with the block form of the band LU factors.
// Every sweep step is one set of independent products of blocks formed once
// per factorisation (M = Lh21 Lh11^{-1}, Q = U(k,k)^{-1} Lh11^{-1},
// G1 = U(k,k)^{-1} U(k,k+1), G2 = U(k,k)^{-1} U(k,k+2)), so that a step
// waits for the previous one only once.
//
// N: x = A^{-1} y.  Forward, block k on the window rows kb .. kb+2b-1:
//      z = P y_win; v_k = Q z_top; carry = z_bot - M z_top
//    (v_k = U(k,k)^{-1} Lh11^{-1} z_top).
//    Backward: x_k = v_k - G1 x_{k+1} - G2 x_{k+2}
//    (= U(k,k)^{-1} (Lh11^{-1} z_top - U(k,k+1) x_{k+1} - U(k,k+2) x_{k+2})).
// H: x = A^{-H} y.  Forward with U^H, in u_k = U(k,k)^H w_k:
//      u_k = y_k - G1(k-1)^H u_{k-1} - G2(k-2)^H u_{k-2}
//    (w_k = U(k,k)^{-H} (y_k - U(k-1,k)^H w_{k-1} - U(k-2,k)^H w_{k-2})).
//    Backward, k descending on the window [u_k ; carry]:
//      top = Q^H u_k - M^H carry; x_win = P^T [top ; carry]
//    (top = Lh11^{-H} w_k - M^H carry; rows kb+b .. kb+2b-1 of x_win are
//    final, rows kb .. kb+b-1 carry on).
// One workgroup per job (system, direction, tile of T columns); the tile's
// window and carries live in LDS.  Inputs and outputs are complex128; the
// arithmetic is in R (float: complex64 path, double: complex128 path).
#include "solve_kernel.h"
#include "tune.h"

namespace fb {
// the kernels live in solve_f32.hip / solve_f64.hip
extern template int launch_tiles<float>(int, const c64*, const c64*, const int16_t*, int64_t, int,
                                        int, const SolveJob*, hipStream_t, const int32_t*);
extern template int launch_tiles<double>(int, const c128*, const c128*, const int16_t*, int64_t,
                                         int, int, const SolveJob*, hipStream_t, const int32_t*);
}  // namespace fb

namespace fb {

// ---------------------------------------------------------------- dispatch
// Tile width of one call's solves: the autotuner's choice where there is one,
// else 32 columns in complex64 and 16 in complex128 (a 32-column tile's
// registers spill there: n = 16384, b = 64, 24 systems x 1056 columns 30.4
// against 27.7 ms).  Each factor fragment serves twice the columns in a wide
// tile, but a call with fewer wide tiles than CUs is bound by the length of a
// tile's sweeps, which are shorter in a narrow one: complex64, n = 16384,
// b = 64, 16 system-directions of 200, 400 and 800 columns took 1.9, 2.7 and
// 5.0 ms in 16-column tiles against 2.6, 2.8 and 4.3 ms.
template <typename R>
int solve_tile(int b, size_t tiles32) {
  const int nb = block_size(b);
  const int v = tuned_variant(sizeof(R), nb);
  if (v >= 0) return variant_tile(v);
  return sizeof(R) == 4 && tiles32 >= (size_t)rule_cus() && variant_fits(sizeof(R), nb, 2) ? 32 : 16;
}

template <typename R>
int launch_solve_jobs(const cx<R>* mats, const cx<R>* matsT, const int16_t* perm, int64_t n,
                      int b, int tile, int njobs, const SolveJob* jobs_dev, double work,
                      hipStream_t st, const int32_t* gate) {
  if (njobs <= 0) return 0;
  if (sizeof(R) == 4 && matsT == nullptr) return FB_ERR_INTERNAL;
  ProfScope ps(FB_PROF_SOLVE, st, work);
  return launch_tiles<R>(tile, mats, matsT, perm, n, block_size(b), njobs, jobs_dev, st, gate);
}

template int launch_solve_jobs<float>(const c64*, const c64*, const int16_t*, int64_t, int, int,
                                      int, const SolveJob*, double, hipStream_t, const int32_t*);
template int launch_solve_jobs<double>(const c128*, const c128*, const int16_t*, int64_t, int,
                                       int, int, const SolveJob*, double, hipStream_t,
                                       const int32_t*);
template int solve_tile<float>(int, size_t);
template int solve_tile<double>(int, size_t);

// ---------------------------------------------------------------- residual
// r = y - (zz x - B x) in FP64 for the columns of a job (zz = z for A x = y,
// conj(z) for A^H x = y), with B in block-tridiagonal form:
// (B x)_k = B(k,k-1) x_{k-1} + B(k,k) x_k + B(k,k+1) x_{k+1}, each an NB x NB
// by NB x 16 product on f64 MFMA (three real products per complex one),
// wave w computing rows 16 w .. 16 w + 15.  As in the solves, tiles are
// computed transposed: y and r move between global memory and the
// accumulators' layout in runs of 256 bytes; x blocks roll through a ring of
// LDS slots.
//
// A wave's share of the three products is a fixed list of 2 NB/16 + 1
// chunks of 16 B columns (the triangles of B(k,k-1) and B(k,k+1) outside
// the band are skipped).  Its B fragments are loaded chunk by chunk RD chunks
// ahead of the MFMAs that use them, across block rows and barriers, so that
// no product waits for its first fragment.  The blocks B(0,-1) and
// B(K-1,K) are zero, as are the x slots beyond the ends, so every block row
// runs the same list.  Per (job, column): sum |r|^2 and sum |y|^2.  r (null:
// not kept) is stored in the type RT that the correction solves compute in.
//
// What bounds it: the FP64 MFMAs (6 (2 b + 16) n flop per column at 72
// TFLOP/s), then B's fragments from L2, a kilobyte per three MFMAs and wave.
// n = 16384, 64 system-directions: b = 64, 1400 columns 28.6 -> 21.1 ms (MFMA
// alone 15.7), b = 128, 576 columns 18.5 -> 16.6 (13.5), against 32-column
// workgroups that staged y and r through LDS, one to a CU.
// Slots of the x ring: three where workgroups share a CU (with registers for
// three waves per SIMD: one chunk of B ahead); four, which save a barrier per
// block row, for blocks of 112 and 128 rows, which have a CU to themselves (b =
// 128: 16.6 ms against 17.4 with three).
constexpr int residual_slots(int nb) { return nb <= 96 ? 3 : 4; }

template <int NB, typename RT>
__global__ void __launch_bounds__(NB * 4, NB <= 96 ? 3 : 2)
k_shift_residual(const c128* __restrict__ Bblk, int64_t n, int K, const ResJob* __restrict__ jobs,
                 int njobs, double* __restrict__ part, const int32_t* __restrict__ gate) {
  constexpr int NRW = NB / 16;
  constexpr int L = 2 * NRW + 1;  // chunks per block row and wave
  constexpr int NS = residual_slots(NB);
  constexpr int RD = NS == 3 ? 1 : 2;
  constexpr int SUB = residual_cols(NB) / 16;  // workgroups per job
  extern __shared__ __align__(16) char lds_raw[];
  c128* X = reinterpret_cast<c128*>(lds_raw);  // NS slots of NB rows of 16 columns
  const int wg = remap_job(blockIdx.x, njobs * SUB);
  if (wg >= njobs * SUB) return;
  const int job = wg / SUB, cs = 16 * (wg % SUB);
  const ResJob jb = jobs[job];
  const int ncol = jb.ncol - cs;
  if (ncol <= 0) return;
  if (gate && !gate[jb.grp]) return;  // the group has finished refining
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const int row = 16 * w + li;  // the lane's block row
  const size_t bb = (size_t)NB * NB;
  const c128 zz = jb.dir ? mk(jb.z.x, -jb.z.y) : jb.z;
  const c128* jx = jb.x + (int64_t)(jb.col0 + cs) * jb.ldx;
  const c128* jy = jb.y + (int64_t)(jb.col0 + cs) * jb.ldy;
  RT* jr = (RT*)jb.r + (int64_t)cs * jb.ldr;
  // Chunk i of the list: B columns 16 (w + i) .. of [B(k,k-1) B(k,k) B(k,k+1)],
  // which lie one after the other, and the same rows of [x_{k-1}; x_k;
  // x_{k+1}], the slots taken as one ring of NS NB rows.  Fragment q:
  // B[16 w + lane % 16][16 (w + i) + 4 q + lane / 16].
  struct Ch {
    c128 a[4];
  };
  auto cload = [&](Ch& f, int k, int i) {
    const c128* A = Bblk + (size_t)k * 3 * bb + (size_t)(16 * (w + i)) * NB;
#pragma unroll
    for (int q = 0; q < 4; ++q) f.a[q] = gld(A + 4 * q * NB + (kq * NB + row));
  };
  // tiles in accumulator order: element r is column kq + 4 r of the lane's
  // row.  Columns beyond ncol read the first one (never stored).
  auto gtile = [&](c128 (&v)[4], const c128* base, int64_t ld, int k) {
    const int64_t i = (int64_t)k * NB + row;
    const c128* p0 = base + (i < n ? i : n - 1);
    const c128* pl = p0 + kq * ld;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = gld(kq + 4 * r < ncol ? pl + 4 * r * ld : p0);
  };
  auto rowok = [&](int k) { return (int64_t)k * NB + row < n; };
  auto at = [&](int slot, int r) {
    return X + (slot * NB + row) * 16 + kq + 4 * (r ^ (li & 3));
  };
  auto put = [&](int slot, const c128 (&v)[4], bool ok) {
#pragma unroll
    for (int r = 0; r < 4; ++r) *at(slot, r) = mk(ok ? v[r].x : 0.0, ok ? v[r].y : 0.0);
  };
  double rr[4], yy[4];
  c128 xr[4], yv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rr[r] = yy[r] = 0.0;
  gtile(xr, jx, jb.ldx, 0);
  Ch carry[RD];
#pragma unroll
  for (int i = 0; i < RD; ++i) cload(carry[i], 0, i);
  put(NS - 1, xr, false);  // x_{-1}
  put(0, xr, rowok(0));
  gtile(xr, jx, jb.ldx, 1);
  gtile(yv, jy, jb.ldy, 0);
  int sm = NS - 1, s0 = 0, sp = 1;  // slots of x_{k-1}, x_k, x_{k+1}
  for (int k = 0; k < K; ++k) {
    put(sp, xr, rowok(k + 1));
    __syncthreads();
    gtile(xr, jx, jb.ldx, k + 2);
    const int kn = k + 1 < K ? k + 1 : k;
    auto bload = [&](c128 (&bv)[4], int i) {
      int g = sm * NRW + w + i;
      g -= g >= NS * NRW ? NS * NRW : 0;
      const c128* b = X + g * 256 + (kq * 16 + (li ^ (kq << 2)));
#pragma unroll
      for (int q = 0; q < 4; ++q) bv[q] = b[4 * q * 16];
    };
    Acc<double, 1> acc;
    acc.zero();
    Ch buf[L + RD];
    c128 bv[2][4];
#pragma unroll
    for (int i = 0; i < RD; ++i) buf[i] = carry[i];
    bload(bv[0], 0);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      if (i + RD < L)
        cload(buf[i + RD], k, i + RD);
      else
        cload(buf[i + RD], kn, i + RD - L);
      if (i + 1 < L) bload(bv[(i + 1) & 1], i + 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double ar = buf[i].a[q].x, ai = buf[i].a[q].y;
        const c128 b = bv[i & 1][q];
        acc.p1[0] = MF<double>::mma(b.x, ar, acc.p1[0]);
        acc.p2[0] = MF<double>::mma(b.y, ai, acc.p2[0]);
        acc.p3[0] = MF<double>::mma(b.x + b.y, ar + ai, acc.p3[0]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < RD; ++i) carry[i] = buf[L + i];
    const bool ok = rowok(k);
    c128 rv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const c128* xp = at(s0, r);
      const c128 xo = mk(xp->x, xp->y);
      const c128 y = mk(ok ? yv[r].x : 0.0, ok ? yv[r].y : 0.0);
      const c128 v = y - zz * xo + acc.get(0, r);
      yy[r] += cabs2(y);
      rr[r] += cabs2(v);
      rv[r] = v;
    }
    if (NS == 3) __syncthreads();  // before x_{k+2} takes the slot of x_{k-1}
    gtile(yv, jy, jb.ldy, k + 1);
    if (jb.r) {
      RT* pl = jr + ((int64_t)k * NB + row) + kq * jb.ldr;
      auto st = [&](int r) { gst(pl + 4 * r * jb.ldr, ccast<decltype(RT::x)>(rv[r])); };
      if (ncol >= 16 && (int64_t)(k + 1) * NB <= n) {
#pragma unroll
        for (int r = 0; r < 4; ++r) st(r);
      } else if (ok) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kq + 4 * r < ncol) st(r);
      }
    }
    sm = s0;
    s0 = sp;
    sp = sp + 1 < NS ? sp + 1 : 0;
  }
  // column sums in a fixed order: per-row partial sums through LDS, then one
  // thread per column adds its NB rows
  __syncthreads();
  double* red = reinterpret_cast<double*>(X);  // 2 x 16 columns x NB rows
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[(kq + 4 * r) * NB + row] = rr[r];
    red[(16 + kq + 4 * r) * NB + row] = yy[r];
  }
  __syncthreads();
  if (t < 16) {
    double sr = 0.0, sy = 0.0;
    for (int i = 0; i < NB; ++i) {
      sr += red[t * NB + i];
      sy += red[(16 + t) * NB + i];
    }
    part[((size_t)job * 32 + cs + t) * 2] = sr;
    part[((size_t)job * 32 + cs + t) * 2 + 1] = sy;
  }
}

// per group: ratio = max over its columns of sqrt(sum|r|^2 / sum|y|^2)
// (columns with y = 0 count as converged when r = 0), and the decision of
// the next refinement pass (RefineCtl)
__global__ void k_refine_decide(const double* __restrict__ part, int njobs,
                                const ResJob* __restrict__ jobs, RefineCtl ctl) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= njobs) return;
  const int g = jobs[j].grp;
  if (ctl.gate && !ctl.gate[g]) return;
  double mx = 0.0;
  for (int c = 0; c < jobs[j].ncol; ++c) {
    double rr = part[((size_t)j * 32 + c) * 2], yy = part[((size_t)j * 32 + c) * 2 + 1];
    double q = yy > 0.0 ? sqrt(rr / yy) : (rr > 0.0 ? 1e300 : 0.0);
    if (!(q <= mx)) mx = q;  // NaN propagates
  }
  const double prev = ctl.ratio[g];
  ctl.ratio[g] = mx;
  if (ctl.pass == 0) ctl.npass[g] = 0;
  const bool more = ctl.ir && !(mx <= ctl.ir_tol) && ctl.pass < ctl.max_pass &&
                    (ctl.pass == 0 || mx < 0.5 * prev);
  ctl.flag[g] = more ? 1 : 0;
  if (more) ctl.npass[g] = ctl.pass + 1;
}

size_t residual_part_doubles(int64_t n, int njobs) {
  (void)n;
  return (size_t)njobs * 32 * 2;
}

template <int NB, typename RT>
static int launch_res_nb(const Band& bd, int njobs, const ResJob* jobs_dev, double* part,
                         const int32_t* gate, hipStream_t st) {
  constexpr int sub = residual_cols(NB) / 16;
  const size_t smem = (size_t)residual_slots(NB) * NB * 16 * sizeof(c128);
  (void)hipFuncSetAttribute((const void*)k_shift_residual<NB, RT>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)hipGetLastError();
  for (int j0 = 0; j0 < njobs; j0 += 1 << 20) {
    int nj = njobs - j0 < (1 << 20) ? njobs - j0 : (1 << 20);
    int grid = 8 * ((nj * sub + 7) / 8);
    k_shift_residual<NB, RT><<<grid, NB * 4, smem, st>>>(bd.Bblk, bd.n, bd.K, jobs_dev + j0, nj,
                                                         part + (size_t)j0 * 64, gate);
    FB_HIP(hipGetLastError());
  }
  return 0;
}

template <typename RT>
int launch_residual_jobs(const Band& bd, int njobs, const ResJob* jobs_dev, double* part,
                         const RefineCtl& ctl, double work, hipStream_t st) {
  if (njobs <= 0) return 0;
  ProfScope ps(FB_PROF_RESID, st, work);
  int rc;
  const int32_t* gate = ctl.gate;
  switch (bd.nb) {
    case 16: rc = launch_res_nb<16, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 32: rc = launch_res_nb<32, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 48: rc = launch_res_nb<48, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 64: rc = launch_res_nb<64, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 80: rc = launch_res_nb<80, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 96: rc = launch_res_nb<96, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 112: rc = launch_res_nb<112, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    case 128: rc = launch_res_nb<128, RT>(bd, njobs, jobs_dev, part, gate, st); break;
    default: return FB_ERR_INTERNAL;
  }
  if (rc) return rc;
  k_refine_decide<<<(njobs + 255) / 256, 256, 0, st>>>(part, njobs, jobs_dev, ctl);
  FB_HIP(hipGetLastError());
  return 0;
}

template int launch_residual_jobs<c64>(const Band&, int, const ResJob*, double*, const RefineCtl&,
                                       double, hipStream_t);
template int launch_residual_jobs<c128>(const Band&, int, const ResJob*, double*,
                                        const RefineCtl&, double, hipStream_t);

}  // namespace fb
