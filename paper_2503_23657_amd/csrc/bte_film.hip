// Source iterations of a 1D film (all cells active, first-order faces) in one
// launch: the transport sweeps (step 2 of the iteration), the band/direction
// sums with the new temperature or lambda (step 3), the lagged reflecting walls
// (Eqs. 6 and 7) and, on the last iteration, the residuals of Eq. 22 (step 4).
// One workgroup per instance keeps the whole state on one CU for every
// iteration of a chunk.
//
// A sweep of one ordinate is the recurrence f_i = S_i + a f_{i-1} along the
// film. In the rows-per-lane kernel a film has one row, so one lane of a wave
// walks the cells one by one (200 cells: 43 us a sweep and 6 us a finalize,
// whatever the number of ordinates). Here a lane takes CPL neighbouring cells,
// composes their affine maps, and a scan over the wave's lanes (DPP within
// rows of 16, then row broadcasts) gives each lane the value entering its
// cells: the chain is CPL + 6 + CPL steps long instead of the film's length.
// The arithmetic is double for both precisions (T is that of the constants and
// the stored state): a scan rounds in another order than the cell-by-cell walk,
// and dJ/dtau, whose terms nearly cancel, showed it in single precision (errors
// up to 1.1e-5 where the walk's was 1.5e-6; now as the walk's). A film is bound
// by latency, not by the rate of its arithmetic.
// Half of the waves sweep rightward, half leftward; a wave adds the sums of its
// ordinates in double registers, the waves' sums meet in LDS.
//
// What bounds it: the dependent chain of a wave's ordinates and, on small
// films, the launch and the host's look at the status once per chunk. The
// solve of 200 cells with 32 ordinates in FP64 (48 iterations in chunks of 8)
// went from 2545 to 325 us, solve and adjoint of 100 cells from 4020 to 820 us.
#include <hip/hip_runtime.h>

#include "bte_device.h"
#include "bte_launch.h"
#include "../../include/bte.h"

namespace bte {
namespace {

// the value of the lane CTRL names (rows of ROWS only), `old` elsewhere
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double old, double v) {
  const long long o = __double_as_longlong(old), x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)o, (int)x, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(x >> 32), CTRL, ROWS, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// the maps f -> A f + B of earlier lanes composed into this lane's
template <int CTRL, int ROWS>
__device__ __forceinline__ void compose(double& A, double& B) {
  const double a = dpp<CTRL, ROWS>(1.0, A), b = dpp<CTRL, ROWS>(0.0, B);
  B = fma(A, b, B);
  A *= a;
}

enum { FC_KS, FC_CQ, FC_A, FC_IN, FC_W0, FC_W1, FC_WO, FC_DEN };

// KEEP: the iterations change the state (else they are only timed: an instance
// that is done runs, too; a switch at run time cost films of 900 cells 3 %)
template <typename T, int CPL, int NW, bool KEEP>
__global__ void __launch_bounds__(NW * 64) film_chunk_kernel(FilmArgs A) {
  constexpr int N = 64 * CPL, NT = NW * 64, HW = NW / 2;
  constexpr int CT = (N + NT - 1) / NT;  // cells per thread of the sums
  extern __shared__ __align__(16) char lds[];
  double* sA = reinterpret_cast<double*>(lds);        // [NW][N] the waves' sums; the residual reduction
  double* sX = sA + NW * 64 * (CPL < 4 ? 4 : CPL);    // [N] Delta T or lambda
  double* sC = sX + N;                                // [n_grp][kFilmConst] group constants, sweep inflow
  double* sO = sC + (size_t)A.n_grp * kFilmConst;                // [n_grp] outflow at a reflecting wall
  const int inst = blockIdx.x;
  const InstDev& I = A.inst[inst];
  const FinInst& F = A.fin[inst];
  const FilmInst& W = A.walls[inst];
  StatusDev* st = reinterpret_cast<StatusDev*>(I.status);
  if (KEEP && st->done) return;
  const bool adj = (A.flags & FIN_ADJ) != 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = I.ncell, iter = st->iter, cur = iter & 1, nxt = (iter + A.n_iter) & 1;
  const int half = wave / HW;
  const int oct = adj ? 1 - half : half;  // the octant whose order this wave's ordinates sweep in
  const int nr = I.n_part / ((n + kC2 - 1) / kC2 * kC2);
  auto plane_index = [&](int c) { return I.cell_of ? c / kC2 * nr * kC2 + c % kC2 : c; };
  // ---- state and constants
  for (int c = tid; c < n; c += NT) sX[c] = F.X[cur][c];
  T* ubf = const_cast<T*>(reinterpret_cast<const T*>(I.ubf));
  for (int g = tid; g < A.n_grp; g += NT) {
    const int4 gi = A.grp_i[(size_t)inst * A.n_grp + g];
    const T* r = reinterpret_cast<const T*>(A.grp_t) + ((size_t)inst * A.n_grp + g) * grp_stride(1);
    double* c = sC + (size_t)g * kFilmConst;
    c[FC_KS] = r[0];
    c[FC_CQ] = r[1];
    c[FC_A] = r[go_a(1, 0)];
    c[FC_DEN] = r[go_den(1)];
    c[FC_IN] = (double)r[go_den(1)] * (double)ubf[(size_t)gi.w * I.n_bface + W.slot[gi.y & 1]];
    c[FC_W0] = r[go_wacc(1, 0)];
    c[FC_W1] = r[go_wacc(1, 1)];
    c[FC_WO] = r[go_wo(1, 0)];
  }
  double q[CPL];  // the source of the lane's cells, in sweep order (cell i or n - 1 - i)
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    const int i = lane * CPL + j, c = oct ? n - 1 - i : i;
    q[j] = i < n ? reinterpret_cast<const T*>(I.xq[cur])[2 * ((size_t)oct * I.pos_per_oct +
                                                              I.pos[(size_t)oct * I.n_part + plane_index(c)]) + 1]
                 : 0.0;
  }
  double qm[CT], res[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int p = 0; p < CT; ++p) {
    const int c = tid + p * NT;
    qm[p] = !adj && c < n ? F.qmag_prev[c] : 0.0;
  }
  __syncthreads();
  const int g0 = half ? A.g_split : 0, g1 = half ? A.n_grp : A.g_split;
  const bool reflect = W.kind[0] != BTE_BC_ISOTHERMAL || W.kind[1] != BTE_BC_ISOTHERMAL;
  const int jo = (n - 1) % CPL, lo = (n - 1) / CPL;  // the last cell of the sweep
  // sum of the waves' values of cell c: wave order, the rightward half first
  auto total = [&](int c) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int o = adj ? 1 - w / HW : w / HW;
      const int i = o ? n - 1 - c : c;
      s += sA[(size_t)w * N + (i % CPL) * 64 + i / CPL];
    }
    return s;
  };

  for (int it = 0; it < A.n_iter; ++it) {
    const bool last = it == A.n_iter - 1;
    const bool withq = !adj && it >= A.n_iter - 2;
    double x[CPL];
    double acc[CPL], acq[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int i = lane * CPL + j, c = oct ? n - 1 - i : i;
      x[j] = i < n ? sX[c] : 0.0;
      acc[j] = acq[j] = 0.0;
    }
    for (int g = g0 + wave % HW; g < g1; g += HW) {
      const double* c = sC + (size_t)g * kFilmConst;
      const double kS = c[FC_KS], cQ = c[FC_CQ], a = c[FC_A], fin = c[FC_IN];
      const double w0 = c[FC_W0], w1 = c[FC_W1];
      double Am = 1.0, Bm = 0.0;
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        Bm = fma(a, Bm, fma(kS, x[j], cQ * q[j]));
        Am *= a;
      }
      compose<0x111, 0xF>(Am, Bm);  // row_shr:1, 2, 4, 8
      compose<0x112, 0xF>(Am, Bm);
      compose<0x114, 0xF>(Am, Bm);
      compose<0x118, 0xF>(Am, Bm);
      compose<0x142, 0xA>(Am, Bm);  // row_bcast:15 into rows 1 and 3
      compose<0x143, 0xC>(Am, Bm);  // row_bcast:31 into rows 2 and 3
      double f = fma(dpp<0x138, 0xF>(1.0, Am), fin, dpp<0x138, 0xF>(0.0, Bm));  // wave_shr:1
      double fo = 0.0;
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        f = fma(a, f, fma(kS, x[j], cQ * q[j]));
        acc[j] = fma(w0, f, acc[j]);
        if (withq) acq[j] = fma(w1, f, acq[j]);
        fo = j == jo ? f : fo;
      }
      if (reflect && lane == lo) sO[g] = c[FC_WO] * fo;
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) sA[(size_t)wave * N + j * 64 + lane] = acc[j];
    __syncthreads();
    if (last) res[0] = res[1] = res[2] = res[3] = 0.0;
#pragma unroll
    for (int p = 0; p < CT; ++p) {
      const int c = tid + p * NT;
      if (c >= n) continue;
      const double v = (adj ? F.g[c] : 0.0) + total(c), d = v - sX[c];
      sX[c] = v;
      if (last) {
        res[0] += d * d;
        res[1] = fmax(res[1], fabs(v));
        if (!isfinite(v)) res[3] = INFINITY;
      }
    }
    // lagged reflecting walls: the new inflow of the ordinates that enter there
    if (reflect) {
      for (int g = tid; g < A.n_grp; g += NT) {
        const int4 gi = A.grp_i[(size_t)inst * A.n_grp + g];
        // (the end an ordinate of this octant enters through)
        const int face = gi.y & 1, kind = W.kind[face];
        if (kind == BTE_BC_ISOTHERMAL) continue;
        double u;
        if (kind == BTE_BC_SPECULAR) {
          const int a = gi.w - gi.x * A.rows;
          const int2 src = A.src[face * A.rows + a];
          if (src.x < 0) continue;
          u = sO[A.grp_ob[src.x * A.B + gi.x].x + src.y] * A.inv_wq[face * A.rows + a];
        } else {
          const int2 gr = A.grp_ob[(1 - face) * A.B + gi.x];
          double s = 0.0;
          for (int k = 0; k < gr.y; ++k) s += sO[gr.x + k];
          u = s * W.inv_half[face];
        }
        sC[(size_t)g * kFilmConst + FC_IN] = sC[(size_t)g * kFilmConst + FC_DEN] * u;
        if (KEEP && last) ubf[(size_t)gi.w * I.n_bface + W.slot[face]] = (T)u;
      }
    }
    __syncthreads();
    if (withq) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) sA[(size_t)wave * N + j * 64 + lane] = acq[j];
      __syncthreads();
#pragma unroll
      for (int p = 0; p < CT; ++p) {
        const int c = tid + p * NT;
        if (c >= n) continue;
        const double v = total(c), m = sqrt(v * v), d = m - qm[p];
        qm[p] = m;
        if (KEEP && last) {
          F.q[c] = v;
          F.qmag_prev[c] = m;
          res[2] += d * d;
          res[3] = isfinite(v) ? fmax(res[3], m) : INFINITY;
        }
      }
      __syncthreads();
    }
  }
  if (!KEEP) return;
  // ---- the new state, in grid order and in both octants' layouts
  T* xq = reinterpret_cast<T*>(I.xq[nxt]);
  for (int c = tid; c < n; c += NT) {
    const double v = sX[c];
    F.X[nxt][c] = v;
    const int pc = plane_index(c);
    for (int o = 0; o < 2; ++o)
      xq[2 * ((size_t)o * I.pos_per_oct + I.pos[(size_t)o * I.n_part + pc])] = (T)v;
  }
  // ---- residuals (Eq. 22) over the film
#pragma unroll
  for (int i = 0; i < 4; ++i) sA[i * NT + tid] = res[i];
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (tid < s) {
      sA[tid] += sA[tid + s];
      sA[NT + tid] = fmax(sA[NT + tid], sA[NT + tid + s]);
      sA[2 * NT + tid] += sA[2 * NT + tid + s];
      sA[3 * NT + tid] = fmax(sA[3 * NT + tid], sA[3 * NT + tid + s]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    const double a0 = sA[0], a1 = sA[NT], a2 = sA[2 * NT], a3 = sA[3 * NT];
    const double nact = st->red[0], rT = sqrt(a0 / nact), rq = sqrt(a2 / nact);
    const double eT = a1 > 0.0 ? rT / a1 : (rT == 0.0 ? 0.0 : INFINITY);
    const double eq = adj ? 0.0 : (a3 > 0.0 ? rq / a3 : (rq == 0.0 ? 0.0 : INFINITY));
    st->iter = iter + A.n_iter;
    st->eps_T = eT;
    st->eps_q = eq;
    st->checked = iter + A.n_iter;
    if (A.tol_T > 0.0 && A.tol_q > 0.0 && eT < A.tol_T && eq < A.tol_q) st->done = 1;
    if (!isfinite(a1) || !isfinite(a3) || !isfinite(a0)) {
      st->nonfinite = 1;
      st->done = 1;
    }
  }
}

template <typename T, int CPL, int NW, bool KEEP>
hipError_t film_launch(const FilmArgs& a, int n_inst, hipStream_t st) {
  auto k = film_chunk_kernel<T, CPL, NW, KEEP>;
  static_assert(NW == film_waves(CPL), "the LDS a launch asks for");
  const size_t lds = film_lds_bytes(CPL, a.n_grp);
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kFilmLds);
  if (attr != hipSuccess || lds > (size_t)kFilmLds) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(n_inst), dim3(NW * 64), lds, st, a);
  return hipGetLastError();
}

template <typename T, int CPL, int NW>
hipError_t film_one(const FilmArgs& a, int n_inst, hipStream_t st) {
  return (a.flags & FILM_TIMING) ? film_launch<T, CPL, NW, false>(a, n_inst, st)
                                 : film_launch<T, CPL, NW, true>(a, n_inst, st);
}

template <typename T>
hipError_t film_any(const FilmArgs& a, int n_inst, int cpl, hipStream_t st) {
  switch (cpl) {
    case 1: return film_one<T, 1, 16>(a, n_inst, st);
    case 2: return film_one<T, 2, 16>(a, n_inst, st);
    case 4: return film_one<T, 4, 16>(a, n_inst, st);
    case 8: return film_one<T, 8, 16>(a, n_inst, st);
    case 16: return film_one<T, 16, 8>(a, n_inst, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_film_chunk(int prec, const FilmArgs& a, int n_inst, int cpl, hipStream_t st) {
  return prec == BTE_PREC_FP32 ? film_any<float>(a, n_inst, cpl, st) : film_any<double>(a, n_inst, cpl, st);
}

}  // namespace bte
