// Deferred correction of the second-order faces (Methods, "Spatial
// discretization"; Eq. rhs_b) for the one-strip rows-per-lane layouts: one
// pass over the stored angular field in the order it is stored.
//
// In the skewed layout (position ((t*64 + l)*NR + k): clock step t, lane l, row
// k of the lane) every interior neighbour of a position sits at a fixed
// distance: one step back or ahead along the step axis, the next row of the
// lane or the neighbouring lane one step back or ahead along the lane axis,
// and (3D) one chunk of kC2 steps back or ahead along the plane axis. A wave
// takes one group (one ordinate) and marches along t with the chunks it needs
// in registers: every field value is loaded once, in whole lines, the lane
// neighbours come by DPP. What a chunk of a block of kC2 columns (3D) needs
// from the blocks beside it, the previous block's last two columns and the
// next block's first in the same plane, is gathered a chunk ahead; the waves of
// a workgroup take neighbouring blocks of one group, so those lines are in the
// L2 they share. Boundary faces come from a code per position.
//
// What bounds it: 8 bytes of HBM traffic per position and group in FP32 (one
// read, one write; the 256^2 square 645 MB in 145 us, 4.4 TB/s), in 3D also
// about 70 VALU per value. The gather kernel (ten loads per value through a
// stencil table; kept for several strips and for walls of one side at several
// temperatures) takes 385 us there, and 1.70 ms against 0.81 ms on the
// 48x48x60 FinFET-like domain with 1920 ordinates.
#include <hip/hip_runtime.h>

#include "bte_device.h"
#include "bte_kutil.h"
#include "bte_launch.h"
#include "../../include/bte.h"

namespace bte {
namespace {

template <typename T, int N>
struct VecN {
  typedef T type __attribute__((ext_vector_type(N)));
};

// DPP wave_shr:1 / wave_shl:1: lane i takes lane i - 1 / i + 1 (the end lane
// keeps its own value, which its boundary code never selects)
template <int CTRL>
__device__ __forceinline__ float dpp1(float v) {
  const int x = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp1(double v) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(x >> 32), (int)(x >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <typename T>
__device__ __forceinline__ T below(T v) { return dpp1<0x138>(v); }
template <typename T>
__device__ __forceinline__ T above(T v) { return dpp1<0x130>(v); }

// Twice the Green-Gauss gradient difference along one axis, between the cell
// and its upwind neighbour, times h: (un - uu) - (uc - uuu) with un, uu, uuu
// the values downwind, upwind and twice upwind. A boundary replaces them by
// ghost values that give the same face values: extrapolated faces 1.5 a - 0.5 b
// are the mean with 2 a - b, an isothermal face W the mean with 2 W - a.
template <typename T>
__device__ __forceinline__ T grad_diff(unsigned st, T uc, T un, T uu, T uuu, T W) {
  const bool nodn = (st & CC_NODN) != 0, iso = (st & CC_ISO) != 0;
  const bool noup = (st & CC_UP) == CC_NOUP, nouu = (st & CC_UP) == CC_NOUU;
  const T gn = noup ? uc : T(2) * uc - uu;                                   // no downwind cell
  const T gu = iso ? T(2) * W - uc : (nodn ? uc : T(2) * uc - un);           // no upwind cell
  const T guu = iso ? T(2) * W - uu : T(2) * uu - uc;                        // no cell twice upwind
  const T a = nodn ? gn : un;
  const T b = noup ? gu : uu;
  const T c = noup ? uc : (nouu ? guu : uuu);
  return (a - b) - (uc - c);
}

template <typename T, int NR, bool D3>
__global__ void __launch_bounds__(256) corr_march_kernel(CorrArgs A) {
  using VR = typename VecN<T, NR>::type;
  constexpr int ND = D3 ? 3 : 2;
  constexpr int ES = (int)sizeof(T);
  constexpr int STEP = 64 * NR * ES;  // bytes of one step
  const InstDev& I = A.inst[A.inst_id];
  if (reinterpret_cast<const StatusDev*>(I.status)->done) return;
  // workgroups go to the 8 XCDs in turn: a contiguous range of units each, so
  // that the blocks of a group share an L2
  const int total = gridDim.x, per = total / 8;
  const int lin = (int)blockIdx.x < per * 8 ? ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8 : (int)blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(lin * 4 + (int)(threadIdx.x >> 6));
  if (wave >= A.n_grp * A.n_unit) return;
  const int lane = threadIdx.x & 63;
  const int g = wave / A.n_unit, unit = wave - g * A.n_unit;
  const int4 gi = A.grp[g];
  const int o = gi.y;
  const long long ppo = I.pos_per_oct;
  const int n_step = (int)(ppo / (64 * NR * A.n_slot));  // steps of slot 0, the prefetch padding included
  const int last = n_step / kC2 - 1;                     // (loads of a later chunk are clamped to it, and unused)
  int cb, ce, qlo = 0, qhi = 0;
  if constexpr (D3) {
    const int2 ur = A.unit[o * A.n_unit + unit];  // the periods of the unit's block
    qlo = ur.x;
    qhi = ur.y;
    if (qlo >= qhi) return;
    cb = qlo;
    ce = min(qhi + A.tail, last);
  } else {
    cb = unit * A.seg;
    ce = min(cb + A.seg, last);
    if (cb >= ce) return;
  }
  const unsigned bytes = (unsigned)((long long)n_step * STEP);
  const rsrc_t UR = mkrsrc(reinterpret_cast<const T*>(I.store_u) + (size_t)g * ppo, bytes);
  const rsrc_t CR = mkrsrc(reinterpret_cast<T*>(I.corr) + (size_t)g * ppo, bytes);
  const rsrc_t CD = mkrsrc(A.code + (size_t)o * n_step * 64, (unsigned)n_step * 256u);
  const int ax[3] = {D3 ? I.ax[0] : 0, D3 ? I.ax[1] : 1, D3 ? I.ax[2] : 2};
  T cf[ND], W[ND];  // factor and isothermal upwind wall value along each kernel axis
#pragma unroll
  for (int e = 0; e < ND; ++e) {
    const int d = ax[e];
    const int ws = A.wslot[o * ND + e];
    W[e] = ws >= 0 ? reinterpret_cast<const T*>(I.ubf)[ws] : T(0);

    const T c = d < I.dim ? (T)A.coef[(size_t)g * 3 + d] * (T(1) / (T)A.h[d]) : T(0);
    cf[e] = T(0.5) * (((o >> d) & 1) ? -c : c);
  }
  const int lo = lane * NR * ES;
  auto chunk_load = [&](VR* w, int c) {
    const int cc = min(c, last);
#pragma unroll
    for (int u = 0; u < kC2; ++u) w[u] = ldv<VR>(UR, lo, (cc * kC2 + u) * STEP);
  };
  auto code_load = [&](unsigned* cd, int c) {
    const int cc = min(c, last);
#pragma unroll
    for (int u = 0; u < kC2; ++u) cd[u] = (unsigned)bld<int>(CD, ((cc * kC2 + u) * 64 + lane) * 4);
  };
  // (a chunk before the first reads chunk 0, whose values no cell selects)
  VR w2[D3 ? kC2 : 1], w1[kC2], w0[kC2], wn[kC2];
  unsigned cd[kC2];
  if constexpr (D3) {
    chunk_load(w2, max(cb - 2, 0));
    chunk_load(w1, max(cb - 1, 0));
  } else {
#pragma unroll
    for (int u = kC2 - 2; u < kC2; ++u) w1[u] = ldv<VR>(UR, lo, (max(cb - 1, 0) * kC2 + u) * STEP);
  }
  chunk_load(w0, cb);
  chunk_load(wn, cb + 1);
  code_load(cd, cb);

  // 3D: the columns beside the block. The lane's period that starts in chunk c
  // is c - lane/8, the one whose last column lies in chunk c is
  // c - (lane + 7)/8; link: the periods of the previous and the next block in
  // the same plane, + 1 (0: none; also what an index outside the table reads)
  const int m = lane & (kC2 - 1);
  const int n_per = D3 ? I.n_per : 0;
  const rsrc_t LK = mkrsrc(D3 ? A.link + (size_t)o * n_per : nullptr, (unsigned)n_per * 8u);
  auto linked = [&](int q, bool next) { return bld<int>(LK, q * 8 + (next ? 4 : 0)); };
  auto column = [&](int q1, int j) {  // column j of the lane in period q1 - 1
    return ldv<VR>(UR, q1 > 0 ? (((q1 - 1) * kC2 + j + lane) * 64 + lane) * NR * ES : kOOB, 0);
  };
  VR e7p = VR(T(0)), e7 = VR(T(0)), e6 = VR(T(0)), x0 = VR(T(0));  // previous block's columns, next block's first
  int lp = 0, ln = 0;
  if constexpr (D3) {
    lp = linked(cb - (lane >> 3), false);
    ln = linked(cb - ((lane + 7) >> 3), true);
    e7p = column(linked(cb - 1 - (lane >> 3), false), kC2 - 1);
    e7 = column(lp, kC2 - 1);
    e6 = column(lp, kC2 - 2);
    x0 = column(ln, 0);
    lp = linked(cb + 1 - (lane >> 3), false);
    ln = linked(cb + 1 - ((lane + 7) >> 3), true);
  }

  for (int c = cb; c < ce; ++c) {
    VR nx[kC2], n7, n6, n0;
    unsigned cdn[kC2];
    chunk_load(nx, c + 2);
    code_load(cdn, c + 1);
    if constexpr (D3) {
      n7 = column(lp, kC2 - 1);
      n6 = column(lp, kC2 - 2);
      n0 = column(ln, 0);
      lp = linked(c + 2 - (lane >> 3), false);
      ln = linked(c + 2 - ((lane + 7) >> 3), true);
    }
    // store offsets of the lane's two periods in this chunk (3D: own ones only)
    const int ql = c - (lane >> 3);
    const int so1 = !D3 || (ql >= qlo && ql < qhi) ? lo : kOOB;
    const int so0 = !D3 || (ql - 1 >= qlo && ql - 1 < qhi) ? lo : kOOB;
#pragma unroll
    for (int u = 0; u < kC2; ++u) {
      const bool idle = cd[u] == CC_IDLE;  // no cell in any of the lane's rows: nothing to store
      const unsigned cw = idle ? 0u : cd[u];
      const VR uc = w0[u];
      const VR b1 = u >= 1 ? w0[u >= 1 ? u - 1 : 0] : w1[kC2 - 1];
      const VR b2 = u >= 2 ? w0[u >= 2 ? u - 2 : 0] : w1[kC2 - 2 + u];
      const VR f1 = u + 1 < kC2 ? w0[u + 1 < kC2 ? u + 1 : 0] : wn[0];
      VR xn = f1, xu = b1, xuu = b2;
      if constexpr (D3) {
        const bool c0 = m == u, c1 = m == ((u + kC2 - 1) & (kC2 - 1)), c7 = m == ((u + 1) & (kC2 - 1));
        const VR e = u == 0 ? e7p : e7;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
          xu[k] = c0 ? e7[k] : xu[k];
          xuu[k] = c0 ? e6[k] : (c1 ? e[k] : xuu[k]);
          xn[k] = c7 ? x0[k] : xn[k];
        }
      }
      // the rows below and above the lane's: lane l - 1 is a step behind in
      // the same column, lane l + 1 a step ahead
      VR r1, r2, rn;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        r1[k] = k >= 1 ? uc[k >= 1 ? k - 1 : 0] : below(b1[NR - 1]);
        r2[k] = k >= 2 ? uc[k >= 2 ? k - 2 : 0] : (NR == 1 ? below(below(b2[0])) : below(b1[NR >= 2 ? NR - 2 + k : 0]));
        rn[k] = k + 1 < NR ? uc[k + 1 < NR ? k + 1 : 0] : above(f1[0]);
      }
      VR out = VR(T(0));
      bool hole = false;
      auto axis = [&](auto e_, const VR& un, const VR& uu, const VR& uuu) {
        constexpr int e = decltype(e_)::value;
        unsigned any = 0;
#pragma unroll
        for (int k = 0; k < NR; ++k) any |= 15u << (4 * (k * ND + e));
        if (__any((cw & any) != 0)) {
          if (e == 0) hole = true;
#pragma unroll
          for (int k = 0; k < NR; ++k)
            out[k] = fma(cf[e], grad_diff<T>(cw >> (4 * (k * ND + e)), uc[k], un[k], uu[k], uuu[k], W[e]), out[k]);
        } else {
#pragma unroll
          for (int k = 0; k < NR; ++k) out[k] = fma(cf[e], (un[k] - uu[k]) - (uc[k] - uuu[k]), out[k]);
        }
      };
      axis(std::integral_constant<int, 0>(), xn, xu, xuu);
      axis(std::integral_constant<int, 1>(), rn, r1, r2);
      if constexpr (D3) axis(std::integral_constant<int, 2>(), wn[u], w1[u], w2[u]);
      if (hole) {
#pragma unroll
        for (int k = 0; k < NR; ++k)
          out[k] = ((cw >> (4 * k * ND)) & CC_UP) == CC_NOCELL ? T(0) : out[k];
      }
      const int so = D3 && m > u ? so0 : so1;
      stv<VR>(out, CR, idle ? kOOB : so, (c * kC2 + u) * STEP);
    }
#pragma unroll
    for (int u = 0; u < kC2; ++u) {
      if constexpr (D3) w2[u] = w1[u];
      w1[u] = w0[u];
      w0[u] = wn[u];
      wn[u] = nx[u];
      cd[u] = cdn[u];
    }
    if constexpr (D3) {
      e7p = e7;
      e7 = n7;
      e6 = n6;
      x0 = n0;
    }
  }
}

template <typename T>
hipError_t march(const CorrArgs& a, int nr, bool d3, hipStream_t st) {
  const dim3 grid((unsigned)(((long long)a.n_grp * a.n_unit + 3) / 4)), block(256);
  if (d3 && nr == 1) hipLaunchKernelGGL((corr_march_kernel<T, 1, true>), grid, block, 0, st, a);
  else if (d3 && nr == 2) hipLaunchKernelGGL((corr_march_kernel<T, 2, true>), grid, block, 0, st, a);
  else if (!d3 && nr == 1) hipLaunchKernelGGL((corr_march_kernel<T, 1, false>), grid, block, 0, st, a);
  else if (!d3 && nr == 2) hipLaunchKernelGGL((corr_march_kernel<T, 2, false>), grid, block, 0, st, a);
  else if (!d3 && nr == 4) hipLaunchKernelGGL((corr_march_kernel<T, 4, false>), grid, block, 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_corr_march(int prec, const CorrArgs& a, int nr, bool d3, hipStream_t st) {
  if (a.n_grp <= 0 || a.n_unit <= 0) return hipSuccess;
  return prec == BTE_PREC_FP32 ? march<float>(a, nr, d3, st) : march<double>(a, nr, d3, st);
}

}  // namespace bte
