// Parameter-free parts of the likelihood, computed once per kernel time
// constant tau (Sec. 2.3.3 notes dSigma needs computing only once; Sec. 2.6.1
// caches everything that does not depend on theta):
//
//  * carries C[s][j] = x_j[64 s], the trace at every subtile start, and
//    CY[s][j] = dx_j/dtau at the same bins.  Over one subtile
//      C[s+1]  = A C[s] + D[s],               A = a^64,
//      CY[s+1] = A (CY[s] + 64 c C[s]) + DY[s],  c = dt / tau^2,
//    with D[s] = sum_b a^(63-b), DY[s] = c sum_b (63-b) a^(63-b) over the
//    spikes of subtile s (the grid form of Eq. (8)/(13)).  The scan runs in
//    FP64 in three passes: local segments of 64 subtiles, a sequential pass
//    over segment aggregates, and a fix-up that adds the carried-in state
//    (after k subtiles: C += A^k C_in, CY += A^k CY_in + 64 k c A^k C_in).
//
//  * On the event grid (continuous time) the same scan runs with the per-slot
//    decays of events.hip: C[s+1] = asub[s] (C[s] + sum_b ainv[64 s + b]).
//
// The spike term dSigma of Eq. (12) is in spikes.hip.
#include "common.h"

namespace {

// EV: event grid, per-subtile decays; seg[...][1] then holds the product of
// the segment's subtile decays (there is no y).  All three passes run along a
// column with few threads, so latency bounds them: masks and aggregates are
// loaded CA ahead and the decays come from LDS.  The three passes take 180 us
// at N = 1000, 1.2e6 bins and 44 us at N = 50, 2e4 bins (one load after the
// other: 271 and 70 us).
constexpr int CA = 8;
template <bool EV>
__global__ void k_carry_local(CarryArgs c) {
  __shared__ double pw[64];
  if (!EV && threadIdx.x < 64) pw[threadIdx.x] = c.tab->pw[threadIdx.x];
  __syncthreads();
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t g = blockIdx.y;
  if (j >= c.Np) return;
  const int64_t s0 = g * c.G;
  const int64_t s1 = (s0 + c.G < c.NS) ? s0 + c.G : c.NS;
  if (EV) {
    double x = 0.0, prod = 1.0;
    for (int64_t sb = s0; sb < s1; sb += CA) {
      uint64_t m0[CA];
#pragma unroll
      for (int e = 0; e < CA; ++e) m0[e] = sb + e < s1 ? c.masks[(sb + e) * c.Np + j] : 0ull;
#pragma unroll
      for (int e = 0; e < CA; ++e) {
        const int64_t s = sb + e;
        if (s >= s1) break;
        c.C64[s * c.Np + j] = x;
        double D = 0.0;
        for (int p = 0; p < c.planes; ++p) {
          uint64_t mk = p ? c.masks[((int64_t)p * c.NS + s) * c.Np + j] : m0[e];
          while (mk) {
            const int b = __builtin_ctzll(mk);
            mk &= mk - 1;
            D += c.ev.ainv[s * 64 + b];
          }
        }
        const double A = c.ev.asub[s];
        x = A * (x + D);
        prod *= A;
      }
    }
    c.seg[(g * c.Np + j) * 2 + 0] = x;
    c.seg[(g * c.Np + j) * 2 + 1] = prod;
    return;
  }
  const double A = c.tab->apow[1];
  double x = 0.0, y = 0.0;
  for (int64_t sb = s0; sb < s1; sb += CA) {
    uint64_t m0[CA];
#pragma unroll
    for (int e = 0; e < CA; ++e) m0[e] = sb + e < s1 ? c.masks[(sb + e) * c.Np + j] : 0ull;
#pragma unroll
    for (int e = 0; e < CA; ++e) {
      const int64_t s = sb + e;
      if (s >= s1) break;
      c.C64[s * c.Np + j] = x;
      if (c.want_y) c.CY64[s * c.Np + j] = y;
      double D = 0.0, DY = 0.0;
      for (int p = 0; p < c.planes; ++p) {
        uint64_t mk = p ? c.masks[((int64_t)p * c.NS + s) * c.Np + j] : m0[e];
        while (mk) {
          int b = __builtin_ctzll(mk);
          mk &= mk - 1;
          const double w = pw[63 - b];
          D += w;
          DY += (double)(63 - b) * w;
        }
      }
      y = A * (y + 64.0 * c.ctau * x) + c.ctau * DY;
      x = A * x + D;
    }
  }
  c.seg[(g * c.Np + j) * 2 + 0] = x;
  c.seg[(g * c.Np + j) * 2 + 1] = y;
}

template <bool EV>
__global__ void k_carry_scan(CarryArgs c, int64_t nseg) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= c.Np) return;
  const double2* __restrict__ seg = (const double2*)c.seg + j;
  double2* __restrict__ segin = (double2*)c.segin + j;
  const int64_t last = c.NS - (nseg - 1) * c.G;  // subtiles of the last segment
  const double Afull = EV ? 0.0 : c.tab->apow[c.G], Alast = EV ? 0.0 : c.tab->apow[last];
  double cin = 0.0, cyin = 0.0;
  for (int64_t gb = 0; gb < nseg; gb += CA) {
    double2 v[CA];
#pragma unroll
    for (int e = 0; e < CA; ++e) v[e] = gb + e < nseg ? seg[(gb + e) * c.Np] : double2{0.0, 0.0};
#pragma unroll
    for (int e = 0; e < CA; ++e) {
      const int64_t g = gb + e;
      if (g >= nseg) break;
      segin[g * c.Np] = double2{cin, cyin};
      if (EV) {
        cin = v[e].y * cin + v[e].x;
        continue;
      }
      const int64_t len = g + 1 < nseg ? c.G : last;
      const double AG = g + 1 < nseg ? Afull : Alast;
      cyin = AG * cyin + 64.0 * (double)len * c.ctau * AG * cin + v[e].y;
      cin = AG * cin + v[e].x;
    }
  }
}

template <bool EV>
__global__ void k_carry_apply(CarryArgs c) {
  __shared__ double apow[64];
  if (!EV && threadIdx.x < 64) apow[threadIdx.x] = c.tab->apow[threadIdx.x];
  __syncthreads();
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t g = blockIdx.y;
  if (j >= c.Np) return;
  const int64_t s0 = g * c.G;
  const int64_t s1 = (s0 + c.G < c.NS) ? s0 + c.G : c.NS;
  const double cin = c.segin[(g * c.Np + j) * 2 + 0];
  const double cyin = c.segin[(g * c.Np + j) * 2 + 1];
  if (EV) {
    double Ak = 1.0;  // decay from the segment start to subtile s
    for (int64_t sb = s0; sb < s1; sb += CA) {
      double v[CA], as[CA];
#pragma unroll
      for (int e = 0; e < CA; ++e) {
        v[e] = sb + e < s1 ? c.C64[(sb + e) * c.Np + j] : 0.0;
        as[e] = sb + e < s1 ? c.ev.asub[sb + e] : 0.0;
      }
#pragma unroll
      for (int e = 0; e < CA; ++e) {
        const int64_t s = sb + e;
        if (s >= s1) break;
        const double x = v[e] + Ak * cin;
        c.C64[s * c.Np + j] = x;
        if (c.C32) c.C32[s * c.Np + j] = (float)x;
        Ak *= as[e];
      }
    }
    return;
  }
  for (int64_t sb = s0; sb < s1; sb += CA) {
    double v[CA], vy[CA];
#pragma unroll
    for (int e = 0; e < CA; ++e) {
      v[e] = sb + e < s1 ? c.C64[(sb + e) * c.Np + j] : 0.0;
      vy[e] = c.want_y && sb + e < s1 ? c.CY64[(sb + e) * c.Np + j] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < CA; ++e) {
      const int64_t s = sb + e, k = s - s0;
      if (s >= s1) break;
      const double Ak = apow[k];
      const double x = v[e] + Ak * cin;
      c.C64[s * c.Np + j] = x;
      if (c.C32) c.C32[s * c.Np + j] = (float)x;
      if (c.want_y) {
        const double y = vy[e] + Ak * cyin + 64.0 * (double)k * c.ctau * Ak * cin;
        c.CY64[s * c.Np + j] = y;
        if (c.CY32) c.CY32[s * c.Np + j] = (float)y;
      }
    }
  }
}

}  // namespace

hipError_t launch_carries(const CarryArgs& c, hipStream_t st) {
  const int64_t nseg = (c.NS + c.G - 1) / c.G;
  dim3 grid((unsigned)((c.Np + 255) / 256), (unsigned)nseg);
  if (c.ev.pw) {
    hipLaunchKernelGGL(k_carry_local<true>, grid, dim3(256), 0, st, c);
    hipLaunchKernelGGL(k_carry_scan<true>, dim3((unsigned)((c.Np + 63) / 64)), dim3(64), 0, st, c, nseg);
    hipLaunchKernelGGL(k_carry_apply<true>, grid, dim3(256), 0, st, c);
  } else {
    hipLaunchKernelGGL(k_carry_local<false>, grid, dim3(256), 0, st, c);
    hipLaunchKernelGGL(k_carry_scan<false>, dim3((unsigned)((c.Np + 63) / 64)), dim3(64), 0, st, c, nseg);
    hipLaunchKernelGGL(k_carry_apply<false>, grid, dim3(256), 0, st, c);
  }
  return hipGetLastError();
}
