// Spike lists of a raster and the spike term (gfx950).
//
// Lists, from the masks:
//   window-major  ent2[]: for every window of 1024 bins and neuron j its bins
//                 in order as offsets 16 (t mod 1024) into the window's tile
//                 (gather.h), padded to groups of four with the offset of a
//                 zero row; end2[w Np + j] the end of j's groups (end2[-1] = 0);
//   time-major    ent1[]: j | (bin mod 2^15) << 16 in (bin, neuron) order, bit
//                 31 set in a bin's first entry; off1[s] the first entry of
//                 subtile s (64 bins); for the recurrence (recur.hip).
//
// Spike term: dSigma[i][j] = sum_t s_i[t] x_j[t] (Eq. (12)), and dSigmaY with
// y = dx/dtau, in FP64, once per tau.  A workgroup holds 16 columns j of the
// trace over a window in LDS and every row i adds them up at its spikes; on
// the event grid the trace at a spike of i is the left limit v_j(t^-) of
// Eq. (12), x decayed over the whole slot before it.  Partials per time split
// are reduced in a fixed order.  Bound by the LDS reads (8 bytes a spike and
// column, in fours: 1.8 times the spikes at N = 1000, where the longest of a
// wave's eight lists sets its pace) and their latency.  N = 1000, 1.2e6 bins,
// 7.7e6 spikes: 2.45 ms; a wave walking its 16 rows' spikes with the sums in
// LDS and the trace selected per spike took 8.95 ms.
#include <algorithm>

#include "gather.h"

namespace {

using namespace glmr_gather;

// ------------------------------------------------------------------ lists
// per window: groups of four of all its neurons; per subtile: spikes
__global__ __launch_bounds__(256) void k_list_count(ListArgs a) {
  __shared__ int sub[GW / 64], quads;
  const int64_t w = blockIdx.x;
  const int tid = threadIdx.x;
  if (tid < GW / 64) sub[tid] = 0;
  if (tid == 0) quads = 0;
  __syncthreads();
  int mine[GW / 64], q = 0;
#pragma unroll
  for (int k = 0; k < GW / 64; ++k) mine[k] = 0;
  for (int64_t j = tid; j < a.Np; j += 256) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < GW / 64; ++k) {
      const int64_t s = w * (GW / 64) + k;
      if (s >= a.NS) continue;
      int n = 0;
      for (int p = 0; p < a.planes; ++p) n += __builtin_popcountll(a.masks[((int64_t)p * a.NS + s) * a.Np + j]);
      mine[k] += n;
      c += n;
    }
    q += (c + 3) >> 2;
  }
  if (q) atomicAdd(&quads, q);
#pragma unroll
  for (int k = 0; k < GW / 64; ++k)
    if (mine[k]) atomicAdd(&sub[k], mine[k]);
  __syncthreads();
  if (tid == 0) a.wcnt[w] = quads;
  if (a.scnt && tid < GW / 64 && w * (GW / 64) + tid < a.NS) a.scnt[w * (GW / 64) + tid] = sub[tid];
}

// window-major lists: the neurons of a window in order, 256 at a time
__global__ __launch_bounds__(256) void k_list_windows(ListArgs a) {
  __shared__ int wsum[4];
  const int64_t w = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = a.woff[w];
  if (w == 0 && tid < 4) a.end2[tid - 4] = 0;
  for (int64_t j0 = 0; j0 < a.Np; j0 += 256) {
    const int64_t j = j0 + tid;
    uint64_t m0[GW / 64];
    int c = 0;
#pragma unroll
    for (int k = 0; k < GW / 64; ++k) {
      const int64_t s = w * (GW / 64) + k;
      m0[k] = (j < a.Np && s < a.NS) ? a.masks[s * a.Np + j] : 0ull;
      c += __builtin_popcountll(m0[k]);
      if (m0[k])
        for (int p = 1; p < a.planes; ++p) c += __builtin_popcountll(a.masks[((int64_t)p * a.NS + s) * a.Np + j]);
    }
    const int q = (c + 3) >> 2;
    int incl = q;  // inclusive prefix over the 256 neurons
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      before += k < wave ? wsum[k] : 0;
      total += wsum[k];
    }
    __syncthreads();
    const int end = base + before + incl;
    base += total;
    if (j >= a.Np) continue;
    a.end2[w * a.Np + j] = end;
    uint16_t* dst = a.ent2 + (int64_t)(end - q) * 4;
    int n = 0;
#pragma unroll
    for (int k = 0; k < GW / 64; ++k) {
      uint64_t m = m0[k];
      while (m) {
        const int b = __builtin_ctzll(m);
        m &= m - 1;
        int rep = 1;
        for (int p = 1; p < a.planes; ++p)
          rep += (int)((a.masks[((int64_t)p * a.NS + w * (GW / 64) + k) * a.Np + j] >> b) & 1ull);
        for (; rep > 0; --rep) dst[n++] = (uint16_t)((k * 64 + b) * GI);
      }
    }
    for (; n < 4 * q; ++n) dst[n] = (uint16_t)(GW * GI);
  }
}

// time-major lists: one wave per subtile, lane = bin; the columns with spikes
// are walked in order, each lane counting (then writing) those of its bin
__global__ __launch_bounds__(256) void k_list_bins(ListArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (s >= a.NS) return;
  auto word = [&](uint64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
  };
  int pos = 0, first = 0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int64_t j0 = 0; j0 < a.Np; j0 += 64) {
      for (int p = 0; p < a.planes; ++p) {
        if (p && pass) break;
        const uint64_t m = a.masks[((int64_t)p * a.NS + s) * a.Np + j0 + lane];
        uint64_t nz = __ballot(m != 0);
        while (nz) {
          const int l = __builtin_ctzll(nz);
          nz &= nz - 1;
          const bool hit = (word(m, l) >> lane) & 1ull;
          if (!hit) continue;
          if (pass == 0) {
            ++pos;
          } else {
            // the bin's first entry carries the flag
            const uint32_t e = (uint32_t)(j0 + l) | (((uint32_t)(s * 64 + lane) & 0x7fffu) << 16);
            a.ent1[pos] = pos == first ? e | 0x80000000u : e;
            ++pos;
            for (int q = 1; q < a.planes; ++q)
              if ((a.masks[((int64_t)q * a.NS + s) * a.Np + j0 + l] >> lane) & 1ull) a.ent1[pos++] = e;
          }
        }
      }
    }
    if (pass == 0) {
      int incl = pos;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      pos = first = a.off1[s] + incl - pos;
    }
  }
}

// Spike term: columns j0 .. j0 + 15 of x (Y: of dx/dtau) over a window in LDS,
// every row i adds up the columns at its spikes.  On the event grid the trace
// at a spike is its left limit, x decayed over the whole slot.
template <bool Y, bool EV, int JB>
__global__ __launch_bounds__(GNT) void k_spk_gather(SpikeTermArgs a) {
  extern __shared__ __align__(16) double tile[];
  const int tid = threadIdx.x, il = tid & (GI - 1), tb = tid / GI;
  const int64_t ncb = a.Np / GI;
  const int64_t j = (int64_t)(blockIdx.x % ncb) * GI + il;
  const int64_t ib0 = (int64_t)(blockIdx.x / ncb) * (GG * JB);
  const int gl = tid & (GL - 1);  // the lane's columns of the sums: 2 gl and the next
  const int64_t split = blockIdx.y;
  const int64_t nw = (a.NS * 64 + GW - 1) / GW, per = (nw + a.splits - 1) / a.splits;
  const int64_t w0 = split * per, w1 = w0 + per < nw ? w0 + per : nw;
  const int64_t i0 = ib0 + (int64_t)(tid / GL) * JB;  // its group's rows
  const bool rows = i0 < a.Np;
  Cols acc[JB];
#pragma unroll
  for (int k = 0; k < JB; ++k) acc[k] = Cols{0.0, 0.0};
  if (tid < GI) tile[GW * GI + tid] = 0.0;
  uint2* es = (uint2*)(tile + ENTRIES);
  const uint2* __restrict__ ent = (const uint2*)a.ent2;
  const int64_t iend = ib0 + GG * JB < a.Np ? ib0 + GG * JB : a.Np;
  const int m0 = 16 * (tb & 3);
  const double ag = EV ? 0.0 : a.tab->pw[1];
  const double pwm = EV ? 0.0 : a.tab->pw[m0];
  // carry, spikes and list bounds of the next window, loaded while this one is gathered
  double Cn = 0.0, CYn = 0.0;
  uint64_t mn = 0;
  Ends en{0, 0};
  auto fetch = [&](int64_t w) {
    const int64_t s = w * (GW / 64) + (tb >> 2);
    const bool in = s < a.NS;
    Cn = in ? a.C64[s * a.Np + j] : 0.0;
    if (Y) CYn = in ? a.CY64[s * a.Np + j] : 0.0;
    mn = in ? a.masks[s * a.Np + j] : 0ull;
    if (rows) en = load_ends<JB>(a.end2, w * a.Np + i0, gl);
  };
  if (w0 < w1) fetch(w0);
  for (int64_t w = w0; w < w1; ++w) {
    const int64_t s = w * (GW / 64) + (tb >> 2);
    const bool in = s < a.NS;
    const double C = Cn;
    const uint64_t mk = mn;
    const Ends ec = en;
    const int base = a.end2[w * a.Np + ib0 - 1], n = a.end2[w * a.Np + iend - 1] - base;
    const uint32_t win = (uint32_t)(mk >> m0) & 0xffffu;
    double x = 0.0, y = 0.0, zs = 0.0, ys = 0.0;
    for (int p = 0; p < (mk ? a.planes : 0); ++p) {
      uint64_t below = (p == 0 ? mk : a.masks[((int64_t)p * a.NS + s) * a.Np + j]) & ((1ull << m0) - 1);
      while (below) {
        const int b = __builtin_ctzll(below);
        below &= below - 1;
        if (EV) {
          zs += a.ev.ainv[s * 64 + b];
        } else {
          const double t = a.tab->pw[m0 - b - 1];
          zs += t;
          if (Y) ys += (double)(m0 - b - 1) * t;
        }
      }
    }
    if (EV) x = in ? a.ev.pw[s * 64 + m0] * (C + zs) : 0.0;
    else x = C * pwm + zs;
    if (Y) y = pwm * (CYn + (double)m0 * a.ctau * C) + a.ctau * ys;
    __syncthreads();  // the previous window's tile has been read
    stage_entries(es, ent, base, n);
    double* dst = tile + tb * 16 * GI + il;
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      double cnt = (double)((win >> m) & 1u);
      if (a.planes > 1 && win)
        for (int p = 1; p < a.planes; ++p)
          cnt += (double)((a.masks[((int64_t)p * a.NS + s) * a.Np + j] >> (m0 + m)) & 1ull);
      const double d = EV ? (in ? a.ev.edec[s * 64 + m0 + m] : 0.0) : ag;
      dst[m * GI] = Y ? y : (EV ? d * x : x);
      if (Y) y = d * (y + a.ctau * x);
      x = d * x + cnt;
    }
    __syncthreads();
    if (w + 1 < w1) fetch(w + 1);
    gather_lists<JB>(acc, tile, ent, base, n, ec, gl, rows);
  }
  if (!rows) return;
  double* out = a.part + split * a.Np * a.Np;
#pragma unroll
  for (int k = 0; k < JB; ++k) *(Cols*)(out + (i0 + k) * a.Np + (j - il + 2 * gl)) = acc[k];
}

__global__ void k_split_reduce(const double* part, int splits, int64_t n, double* out) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x) {
    double v = 0.0;
    for (int sp = 0; sp < splits; ++sp) v += part[sp * n + k];
    out[k] = v;
  }
}

template <bool Y, bool EV>
hipError_t spk_gather(const SpikeTermArgs& a, hipStream_t st) {
  const int jb = gather_jb(a.Np);
  const int64_t blocks = (a.Np / GI) * ((a.Np + GG * jb - 1) / (GG * jb));
  switch (jb) {
    case 1: return run_gather(k_spk_gather<Y, EV, 1>, a, blocks, a.splits, st);
    case 2: return run_gather(k_spk_gather<Y, EV, 2>, a, blocks, a.splits, st);
    case 4: return run_gather(k_spk_gather<Y, EV, 4>, a, blocks, a.splits, st);
    default: return run_gather(k_spk_gather<Y, EV, 8>, a, blocks, a.splits, st);
  }
}

}  // namespace

hipError_t launch_list_count(const ListArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_list_count, dim3((unsigned)((a.NS * 64 + GW - 1) / GW)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_list_windows(const ListArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_list_windows, dim3((unsigned)((a.NS * 64 + GW - 1) / GW)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_list_bins(const ListArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_list_bins, dim3((unsigned)((a.NS + 3) / 4)), dim3(256), 0, st, a);
  return hipGetLastError();
}

int64_t gather_blocks(int64_t cols, int64_t Np) { return blocks_of(cols, Np); }

hipError_t launch_spike_term(const SpikeTermArgs& a, hipStream_t st) {
  hipError_t e = a.ev.pw ? spk_gather<false, true>(a, st) : spk_gather<false, false>(a, st);
  if (e != hipSuccess) return e;
  const int64_t n = a.Np * a.Np;
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_split_reduce, dim3(blocks), dim3(256), 0, st, a.part, a.splits, n, a.dsig);
  if (a.CY64 && a.dsigY) {
    e = spk_gather<true, false>(a, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_split_reduce, dim3(blocks), dim3(256), 0, st, a.part, a.splits, n, a.dsigY);
  }
  return hipGetLastError();
}
