// The likelihood by the trace's recurrence (FP64 and FP32 modes) on the
// raster's spike lists (gfx950).
//
// The potentials obey the trace's own recurrence (Eq. (13)): with
// V_i[t] = sum_j J_ij x_j[t] and d_t the decay over bin t (a on the regular
// grid, e^{-delta_t} on the event grid),
//   V_i[t+1] = d_t V_i[t] + sum_{spikes j of bin t} J_ij,
// so a bin costs as many additions a row as it holds spikes (6.6 of 1000
// neurons at 5 to 10 spikes per second and 1 ms) instead of the N products of
// the dense contraction.  The integral of Eq. (12) has the same structure
// backwards in time: G_ij = sum_t W_i[t] x_j[t] = sum_{spikes t of j} R_i[t] with
//   R_i[t-1] = W_i[t] + d_t R_i[t]
// (W_i = exp V_i, or the interval integral of Eq. (14)).  All sums are FP64,
// in a fixed order.
//
//   k_rec_fwd     one wave per 64 rows i and time segment: the recurrence for
//                 V from its value at the segment start, exp (or the interval
//                 integrals), row sums, and W in [bin][row] order.
//   k_rec_gather  one workgroup per 16 rows i and time split, windows of 1024
//                 bins walked backwards: R in LDS, then every neuron j adds up
//                 R at its spikes in a register.
// Segments and splits start from the carries C (trace at every 64th bin):
// V at a segment start is C J^T (k_carry_gemm; a 1/64 .. 1/1024 of the dense
// work), and a split's W acts on all earlier spikes through
// sum_t W_i[t] (decay since its start) times C_j at its start (k_rec_reduce).
//
// What bounds it (N = 1000, 1.2e6 bins, 7.7e6 spikes, one evaluation with the
// gradient): k_rec_fwd 2.5 ms (FP32) and 2.9 ms (FP64: twice the bytes of J
// from the L2), half of it vector and scalar issue (21 of the instructions a
// bin are the exponential, 7 a spike); k_rec_gather 3.1 ms, LDS reads and the
// phases that form a tile.  The dense kernels took 56 and 58 ms.  On the event
// grid (FP64): k_rec_fwd_ev 0.130 ms at N = 150, 6.6e4 slots and 4.1 us per
// thousand slots at N = 1000, the FP64 arithmetic of the integrals and, with four
// waves a SIMD, its latency (at N = 150 0.145 ms with one term more, 0.47 ms
// written out per lane, with the closed forms as a call).
#include <algorithm>

#include "evfun.h"
#include "gather.h"

namespace {

using namespace glmr_gather;

// The rows of 16 lanes of a wave: in every lane, its pair's even and odd row.
struct Pair16 {
  double even, odd;
};
__device__ __forceinline__ Pair16 swap_rows(double x) {
  const u32x2 u = __builtin_bit_cast(u32x2, x);
  const auto lo = __builtin_amdgcn_permlane16_swap(u[0], u[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(u[1], u[1], false, false);
  return Pair16{__builtin_bit_cast(double, u32x2{lo[0], hi[0]}), __builtin_bit_cast(double, u32x2{lo[1], hi[1]})};
}
// the value 32 lanes on, in every lane that of the upper half
__device__ __forceinline__ double upper_half(double x) {
  const u32x2 u = __builtin_bit_cast(u32x2, x);
  const auto lo = __builtin_amdgcn_permlane32_swap(u[0], u[0], false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(u[1], u[1], false, false);
  return __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}

// Kernel G: rows i0 .. i0 + 15, windows of a split from the last to the
// first.  A thread holds 16 bins of one row: their W are loaded while the
// window before is gathered, a first backward pass gives the 16 bins' share
// of R, the shares are combined across the workgroup (a suffix scan), and a
// second pass with the carried-in value writes R to LDS.
template <typename WT, bool EV, int JB>
__global__ __launch_bounds__(GNT) void k_rec_gather(RecGArgs a) {
  extern __shared__ __align__(16) double tile[];
  double* wh = tile + TILE;       // [16 waves][GI] a wave's 64 bins: share of R before them
  double* wp = wh + 16 * GI;      // and their decay
  double* ce = wp + 16 * GI;      // [2][GI] R at a window's last bin, by the parity of the window
  uint2* es = (uint2*)(tile + ENTRIES);
  const uint2* __restrict__ ent = (const uint2*)a.ent2;
  const int tid = threadIdx.x, il = tid & (GI - 1), tb = tid / GI, wave = tid >> 6, tl = tb & 3;
  const int64_t nib = (a.N + GI - 1) / GI;
  const int64_t i = (int64_t)(blockIdx.x % nib) * GI + il;
  const int64_t jb0 = (int64_t)(blockIdx.x / nib) * (GG * JB);
  const int64_t split = blockIdx.y;
  const int64_t nw = (a.Lc + GW - 1) / GW;
  const int64_t w0 = split * a.wps, w1 = w0 + a.wps < nw ? w0 + a.wps : nw;
  const int gl = tid & (GL - 1);  // the lane's columns of the sums: 2 gl and the next
  const int64_t j0 = jb0 + (int64_t)(tid / GL) * JB;
  const bool rows = j0 < a.Np;
  Cols acc[JB];
#pragma unroll
  for (int k = 0; k < JB; ++k) acc[k] = Cols{0.0, 0.0};
  if (tid < GI) tile[GW * GI + tid] = 0.0;
  const double ag = a.a;
  // W of the window by raw buffer loads: the row offsets sit in scalar
  // registers and bins past the recording read as zero
  const int64_t valid = a.B - a.t0 < a.Lc ? a.B - a.t0 : a.Lc;
  const int voff = (int)((tb * 16 * a.Np + i) * (int64_t)sizeof(WT)), pitch = (int)(a.Np * (int64_t)sizeof(WT));
  WT wn[16];
  auto fetch = [&](int64_t w) {
    const int64_t n = valid - w * GW < GW ? valid - w * GW : GW;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const WT*)a.W + w * GW * a.Np), (short)0, n > 0 ? (int)(n * pitch) : 0, 0x00020000);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if constexpr (sizeof(WT) == 8)
        wn[m] = __builtin_bit_cast(WT, __builtin_amdgcn_raw_buffer_load_b64(r, voff, m * pitch, 0));
      else
        wn[m] = __builtin_bit_cast(WT, __builtin_amdgcn_raw_buffer_load_b32(r, voff, m * pitch, 0));
    }
  };
  const int64_t jend = jb0 + GG * JB < a.Np ? jb0 + GG * JB : a.Np;
  const int64_t wg = a.t0 / GW;  // the chunk's first window
  Ends en{0, 0};
  double cend = 0.0;  // R at the last bin of the window (uniform grid: in wave 0)
  if (!EV && tid < GI) ce[((w1 - 1) & 1) * GI + tid] = 0.0;
  double P = 1.0, P64 = 1.0;  // decay over 16 and (bins) 64 steps
  if (!EV) {
    P = ag * ag;
    P *= P;
    P *= P;
    P *= P;
    P64 = P * P;
    P64 *= P64;
  }
  if (w1 > w0) {
    fetch(w1 - 1);
    if (rows) en = load_ends<JB>(a.end2, (wg + w1 - 1) * a.Np + j0, gl);
  }
  for (int64_t w = w1 - 1; w >= w0; --w) {
    double h = 0.0;
    double dn[EV ? 16 : 1];
    if (EV) {
      const double* __restrict__ ed = a.ev.edec + a.t0 + w * GW + tb * 16;
      const bool in = a.t0 + w * GW + tb * 16 < a.NS64;
#pragma unroll
      for (int m = 0; m < 16; ++m) dn[m] = in ? ed[m] : 1.0;
      P = 1.0;
    }
#pragma unroll
    for (int m = 15; m >= 0; --m) {
      h = (double)wn[m] + (EV ? dn[m] : ag) * h;
      if (EV) P *= dn[m];
    }
    // hx, Px: what the later blocks of the wave (its rows of 16 lanes) add to
    // R at this block's end, and their decay; in row 0, ht and Pt with this block
    double hx, Px, ht, Pt;
    if constexpr (EV) {
      double hs = h, Ps = P;
      const double h1 = __shfl_down(hs, 16, 64), P1 = __shfl_down(Ps, 16, 64);
      if (tl < 3) { hs += Ps * h1; Ps *= P1; }
      const double h2 = __shfl_down(hs, 32, 64), P2 = __shfl_down(Ps, 32, 64);
      if (tl < 2) { hs += Ps * h2; Ps *= P2; }
      ht = hs;
      Pt = Ps;
      hx = __shfl_down(hs, 16, 64);
      Px = __shfl_down(Ps, 16, 64);
      if (tl == 3) { hx = 0.0; Px = 1.0; }
    } else {  // pairs of rows, then the pair two rows on; the decays are known
      // (by permutes through LDS, and with every wave going over all sixteen
      // shares and decays below, the kernel took 5 % longer)
      const bool odd = tl & 1;
      const Pair16 p = swap_rows(h);
      const double late = odd ? h : p.odd, pair = (odd ? p.even : h) + P * late, next = upper_half(pair);
      ht = pair + P * P * next;
      Pt = P64;
      hx = tl == 0 ? late + P * next : tl == 1 ? next : tl == 2 ? late : 0.0;
      Px = tl == 0 ? P * P * P : tl == 1 ? P * P : tl == 2 ? P : 1.0;
    }
    if (tl == 0) {
      wh[wave * GI + il] = ht;
      if (EV) wp[wave * GI + il] = Pt;
    }
    const Ends ec = en;
    const int base = a.end2[(wg + w) * a.Np + jb0 - 1], n = a.end2[(wg + w) * a.Np + jend - 1] - base;
    __syncthreads();  // (also: the previous window's tile has been read)
    stage_entries(es, ent, base, n);
    // into this wave from the later ones; on the uniform grid only wave 0
    // goes on to the window's start and passes it on through LDS (half the
    // reads, but the registers of the slots' decays leave no room for it)
    double c;
    if constexpr (EV) {
      double all = cend;
      c = cend;
#pragma unroll 4
      for (int v = 15; v >= 0; --v) {
        if (v == wave) c = all;
        all = wh[v * GI + il] + wp[v * GI + il] * all;
      }
      cend = all;
    } else {
      c = ce[(w & 1) * GI + il];
#pragma unroll 4
      for (int v = 15; v > wave; --v) c = wh[v * GI + il] + P64 * c;
      if (wave == 0) {
        cend = wh[il] + P64 * c;
        if (tl == 0) ce[((w - 1) & 1) * GI + il] = cend;
      }
    }
    double r = hx + Px * c;
    // converted again and not kept as FP64 across the barrier: on the event grid
    // that spilled 34 registers (kernel G 101 instead of 53 ms at N = 1000, one hour)
    if constexpr (sizeof(WT) == 4) {
#pragma unroll
      for (int m = 0; m < 16; ++m) asm volatile("" : "+v"(wn[m]));
    }
    double* dst = tile + tb * 16 * GI + il;
#pragma unroll
    for (int m = 15; m >= 0; --m) {
      dst[m * GI] = r;
      r = (double)wn[m] + (EV ? dn[m] : ag) * r;
    }
    __syncthreads();
    if (w > w0) {
      fetch(w - 1);
      if (rows) en = load_ends<JB>(a.end2, (wg + w - 1) * a.Np + j0, gl);
    }
    gather_lists<JB>(acc, tile, ent, base, n, ec, gl, rows);
  }
  if (blockIdx.x / nib == 0 && tb == 0) a.head[split * a.Np + i] = cend;
  if (!rows) return;
  double* out = (double*)a.Gp + split * a.Np * a.Np;
#pragma unroll
  for (int k = 0; k < JB; ++k) *(Cols*)(out + (j0 + k) * a.Np + (i - il + 2 * gl)) = acc[k];
}

// sum over the splits p0, p0 + step, ... of Gp[p][j][i] + head[p][i] C[start of p][j],
// eight loads in flight
__device__ __forceinline__ double sum_splits(const RecGArgs& a, int64_t i, int64_t j, int p0, int step) {
  const int64_t cstep = a.wps * (GW / 64) * a.Np, gstep = a.Np * a.Np;
  const double* __restrict__ gp = (const double*)a.Gp + j * a.Np + i;
  const double* __restrict__ C = a.C64 + (a.t0 >> 6) * a.Np + j;
  const double* __restrict__ hd = a.head + i;
  double v = 0.0;
#pragma unroll 8
  for (int p = p0; p < a.n_splits; p += step) v += gp[p * gstep] + hd[p * a.Np] * C[p * cstep];
  return v;
}

// G[i][j] (+)= that sum: 32 rows x 8 columns a workgroup (with 32 x 32
// a workgroup and a split at a time the few workgroups of a small network
// waited on memory: 87 us at 256 rows and 65 splits)
__global__ __launch_bounds__(256) void k_rec_reduce(RecGArgs a, int first) {
  __shared__ double t[8][33];
  const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 8;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t i = i0 + tx, j = j0 + ty;
  const double v = i < a.N ? sum_splits(a, i, j, 0, 1) : 0.0;
  t[ty][tx] = v;
  __syncthreads();
  double* g = a.G64 + (i0 + (threadIdx.x >> 3)) * a.Np + j0 + (threadIdx.x & 7);
  *g = (first ? 0.0 : *g) + t[threadIdx.x & 7][threadIdx.x >> 3];
}

// The end of an evaluation in one launch, workgroups of two kinds.  The first
// Np / RROWS take RROWS rows each: the sums of kernel U's partials over the
// segments, L_i, dL/dmu_i and dL/dtau_i.  The others (with the gradient) take
// a 32 x 8 tile of the last chunk's reduction (k_rec_reduce), a quarter of the
// splits a thread, and write dL/dJ: it needs no row sum.  All are short and
// bound by latency, hence many small workgroups with 8 or 16 loads in flight a
// thread: 14 us at N = 150, 65 splits and 2064 segments on the event grid (32
// x 32 tiles without a split of the splits: 25 us; reduction, row sums,
// assembly and totals as four kernels: 24 us and three gaps), 9 us for the
// rows alone at N = 500 (32 rows a workgroup: 19 us).
constexpr int RROWS = 8;
__global__ __launch_bounds__(1024) void k_rec_finish(RecGArgs a, AssembleArgs s, int first) {
  const int tid = threadIdx.x;
  const int64_t nb = s.Np / 32, rb = s.Np / RROWS;
  if (blockIdx.x >= rb) {
    __shared__ double t[4][8][33];
    const int64_t k = blockIdx.x - rb, i0 = k % nb * 32, j0 = k / nb * 8;
    const int tx = tid & 31, ty = (tid >> 5) & 7, q = tid >> 8;
    t[q][ty][tx] = i0 + tx < a.N ? sum_splits(a, i0 + tx, j0 + ty, q, 4) : 0.0;
    __syncthreads();
    const int u = tid >> 3, w = tid & 7;
    const int64_t r = i0 + u, c = j0 + w;
    if (tid >= 256 || r >= s.N) return;
    const double G = (first ? 0.0 : a.G64[r * s.Np + c]) + ((t[0][w][u] + t[1][w][u]) + (t[2][w][u] + t[3][w][u]));
    const double g = c < s.N ? s.dsig[r * s.Np + c] - s.dt * s.rowscale[r] * G : 0.0;
    s.gJ[r * s.Np + c] = g;
    if (s.out_gJ && c < s.N) s.out_gJ[r * s.N + c] = g;
    return;
  }
  __shared__ double sums[2][16][RROWS], dot[2][RROWS];
  const int64_t i0 = (int64_t)blockIdx.x * RROWS;
  const int lane = tid & 63, wave = tid >> 6;
  // sixteen segments' loads in flight, then over the wave's lanes of a row
  for (int which = 0; which < 2; ++which) {
    const double* __restrict__ rp = which ? s.rowpartV : s.rowpart;
    double v = 0.0;
    for (int64_t k0 = tid / RROWS; rp && k0 < s.n_tiles; k0 += 1024 / RROWS * 16) {
      double w[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t k = k0 + 1024 / RROWS * e;
        w[e] = k < s.n_tiles ? rp[k * s.Np + i0 + tid % RROWS] : 0.0;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) v += w[e];
    }
#pragma unroll
    for (int o = 32; o >= RROWS; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane < RROWS) sums[which][wave][lane] = v;
  }
  // sum_j J_ij dSigma_ij (and of dSigmaY), a wave a row
  if (wave < RROWS) {
    const int64_t at = (i0 + wave) * s.Np;
    double v = 0.0, vy = 0.0;
#pragma unroll 4
    for (int64_t j = lane; j < s.N; j += 64) {
      v += s.Jr[at + j] * s.dsig[at + j];
      if (s.dsigY) vy += s.Jr[at + j] * s.dsigY[at + j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      v += __shfl_xor(v, o, 64);
      vy += __shfl_xor(vy, o, 64);
    }
    if (lane == 0) {
      dot[0][wave] = v;
      dot[1][wave] = vy;
    }
  }
  __syncthreads();
  // the workgroup's rows in one piece (some arrays are host memory)
  const int64_t i = i0 + tid;
  if (tid >= RROWS || i >= s.N) return;
  double total[2] = {0.0, 0.0};
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    total[0] += sums[0][w][tid];
    total[1] += sums[1][w][tid];
  }
  const double sc = s.dt * s.rowscale[i], integ = sc * total[0];
  const double ll = (double)s.q[i] * s.mu[i] + dot[0][tid] - integ, gm = (double)s.q[i] - integ;
  s.ll_rows[i] = ll;
  if (s.host_rows) s.host_rows[i] = ll;
  if (s.out_rows) s.out_rows[i] = ll;
  if (s.gmu) s.gmu[i] = gm;
  if (s.out_gmu) s.out_gmu[i] = gm;
  if (s.tau_rows) {
    const double tr = dot[1][tid] - sc * total[1];
    s.tau_rows[i] = tr;
    if (s.host_rows) s.host_rows[s.N + i] = tr;
  }
}

// ------------------------------------------------------------------ forward
constexpr uint32_t ENT_FIRST = 0x80000000u;
__device__ __forceinline__ int ent_bin(uint32_t e, uint32_t base) { return (int)(((e >> 16) - base) & 0x7fffu); }

template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <typename T>
__device__ __forceinline__ void buf_store(T v, __amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, 0);
}

// R neighbouring values of T by one buffer access
template <typename T, int R>
struct Vals {
  T v[R];
};
template <typename T, int R>
__device__ __forceinline__ Vals<T, R> buf_load_r(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (R == 1) return Vals<T, R>{{buf_load<T>(r, voff, soff)}};
  else if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(Vals<T, R>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  else
    return __builtin_bit_cast(Vals<T, R>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <typename T, int R>
__device__ __forceinline__ void buf_store_r(const Vals<T, R>& x, __amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (R == 1) buf_store<T>(x.v[0], r, voff, soff);
  else if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, x), r, voff, soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, voff, soff, 0);
}

// One wave per 64 R rows (a lane holds R neighbours) and segment of g.seg bins
// (PART: less than a subtile).  With two rows a lane the scalar unit and the
// entries' loads serve twice the sums.  A batch is 8 entries (uniform loads, a batch ahead); each
// entry's row of J^T is loaded as the entry 8 before it is used.  Row offsets
// are 32-bit scalars of one buffer: with 64-bit addresses and a bin comparison
// per entry the scalar unit, which a CU's four SIMDs share, set the time (174
// scalar instructions a bin and wave at N = 1000).
constexpr int FB8 = 8;

template <typename T, int R, bool TAU, bool STORE, bool FUSED, bool PART>
__global__ __launch_bounds__(256) void k_rec_fwd(const uint32_t* __restrict__ ent, const int32_t* __restrict__ off,
                                                 const T* __restrict__ Jt, const double* __restrict__ Dc,
                                                 const double* __restrict__ Vc, const double* __restrict__ C64,
                                                 const double* __restrict__ CY64, T* __restrict__ W,
                                                 double* __restrict__ rowpart, double* __restrict__ rowpartV,
                                                 RecFDims g) {
  const int lane = threadIdx.x & 63;
  const uint32_t nib = (uint32_t)((g.N + 64 * R - 1) / (64 * R));
  const int i = ((int)(blockIdx.x % nib) * 64 + lane) * R;
  const int64_t sg = (int64_t)(blockIdx.x / nib) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (sg >= g.n_seg) return;
  const int64_t t0 = g.t0 + sg * g.seg;              // the segment's first bin
  const int64_t s0 = t0 >> 6;
  const int skip = PART ? (int)(t0 & 63) : 0;        // bins of its subtile before it
  const int64_t left = g.B - s0 * 64;
  const int tend = (int)(left < skip + g.seg ? left : skip + g.seg);  // bins counted from 64 s0
  const int pitch = (int)(g.Np * (int64_t)sizeof(T)), voff = i * (int)sizeof(T);
  const __amdgpu_buffer_rsrc_t jr =
      __builtin_amdgcn_make_buffer_rsrc((void*)Jt, (short)0, (int)(g.Np * pitch), 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(STORE ? W + (t0 - g.tw) * g.Np : nullptr), (short)0, STORE ? (int)(g.seg * pitch) : 0, 0x00020000);
  const double ag = g.a;
  double D[R], V[R], sum[R], sumv[R], acc[R];
#pragma unroll
  for (int k = 0; k < R; ++k) D[k] = V[k] = sum[k] = sumv[k] = acc[k] = 0.0;
  if (FUSED) {
    const double* __restrict__ C = C64 + s0 * g.Np;
    const double* __restrict__ CY = CY64 + s0 * g.Np;
#pragma unroll 8
    for (int j = 0; j < (int)g.N; ++j) {
      const Vals<T, R> w = buf_load_r<T, R>(jr, voff, j * pitch);
#pragma unroll
      for (int k = 0; k < R; ++k) {
        D[k] += (double)w.v[k] * C[j];
        if (TAU) V[k] += (double)w.v[k] * CY[j];
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      D[k] = Dc[(s0 / g.kc - g.row0) * g.Np + i + k];
      if (TAU) V[k] = Vc[(s0 / g.kc - g.row0) * g.Np + i + k];
    }
  }
  int t = 0, wo = 0;  // bin, and offset of its row in W
  auto emit = [&]() {
    if (PART && t < skip) return;
    Vals<T, R> w;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const double lam = exp_f64(D[k]);
      sum[k] += lam;
      if (TAU) sumv[k] += lam * V[k];
      w.v[k] = (T)lam;
    }
    if (STORE) {
      buf_store_r<T, R>(w, wr, voff, wo);
      wo += pitch;
    }
  };
  auto step = [&]() {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (TAU) V[k] = ag * (V[k] + g.ctau * D[k]);
      D[k] = ag * D[k] + acc[k];
      acc[k] = 0.0;
    }
    ++t;
    emit();
  };
  if (tend > skip) {
    emit();
    const int e0 = off[s0];
    const int64_t s1 = (t0 + g.seg + 63) >> 6;
    const int e1 = off[s1 < g.NS ? s1 : g.NS];
    const uint32_t base = (uint32_t)(s0 * 64) & 0x7fffu;
    auto row = [&](uint32_t q) { return buf_load_r<T, R>(jr, voff, (int)(q & 0xffffu) * pitch); };
    const uint32_t last = ENT_FIRST | ((((uint32_t)(tend - 1) + base) & 0x7fffu) << 16);
    uint32_t ec[FB8], en[FB8];
    Vals<T, R> rn[FB8];
    if (e0 < e1) {
#pragma unroll
      for (int q = 0; q < FB8; ++q) ec[q] = ent[e0 + q];
#pragma unroll
      for (int q = 0; q < FB8; ++q) rn[q] = row(ec[q]);
#pragma unroll
      for (int q = 0; q < FB8; ++q) en[q] = ent[e0 + FB8 + q];
    }
    for (int e = e0; e < e1; e += FB8) {
      if (e + FB8 > e1) {
        // past the segment's entries: a first entry of its last bin, whose
        // row is added after the last step
#pragma unroll
        for (int q = 0; q < FB8; ++q) ec[q] = e + q < e1 ? ec[q] : last;
      }
#pragma unroll
      for (int q = 0; q < FB8; ++q) {
        if (ec[q] & ENT_FIRST) {
          const int b = ent_bin(ec[q], base), to = b < tend - 1 ? b : tend - 1;
          while (t < to) step();
        }
#pragma unroll
        for (int k = 0; k < R; ++k) acc[k] += (double)rn[q].v[k];
        rn[q] = row(en[q]);
      }
#pragma unroll
      for (int q = 0; q < FB8; ++q) ec[q] = en[q];
#pragma unroll
      for (int q = 0; q < FB8; ++q) en[q] = ent[e + 2 * FB8 + q];
    }
    while (t < tend - 1) step();
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    rowpart[(g.seg0 + sg) * g.Np + i + k] = sum[k];
    if (TAU) rowpartV[(g.seg0 + sg) * g.Np + i + k] = sumv[k];
  }
}

// ------------------------------------------------------------------ forward, event grid
// The interval integrals F, H of a slot by the staged expansion (evfun.h).  A
// wave forms the coefficients of 32 slots at a time, a slot a lane, in LDS; a
// step then reads them at one address and takes an exponential and two Horner
// sums a piece.  The expansion as written out per slot and lane took three
// times the multiplications, and the closed forms past its bound, which some
// lane of a wave takes at nearly every slot of a small network, as a call 247
// registers.
using glmr_ev::EVC;
using glmr_ev::EVE;
constexpr int EVS = 32;  // slots in LDS

template <typename T, bool STORE, bool FUSED, bool PART>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_rec_fwd_ev(
    const uint32_t* __restrict__ ent, const int32_t* __restrict__ off, const T* __restrict__ Jt,
    const double* __restrict__ Dc, const double* __restrict__ C64, const double* __restrict__ edec,
    const double* __restrict__ delta, T* __restrict__ W, double* __restrict__ rowpart, RecFDims g) {
  __shared__ __align__(16) double coef[4][EVS * EVC];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nib = (uint32_t)((g.N + 63) / 64);
  const int i = (int)(blockIdx.x % nib) * 64 + lane;
  const int64_t sg = (int64_t)(blockIdx.x / nib) * 4 + wave;
  if (sg >= g.n_seg) return;
  const int64_t t0 = g.t0 + sg * g.seg;
  const int64_t s0 = t0 >> 6;
  const int skip = PART ? (int)(t0 & 63) : 0;
  const int64_t left = g.B - s0 * 64;
  const int tend = (int)(left < skip + g.seg ? left : skip + g.seg);
  const int pitch = (int)(g.Np * (int64_t)sizeof(T)), voff = i * (int)sizeof(T);
  const __amdgpu_buffer_rsrc_t jr =
      __builtin_amdgcn_make_buffer_rsrc((void*)Jt, (short)0, (int)(g.Np * pitch), 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(STORE ? W + (t0 - g.tw) * g.Np : nullptr), (short)0, STORE ? (int)(g.seg * pitch) : 0, 0x00020000);
  double D = 0.0;
  if (FUSED) {
    const double* __restrict__ C = C64 + s0 * g.Np;
#pragma unroll 8
    for (int j = 0; j < (int)g.N; ++j) D += (double)buf_load<T>(jr, voff, j * pitch) * C[j];
  } else {
    D = Dc[(s0 / g.kc - g.row0) * g.Np + i];
  }
  double sum = 0.0;
  if (tend > skip) {
    double* mine = coef[wave];
    int e = off[s0];
    const int64_t s1 = (t0 + g.seg + 63) >> 6;
    const int e1 = off[s1 < g.NS ? s1 : g.NS];
    const uint32_t base = (uint32_t)(s0 * 64) & 0x7fffu;
    // about one entry a slot: 64 entries a load, one a lane, and four rows
    // ahead in a shift register
    auto row = [&](uint32_t q) { return buf_load<T>(jr, voff, (int)(q & 0xffffu) * pitch); };
    uint32_t ev = ent[e + lane], evn = ent[e + 64 + lane];
    int at = 0;  // of entry e in ev
    auto entry = [&](int k) {
      return (uint32_t)(k < 64 ? __builtin_amdgcn_readlane((int)ev, k) : __builtin_amdgcn_readlane((int)evn, k - 64));
    };
    uint32_t q0 = entry(0), q1 = entry(1), q2 = entry(2), q3 = entry(3);
    T r0 = row(q0), r1 = row(q1), r2 = row(q2), r3 = row(q3);
    int wo = 0;
    for (int t = 0;;) {
      if ((t & (EVS - 1)) == 0) {  // a wave's LDS operations are in order: no barrier
        __builtin_amdgcn_wave_barrier();
        if (lane < EVS) glmr_ev::stage_pieces(delta[s0 * 64 + t + lane], edec[s0 * 64 + t + lane], mine + lane * EVC);
        __builtin_amdgcn_wave_barrier();
      }
      const double dec = mine[(t & (EVS - 1)) * EVC + EVE + 5];
      if (!PART || t >= skip) {
        const double2* src = (const double2*)(mine + (t & (EVS - 1)) * EVC);
        double c[EVE + 6];
#pragma unroll
        for (int v = 0; v < (EVE + 6) / 2; ++v) {
          const double2 x = src[v];
          c[2 * v] = x.x;
          c[2 * v + 1] = x.y;
        }
        double F, H;
        const int p = __builtin_amdgcn_readfirstlane((int)c[EVE + 3]);
        const bool out = !glmr_ev::interval_pieces(c, p, D, &F, &H);
        if (out) glmr_ev::interval_any(D, c[EVE + 4], &F, &H);
        sum += F;
        if (STORE) {
          buf_store<T>((T)H, wr, voff, wo);
          wo += pitch;
        }
      }
      if (t >= tend - 1) break;
      double acc = 0.0;
      while (e < e1 && ent_bin(q0, base) <= t) {
        acc += (double)r0;
        q0 = q1; q1 = q2; q2 = q3;
        r0 = r1; r1 = r2; r2 = r3;
        q3 = entry(at + 4);
        r3 = row(q3);
        ++e;
        if (++at == 64) {
          ev = evn;
          evn = ent[e + 64 + lane];
          at = 0;
        }
      }
      D = fma(dec, D, acc);
      ++t;
    }
  }
  rowpart[(g.seg0 + sg) * g.Np + i] = sum;
}

// Dc[r][i] = sum_j C[(row0 + r) kc][j] J[i][j]: 32 x 64 tiles on the FP64 MFMA,
// KS columns j a step through LDS.  The tiles are few (592 at N = 1000 and
// 1.2e6 bins, 592 at N = 500 and 3e5) and the busiest CU sets the time: with 64
// x 64 tiles, two to some CUs and one to the others, and 16 columns a step, the
// load of a step took longer than its MFMAs and the kernel 98 and 60 us
// instead of 62 and 44.
constexpr int KS = 32;
template <typename JT>
__global__ __launch_bounds__(256) void k_carry_gemm(const double* __restrict__ C, const JT* __restrict__ Jt,
                                                    double* __restrict__ out, int64_t rows, int64_t row0, int64_t kc,
                                                    int64_t NS, int64_t Np) {
  __shared__ double As[32][KS + 2], Bs[KS][66];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nt = Np / 64;
  const int64_t i0 = (int64_t)(blockIdx.x % nt) * 64, r0 = (int64_t)(blockIdx.x / nt) * 32;
  const int wr = wave & 1, wc = wave >> 1;  // a wave's 16 rows and 32 columns
  f64x4 acc[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
  double an[KS / 8], bn[KS / 4];
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < KS / 8; ++q) {
      const int r = tid / KS + 256 / KS * q, c = tid % KS;
      const int64_t s = (row0 + r0 + r) * kc;
      an[q] = (r0 + r < rows && s < NS) ? C[s * Np + k0 + c] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < KS / 4; ++q) bn[q] = (double)Jt[(k0 + (tid >> 6) + 4 * q) * Np + i0 + lane];
  };
  fetch(0);
  for (int64_t k0 = 0; k0 < Np; k0 += KS) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KS / 8; ++q) As[tid / KS + 256 / KS * q][tid % KS] = an[q];
#pragma unroll
    for (int q = 0; q < KS / 4; ++q) Bs[(tid >> 6) + 4 * q][lane] = bn[q];
    __syncthreads();
    if (k0 + KS < Np) fetch(k0 + KS);
#pragma unroll
    for (int k = 0; k < KS; k += 4) {
      const double a = As[wr * 16 + (lane & 15)][k + (lane >> 4)];
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Bs[k + (lane >> 4)][wc * 32 + b * 16 + (lane & 15)], acc[b], 0,
                                                      0, 0);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = r0 + wr * 16 + (lane >> 4) + 4 * r;
      if (row < rows) out[row * Np + i0 + wc * 32 + b * 16 + (lane & 15)] = acc[b][r];
    }
}

// J^T in the mode's type, the weights as used, e^mu
template <typename JT>
__global__ __launch_bounds__(256) void k_prepare_t(int N, int64_t Np, const double* J, int64_t ld, const double* mu,
                                                   JT* Jt, double* Jr, double* rowscale, double* J64, double* mu64) {
  __shared__ JT t[32][33];
  const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t i = i0 + ty + 8 * q, j = j0 + tx;
    const double x = (i < N && j < N) ? J[i * ld + j] : 0.0;
    const JT v = (JT)x;
    if (J64 && i < N && j < N) J64[i * Np + j] = x;
    Jr[i * Np + j] = (double)v;
    t[ty + 8 * q][tx] = v;
    if (j == 0) {
      const double m = i < N ? mu[i] : 0.0;
      rowscale[i] = (i < N) ? exp(m) : 0.0;
      if (J64 && i < N) mu64[i] = m;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) Jt[(j0 + ty + 8 * q) * Np + i0 + tx] = t[tx][ty + 8 * q];
}

template <typename WT, bool EV>
hipError_t rec_gather(const RecGArgs& a, hipStream_t st) {
  const int jb = gather_jb(a.Np);
  const int64_t blocks = ((a.N + GI - 1) / GI) * ((a.Np + GG * jb - 1) / (GG * jb));
  switch (jb) {
    case 1: return run_gather(k_rec_gather<WT, EV, 1>, a, blocks, a.n_splits, st);
    case 2: return run_gather(k_rec_gather<WT, EV, 2>, a, blocks, a.n_splits, st);
    case 4: return run_gather(k_rec_gather<WT, EV, 4>, a, blocks, a.n_splits, st);
    default: return run_gather(k_rec_gather<WT, EV, 8>, a, blocks, a.n_splits, st);
  }
}

template <typename T, bool TAU, bool STORE, bool FUSED, bool PART>
hipError_t rec_fwd_run(const RecFArgs& a, hipStream_t st) {
  const RecFDims& g = a.g;
  const int64_t nib = (g.N + 63) / 64, segs = (g.n_seg + 3) / 4;
  const unsigned blocks = (unsigned)(nib * segs);
  // Two rows a lane where J is in FP64, whose loads bound the kernel (from the
  // L2, 8 bytes a lane; likelihood alone at N = 1000, 4e5 bins: 1431 us with
  // one row, 990 with two; in FP32 873 and 867, the conversions bound it), and
  // where at most one block of 64 rows in eight is padding.  Segments shorter
  // than a subtile are those of recordings with too few waves.
  if constexpr (sizeof(T) == 8 && !FUSED && !PART)
    if (!a.edec && (nib % 2 == 0 || nib >= 7)) {
      hipLaunchKernelGGL((k_rec_fwd<T, 2, TAU, STORE, false, false>), dim3((unsigned)((nib + 1) / 2 * segs)), dim3(256),
                         0, st, a.ent1, a.off1, (const T*)a.Jt, a.Dc, a.Vc, a.C64, a.CY64, (T*)a.W, a.rowpart,
                         a.rowpartV, g);
      return hipGetLastError();
    }
  if (a.edec)
    hipLaunchKernelGGL((k_rec_fwd_ev<T, STORE, FUSED, PART>), dim3(blocks), dim3(256), 0, st, a.ent1, a.off1,
                       (const T*)a.Jt, a.Dc, a.C64, a.edec, a.delta, (T*)a.W, a.rowpart, g);
  else
    hipLaunchKernelGGL((k_rec_fwd<T, 1, TAU, STORE, FUSED, PART>), dim3(blocks), dim3(256), 0, st, a.ent1, a.off1,
                       (const T*)a.Jt, a.Dc, a.Vc, a.C64, a.CY64, (T*)a.W, a.rowpart, a.rowpartV, g);
  return hipGetLastError();
}

template <typename T, bool TAU, bool STORE>
hipError_t rec_fwd(const RecFArgs& a, hipStream_t st) {
  const bool part = a.g.seg < 64;
  if (a.fused)
    return part ? rec_fwd_run<T, TAU, STORE, true, true>(a, st) : rec_fwd_run<T, TAU, STORE, true, false>(a, st);
  return part ? rec_fwd_run<T, TAU, STORE, false, true>(a, st) : rec_fwd_run<T, TAU, STORE, false, false>(a, st);
}

template <typename T>
hipError_t carry_gemm(const RecFArgs& a, const double* C, double* out, hipStream_t st) {
  const int64_t blocks = (a.g.Np / 64) * ((a.rows + 31) / 32);
  hipLaunchKernelGGL(k_carry_gemm<T>, dim3((unsigned)blocks), dim3(256), 0, st, C, (const T*)a.Jt, out, a.rows,
                     a.g.row0, a.g.kc, a.g.NS, a.g.Np);
  return hipGetLastError();
}

template <typename T>
hipError_t rec_forward(const RecFArgs& a, hipStream_t st) {
  const bool tau = a.rowpartV != nullptr, store = a.W != nullptr;
  if (!a.fused) {
    hipError_t e = carry_gemm<T>(a, a.C64, a.Dc, st);
    if (e == hipSuccess && tau) e = carry_gemm<T>(a, a.CY64, a.Vc, st);
    if (e != hipSuccess) return e;
  }
  if (tau) return store ? rec_fwd<T, true, true>(a, st) : rec_fwd<T, true, false>(a, st);
  return store ? rec_fwd<T, false, true>(a, st) : rec_fwd<T, false, false>(a, st);
}

}  // namespace

hipError_t launch_rec_forward(int prec, const RecFArgs& a, hipStream_t st) {
  return prec == PREC_F64 ? rec_forward<double>(a, st) : rec_forward<float>(a, st);
}

hipError_t launch_rec_gather(int prec, const RecGArgs& a, hipStream_t st) {
  if (prec == PREC_F64) return a.ev.edec ? rec_gather<double, true>(a, st) : rec_gather<double, false>(a, st);
  return a.ev.edec ? rec_gather<float, true>(a, st) : rec_gather<float, false>(a, st);
}

hipError_t launch_rec_reduce(const RecGArgs& a, int first, hipStream_t st) {
  hipLaunchKernelGGL(k_rec_reduce, dim3((unsigned)(a.Np / 32), (unsigned)(a.Np / 8)), dim3(256), 0, st, a, first);
  return hipGetLastError();
}

hipError_t launch_rec_finish(const RecGArgs& a, const AssembleArgs& s, int first, int grad, hipStream_t st) {
  const int64_t nb = s.Np / 32;
  hipLaunchKernelGGL(k_rec_finish, dim3((unsigned)(s.Np / RROWS + (grad ? nb * (s.Np / 8) : 0))), dim3(1024), 0, st, a, s, first);
  return hipGetLastError();
}

hipError_t launch_prepare_t(int prec, int N, int64_t Np, const double* J, int64_t ld, const double* mu, void* Jt,
                            double* Jr, double* rowscale, double* J64, double* mu64, hipStream_t st) {
  const unsigned nb = (unsigned)(Np / 32);
  if (prec == PREC_F64)
    hipLaunchKernelGGL(k_prepare_t<double>, dim3(nb, nb), dim3(256), 0, st, N, Np, J, ld, mu, (double*)Jt, Jr, rowscale,
                       J64, mu64);
  else
    hipLaunchKernelGGL(k_prepare_t<float>, dim3(nb, nb), dim3(256), 0, st, N, Np, J, ld, mu, (float*)Jt, Jr, rowscale,
                       J64, mu64);
  return hipGetLastError();
}
