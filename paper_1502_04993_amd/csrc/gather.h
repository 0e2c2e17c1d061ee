// Sums over a raster's spikes of one of a window's quantities (gfx950): a tile
// of 1024 bins x 16 columns (FP64, 128 KB of LDS) holds the quantity, and every
// neuron adds up the tile's rows at its own spikes in registers, from the
// window-major spike lists (spikes.hip).  Used by the spike term (columns of
// the trace) and by kernel G of the recurrence (rows of R, recur.hip).
#pragma once

#include "common.h"

namespace glmr_gather {

constexpr int GW = GLMR_GW;          // bins per window
constexpr int GI = 16;               // tile columns
constexpr int GNT = 1024;            // threads of the gather workgroups
// Lanes of a group, two columns each, so that a lane reads 16 bytes of a row
// at a time (16 lanes of one column, 8 bytes: kernel G 3.4 against 3.1 ms and
// the spike term 2.55 against 2.45 ms at N = 1000, 1.2e6 bins, although the
// longest of eight lists is longer than that of four).
constexpr int GL = 8;
constexpr int GG = GNT / GL;         // groups
constexpr int TILE = (GW + 1) * GI;  // doubles; the last row is zero
constexpr int CAP = 3070;            // groups of four entries staged in LDS
constexpr int SCAN = 34 * GI;        // doubles of kernel G's scan
constexpr int ENTRIES = TILE + SCAN; // where the staged entries start (in 8 bytes)
constexpr size_t GATHER_LDS = (size_t)(ENTRIES + CAP + 2) * 8;
static_assert(GATHER_LDS <= 160 * 1024, "tile, scan and entries fit in a CU's LDS");

// value of v in lane K of the 8-lane group
template <int K>
__device__ __forceinline__ int group_bcast(int v) {
  const int u = __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xf, 0x3, false);  // row_newbcast, lower half of the rows
  return __builtin_amdgcn_update_dpp(u, v, 0x150 + 8 + K, 0xf, 0xc, false);     // upper half
}

// A window's share of the lists for the JB neurons of a group (from idx in
// end2): where they begin, and in lane k the end of neuron k's.
struct Ends {
  int begin, end;
};
template <int JB>
__device__ __forceinline__ Ends load_ends(const int32_t* __restrict__ end2, int64_t idx, int il) {
  return Ends{end2[idx - 1], end2[idx + (il < JB ? il : 0)]};
}

// acc[k] += the tile's rows at the entries of the group's neuron k: its 8
// lanes hold 16 tile columns and take one neuron after another; the lists of
// consecutive neurons follow each other, so the next four entries are always
// being loaded.
struct Cols {
  double a, b;  // a lane's two columns
};
// LDS byte address 8 u + base of the low or high half u of e, in one instruction
__device__ __forceinline__ uint32_t addr_lo(uint32_t e, uint32_t base) {
  uint32_t a;
  asm("v_mad_u32_u16 %0, %1, 8, %2" : "=v"(a) : "v"(e), "v"(base));
  return a;
}
__device__ __forceinline__ uint32_t addr_hi(uint32_t e, uint32_t base) {
  uint32_t a;
  asm("v_mad_u32_u16 %0, %1, 8, %2 op_sel:[1,0,0,0]" : "=v"(a) : "v"(e), "v"(base));
  return a;
}
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const f64x2 lds_f64x2;
typedef __attribute__((address_space(3))) const u32x2 lds_u32x2;
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// col: byte address of the lane's columns; p, lim: of entries
template <int K, int JB>
__device__ __forceinline__ void walk(Cols (&acc)[JB], uint32_t col, uint32_t& p, u32x2& nx, uint32_t ends,
                                     uint32_t lim) {
  if constexpr (K < JB) {
    const uint32_t e0 = (uint32_t)group_bcast<K>((int)ends), end = e0 < lim ? e0 : lim;
    while (p < end) {
      const u32x2 e = nx;
      p += 8;
      nx = *(lds_u32x2*)p;
      const f64x2 v0 = *(lds_f64x2*)addr_lo(e[0], col), v1 = *(lds_f64x2*)addr_hi(e[0], col);
      const f64x2 v2 = *(lds_f64x2*)addr_lo(e[1], col), v3 = *(lds_f64x2*)addr_hi(e[1], col);
      acc[K].a += (v0[0] + v1[0]) + (v2[0] + v3[0]);
      acc[K].b += (v0[1] + v1[1]) + (v2[1] + v3[1]);
    }
    walk<K + 1, JB>(acc, col, p, nx, ends, lim);
  }
}

// The window's entries of a workgroup's neurons, groups base .. base + n - 1,
// pass through LDS in pieces of CAP (one piece for three groups a neuron and
// window at 1024 neurons, about 10 spikes a second in 1 ms bins).  The first piece is copied with the
// tile, before its barrier; every thread of the workgroup calls both.
__device__ __forceinline__ void stage_entries(uint2* es, const uint2* __restrict__ ent, int base, int n) {
  n = n < CAP ? n : CAP;
  for (int q = threadIdx.x; q <= n; q += GNT) es[q] = ent[base + q];  // one past the end is loaded ahead
}

// Address of the end of a neuron's list in the piece staged at e8; end: in
// groups from the piece's first.  A list that ended in an earlier piece ends
// here at the piece's start (its end, below zero, must not wrap around).
__host__ __device__ __forceinline__ uint32_t piece_end(uint32_t e8, int end) {
  return e8 + 8 * (uint32_t)(end < 0 ? 0 : end < CAP ? end : CAP);
}

template <int JB>
__device__ __forceinline__ void gather_lists(Cols (&acc)[JB], double* lds, const uint2* __restrict__ ent, int base,
                                             int n, Ends e, int il, bool rows) {
  uint2* es = (uint2*)(lds + ENTRIES);
  const uint32_t l0 = lds_addr(lds), col = l0 + 16 * il, e8 = l0 + 8 * ENTRIES;
  int p = e.begin - base;
#pragma unroll 1
  for (int q0 = 0; q0 < n; q0 += CAP) {
    if (q0 > 0) {
      __syncthreads();
      stage_entries(es, ent, base + q0, n - q0);
      __syncthreads();
    }
    if (rows && p >= q0 && p < q0 + CAP) {  // a group that is done stays where its lists ended
      uint32_t pl = e8 + 8 * (p - q0);
      u32x2 nx = *(lds_u32x2*)pl;
      walk<0, JB>(acc, col, pl, nx, piece_end(e8, e.end - base - q0), e8 + 8 * CAP);
      p = q0 + (int)(pl - e8) / 8;
    }
  }
}

// neurons per group: the smallest that covers them, at most 8 (16 FP64 sums a
// lane; more neurons take further blocks of 1024)
inline int gather_jb(int64_t Np) {
  int jb = 1;
  while (jb < 8 && GG * jb < Np) jb *= 2;
  return jb;
}

// workgroups of one time split over `cols` tile columns
inline int64_t blocks_of(int64_t cols, int64_t Np) {
  const int jb = gather_jb(Np);
  return ((cols + GI - 1) / GI) * ((Np + GG * jb - 1) / (GG * jb));
}

template <typename K, typename A>
hipError_t run_gather(K kern, const A& a, int64_t blocks, int splits, hipStream_t st) {
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)GATHER_LDS);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)splits), dim3(GNT), GATHER_LDS, st, a);
  return hipGetLastError();
}

}  // namespace glmr_gather
