// The edge list of gsn_export: the half-edges (u, v) with u < v of the compact adjacency, in
// row order, which is ascending (u, v) order (rows are ascending by neighbour, so a row's
// part with v > u is its tail).
//
// Two launches: every workgroup counts its kBlock rows, then writes them from the sum of the
// counts before it, as three rows of the list (u, v, age).  Listing the edges on the host took
// a copy of the whole adjacency and a pass over it: a read-out of 200,000 units and 230,000
// edges took 2.3 ms, and 0.5 ms this way, nearly all of it the copies into the caller's memory.
#include "gsn_internal.h"

namespace gsn {
namespace {

// first entry of row [r0, r1) above u
__device__ __forceinline__ int32_t upper_part(const int32_t* __restrict__ col, int32_t r0,
                                              int32_t r1, int32_t u) {
  int32_t k = r0;
  while (k < r1) {
    // four entries per round of loads (past the end the last one repeats)
    int32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = col[min(k + i, r1 - 1)];
    int32_t low = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) low += k + i < r1 && c[i] <= u;
    k += low;
    if (low < 4) break;
  }
  return k;
}

__global__ __launch_bounds__(kBlock) void ex_count(int32_t n, const int32_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col,
                                                   int32_t* __restrict__ bsum) {
  __shared__ int32_t wt[kBlock / 64];
  const int32_t u = blockIdx.x * kBlock + threadIdx.x;
  int32_t c = 0;
  if (u < n) {
    const int32_t r0 = rp[u], r1 = rp[u + 1];
    c = r1 - upper_part(col, r0, r1, u);
  }
  c = block_sum(c, wt);
  if (threadIdx.x == 0) bsum[blockIdx.x] = c;
}

// eu, ev, ea: the list's rows, cap entries each (a list of more, which only a corrupted
// adjacency could hold, is cut)
__global__ __launch_bounds__(kBlock) void ex_write(int32_t n, const int32_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col,
                                                   const int32_t* __restrict__ age,
                                                   const int32_t* __restrict__ bsum, int32_t nb,
                                                   int fold, int32_t cap,
                                                   int32_t* __restrict__ eu,
                                                   int32_t* __restrict__ ev,
                                                   int32_t* __restrict__ ea) {
  __shared__ int32_t wt[kBlock / 64];
  __shared__ int32_t red[2 * kBlock / 64];
  const int32_t u = blockIdx.x * kBlock + threadIdx.x;
  int32_t k0 = 0, r1 = 0;
  if (u < n) {
    r1 = rp[u + 1];
    k0 = upper_part(col, rp[u], r1, u);
  }
  int32_t before, total;
  if (fold) fold_offsets(bsum, nb, red, &before, &total);
  else before = bsum[blockIdx.x];
  const int32_t c = r1 - k0;
  int32_t o = before + block_inclusive_scan(c, wt) - c;
  for (int32_t k = k0; k < r1 && o < cap; ++k, ++o) {
    eu[o] = u;
    ev[o] = col[k];
    ea[o] = age[k];
  }
}

}  // namespace

hipError_t launch_export_edges(const DevState& s, int cur, int32_t n, int32_t edges,
                               hipStream_t st) {
  const int nb = (n + kBlock - 1) / kBlock;
  if (nb == 0 || edges <= 0) return hipSuccess;
  const int nxt = cur ^ 1;
  ex_count<<<nb, kBlock, 0, st>>>(n, s.rp[cur], s.col[cur], s.bsum);
  if (nb > kFoldBlocks) {
    const hipError_t e = launch_scan_blocks(s.bsum, nb, INT64_MAX, nullptr, s.status, -1, st);
    if (e != hipSuccess) return e;
  }
  ex_write<<<nb, kBlock, 0, st>>>(n, s.rp[cur], s.col[cur], s.age[cur], s.bsum, nb,
                                  nb <= kFoldBlocks ? 1 : 0, edges, s.col[nxt],
                                  s.col[nxt] + edges, s.age[nxt]);
  return hipGetLastError();
}

}  // namespace gsn
