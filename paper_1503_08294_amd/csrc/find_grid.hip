// Indexed find winners: the hash index of the paper's "Indexed" implementation (Sec. 3.1)
// applied to every signal of the batch.  A grid of cubes of side h over an axis-parallel
// box holds the units, counting-sorted by cube every call (units move every iteration); the
// winner and the second of a signal are searched among the units of its cube and the 26
// neighbours (a group of 32 lanes per signal, the lanes' top-2 keys
// merged), and signals whose 27 cubes hold fewer than two units get the
// exhaustive search.  Results equal the oracle's indexed search bit for bit: the same cell
// function, the same direct-form distance, the same (d, index) order.  In exact mode the
// 27-cube result is kept only where it is certified to be the exhaustive one.
//
// The build waits on atomics and on the number of its launches, the query on dependent loads.
// The count's returned rank places a unit, so the scatter makes no atomic; the scan takes two
// launches; and a query deals the units of the nine rows of three cubes (consecutive in the
// sorted order) out to its 32 lanes, where a lane per cube left most lanes idle behind the
// fullest cube.  At 200,000 units, 16,384 signals and 163,000 cubes (a side of 3.3 spacings): count
// 12.8 -> 13.2 us, scan 11.1 -> 8.3, scatter 16.3 -> 5.5, query 35.7 -> 9.8, the call 83 -> 44.
#include "gsn_internal.h"

namespace gsn {
namespace {

constexpr int kGroupLanes = 32;            // lanes per signal, which share the 27 cubes' units
constexpr int kQueryBlock = 256;           // 8 signals per workgroup
constexpr int kFallbackBlocks = 256;
constexpr int kScanPart = 4 * kBlock;      // cubes per workgroup of the scan
constexpr int kRankBits = 8;               // of a unit's rank in its cube, beside its cube
constexpr int32_t kRankMax = (1 << kRankBits) - 1;   // ranks from here on come from a cursor
static_assert(GSN_MAX_GRID_CELLS <= (1 << (31 - kRankBits + 1)), "cube and rank in 32 bits");

inline int blocks(int64_t n) { return static_cast<int>((n + kBlock - 1) / kBlock); }

__device__ __forceinline__ int32_t grid_axis(float p, float lo, float inv_h, int32_t dim) {
  const float t = (p - lo) * inv_h;
  if (!(t >= 0.0f)) return 0;                              // below the box (and NaN)
  if (t >= static_cast<float>(dim)) return dim - 1;        // beyond it
  const int32_t c = static_cast<int32_t>(floorf(t));
  return c < dim ? c : dim - 1;
}

struct GridArgs {
  float lo0, lo1, lo2, inv_h;
  int32_t d0, d1, d2;
  int exact;
};

__device__ __forceinline__ void cell_of(const GridArgs& g, float x, float y, float z,
                                        int32_t* c) {
  c[0] = grid_axis(x, g.lo0, g.inv_h, g.d0);
  c[1] = grid_axis(y, g.lo1, g.inv_h, g.d1);
  c[2] = grid_axis(z, g.lo2, g.inv_h, g.d2);
}

__device__ __forceinline__ float direct_d(float sx, float sy, float sz, float wx, float wy,
                                          float wz) {
  const float dx = sx - wx, dy = sy - wy, dz = sz - wz;
  return (dx * dx + dy * dy) + dz * dz;
}

// Certification of a signal's 27-cube result (exact mode).  With t = fl(fl(p - lo) inv_h)
// and x = (p - lo) inv_h exactly, t = x (1 + eta), |eta| <= 2u + u^2.  A unit in a cube two
// or more above the signal's on axis a has t_w >= c + 2, so x_w >= (c + 2) / (1 + |eta|);
// the signal has t_s < c + 1 (or t_s < 0), so x_s <= max(t_s, 0) / (1 - |eta|); below
// likewise with x_w < (c - 1) / (1 - |eta|) and x_s >= t_s / (1 + |eta|).  Every unit outside
// the 27 cubes is outside on some axis, so its true distance is at least r = the least of
// these gaps divided by inv_h (gaps computed in binary64 with a relative margin of 3e-7 >
// 2.01 u per factor and an absolute one for subnormal differences).  Its computed binary32
// distance is at least (1 - 5u) times the true one, so if d2 < r^2 (1 - 4e-7) every outside
// unit's computed distance exceeds d2 and the 27-cube top-2 is the exhaustive one.
__device__ bool certified(const GridArgs& g, float sx, float sy, float sz, const int32_t* c,
                          float d2) {
  const double up = 1.0 + 3e-7, dn = 1.0 - 3e-7;
  const float p[3] = {sx, sy, sz};
  const float lo[3] = {g.lo0, g.lo1, g.lo2};
  const int32_t dims[3] = {g.d0, g.d1, g.d2};
  double gap = __builtin_huge_val();  // in cells
  for (int a = 0; a < 3; ++a) {
    const double t = static_cast<double>((p[a] - lo[a]) * g.inv_h);
    if (c[a] + 2 <= dims[a] - 1) gap = fmin(gap, (c[a] + 2) * dn - fmax(t, 0.0) * up);
    if (c[a] - 2 >= 0) gap = fmin(gap, t * dn - (c[a] - 1) * up);
  }
  if (gap == __builtin_huge_val()) return d2 < __builtin_huge_valf();  // the cubes hold all
  gap -= 1e-30;
  if (!(gap > 0.0)) return false;
  const double r = gap / static_cast<double>(g.inv_h) * (1.0 - 1e-12);
  return static_cast<double>(d2) < r * r * (1.0 - 4e-7);
}

__device__ __forceinline__ void top2_insert(unsigned long long k, unsigned long long& k1,
                                            unsigned long long& k2) {
  if (k < k1) {
    k2 = k1;
    k1 = k;
  } else if (k < k2) {
    k2 = k;
  }
}

__global__ void gx_clear(int32_t* __restrict__ cnt, int32_t cells, int32_t* __restrict__ nfb) {
  const int32_t stride = gridDim.x * kBlock;
  for (int32_t c = blockIdx.x * kBlock + threadIdx.x; c < cells; c += stride) cnt[c] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *nfb = 0;
}

__global__ void gx_count(int32_t n, const float* __restrict__ x, const float* __restrict__ y,
                         const float* __restrict__ z, GridArgs g, int32_t* __restrict__ ucell,
                         int32_t* __restrict__ cnt) {
  const int32_t u = blockIdx.x * kBlock + threadIdx.x;
  if (u >= n) return;
  int32_t c[3];
  cell_of(g, x[u], y[u], z[u], c);
  const int32_t lin = (c[2] * g.d1 + c[1]) * g.d0 + c[0];
  // the count's old value is the unit's rank in its cube (the order inside a cube is immaterial)
  const int32_t rank = min(atomicAdd(&cnt[lin], 1), kRankMax);
  ucell[u] = static_cast<int32_t>((static_cast<uint32_t>(lin) << kRankBits) |
                                  static_cast<uint32_t>(rank));
}

__device__ __forceinline__ int4 load_counts(const int32_t* __restrict__ cnt, int32_t c,
                                            int32_t cells) {
  if (c + 3 < cells) return *reinterpret_cast<const int4*>(cnt + c);
  return make_int4(c < cells ? cnt[c] : 0, c + 1 < cells ? cnt[c + 1] : 0,
                   c + 2 < cells ? cnt[c + 2] : 0, 0);
}

__global__ __launch_bounds__(kBlock) void gx_bsum(int32_t cells, const int32_t* __restrict__ cnt,
                                                  int32_t* __restrict__ bsum) {
  __shared__ int32_t wt[kBlock / 64];
  const int32_t c = (blockIdx.x * kBlock + threadIdx.x) * 4;
  const int4 v = load_counts(cnt, c, cells);
  const int32_t t = block_sum(v.x + v.y + v.z + v.w, wt);
  if (threadIdx.x == 0) bsum[blockIdx.x] = t;
}

// start[c] = units in the cubes before c; cnt[c] becomes the cursor of the units of rank
// kRankMax and up.  With fold, each workgroup sums the parts before its own itself.
__global__ __launch_bounds__(kBlock) void gx_start(int32_t cells, int32_t n,
                                                   int32_t* __restrict__ cnt,
                                                   const int32_t* __restrict__ bsum, int32_t nb,
                                                   int fold, int32_t* __restrict__ start) {
  __shared__ int32_t red[2 * kBlock / 64];
  __shared__ int32_t wt[kBlock / 64];
  const int32_t c = (blockIdx.x * kBlock + threadIdx.x) * 4;
  const int4 v = load_counts(cnt, c, cells);
  int32_t before, total;
  if (fold) fold_offsets(bsum, nb, red, &before, &total);
  else before = bsum[blockIdx.x];
  const int32_t sum = v.x + v.y + v.z + v.w;
  const int32_t o0 = before + block_inclusive_scan(sum, wt) - sum;
  const int32_t o[4] = {o0, o0 + v.x, o0 + v.x + v.y, o0 + v.x + v.y + v.z};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (c + k < cells) {
      start[c + k] = o[k];
      cnt[c + k] = o[k] + kRankMax;
    }
  if (c == 0) start[cells] = n;
}

__global__ void gx_scatter(int32_t n, const float* __restrict__ x, const float* __restrict__ y,
                           const float* __restrict__ z, const int32_t* __restrict__ ucell,
                           const int32_t* __restrict__ start, int32_t* __restrict__ cursor,
                           float4* __restrict__ sorted) {
  const int32_t u = blockIdx.x * kBlock + threadIdx.x;
  if (u >= n) return;
  const uint32_t w = static_cast<uint32_t>(ucell[u]);
  const int32_t lin = static_cast<int32_t>(w >> kRankBits);
  const int32_t rank = static_cast<int32_t>(w & kRankMax);
  const float4 p = make_float4(x[u], y[u], z[u], __int_as_float(u));
  const int32_t pos = rank < kRankMax ? start[lin] + rank : atomicAdd(&cursor[lin], 1);
  if (pos >= 0 && pos < n) sorted[pos] = p;   // always true when counts match cubes
}

// 32 lanes per signal.  Lane r < 9 reads the bounds of row r: the cubes (cx - 1 .. cx + 1,
// cy + r % 3 - 1, cz + r / 3 - 1), consecutive in the sorted order.  The rows' units are
// numbered through and unit i goes to lane i mod 32.  Fewer than two candidates (or, in exact
// mode, a result that cannot be certified) sends the signal to the fallback list.
__global__ __launch_bounds__(kQueryBlock) void gx_query(
    const float* __restrict__ sig, int32_t m, GridArgs g, const int32_t* __restrict__ start,
    const float4* __restrict__ sorted, int32_t* __restrict__ winner,
    int32_t* __restrict__ second, float* __restrict__ d1, float* __restrict__ d2,
    int32_t* __restrict__ fb_list, int32_t* __restrict__ nfb) {
  constexpr int kRowsOf = 9;
  __shared__ int32_t first[kQueryBlock / kGroupLanes][kRowsOf + 1];   // number of a row's first
  __shared__ int32_t shift[kQueryBlock / kGroupLanes][kRowsOf];       // sorted slot - unit number
  const int32_t gt = blockIdx.x * kQueryBlock + threadIdx.x;
  const int32_t j = gt / kGroupLanes;
  const int q = gt % kGroupLanes, gr = threadIdx.x / kGroupLanes;
  if (j >= m) return;  // whole groups: m groups fill the grid exactly up to the last block
  const float sx = sig[j], sy = sig[m + j], sz = sig[2 * m + j];
  int32_t c[3];
  cell_of(g, sx, sy, sz, c);
  int32_t a = 0, len = 0;
  if (q < kRowsOf) {
    const int32_t cy = c[1] + q % 3 - 1, cz = c[2] + q / 3 - 1;
    if (cy >= 0 && cy < g.d1 && cz >= 0 && cz < g.d2) {
      const int32_t base = (cz * g.d1 + cy) * g.d0;
      a = start[base + max(c[0] - 1, 0)];
      len = start[base + min(c[0] + 1, g.d0 - 1) + 1] - a;
    }
  }
  int32_t inc = len;
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const int32_t v = __shfl_up(inc, o, kGroupLanes);
    if (q >= o) inc += v;
  }
  if (q < kRowsOf) {
    first[gr][q] = inc - len;
    shift[gr][q] = a - (inc - len);
  }
  if (q == kRowsOf) first[gr][kRowsOf] = inc;
  wave_lds_fence();
  int32_t f[kRowsOf + 1];
#pragma unroll
  for (int r = 0; r <= kRowsOf; ++r) f[r] = first[gr][r];
  const int32_t found = f[kRowsOf];
  unsigned long long k1 = kNone, k2 = kNone;
  // two units per step, their loads side by side (past the last one the last repeats)
  for (int32_t i = q; i < found; i += 2 * kGroupLanes) {
    float4 w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int32_t ih = min(i + h * kGroupLanes, found - 1);
      int32_t r = 0;
#pragma unroll
      for (int k = 1; k < kRowsOf; ++k) r += f[k] <= ih;
      w[h] = sorted[ih + shift[gr][r]];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned long long k =
          i + h * kGroupLanes < found
              ? pack_key(direct_d(sx, sy, sz, w[h].x, w[h].y, w[h].z), __float_as_int(w[h].w))
              : kNone;
      k2 = min(k2, max(k1, k));
      k1 = min(k1, k);
    }
  }
  merge_group<kGroupLanes>(k1, k2);
  if (q != 0) return;
  if (found < 2 ||
      (g.exact && !certified(g, sx, sy, sz, c, __uint_as_float(static_cast<uint32_t>(k2 >> 32))))) {
    fb_list[atomicAdd(nfb, 1)] = j;
    return;
  }
  winner[j] = static_cast<int32_t>(k1 & 0xFFFFFFFFu);
  second[j] = static_cast<int32_t>(k2 & 0xFFFFFFFFu);
  d1[j] = __uint_as_float(static_cast<uint32_t>(k1 >> 32));
  d2[j] = __uint_as_float(static_cast<uint32_t>(k2 >> 32));
}

// The exhaustive search for the signals on the fallback list: one workgroup per signal at a
// time (a fixed grid looping over the list), the threads' top-2 keys merged in LDS.
__global__ void gx_fallback(const float* __restrict__ sig, int32_t m, int32_t n,
                            const float* __restrict__ x, const float* __restrict__ y,
                            const float* __restrict__ z, const int32_t* __restrict__ fb_list,
                            const int32_t* __restrict__ nfb, int32_t* __restrict__ winner,
                            int32_t* __restrict__ second, float* __restrict__ d1,
                            float* __restrict__ d2) {
  __shared__ unsigned long long s1[kBlock], s2[kBlock];
  const int32_t count = *nfb;
  for (int32_t e = blockIdx.x; e < count; e += gridDim.x) {
    const int32_t j = fb_list[e];
    const float sx = sig[j], sy = sig[m + j], sz = sig[2 * m + j];
    unsigned long long k1 = kNone, k2 = kNone;
    for (int32_t i = threadIdx.x; i < n; i += kBlock)
      top2_insert(pack_key(direct_d(sx, sy, sz, x[i], y[i], z[i]), i), k1, k2);
    s1[threadIdx.x] = k1;
    s2[threadIdx.x] = k2;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
      if (threadIdx.x < w) {
        const unsigned long long a1 = s1[threadIdx.x], a2 = s2[threadIdx.x];
        const unsigned long long b1 = s1[threadIdx.x + w], b2 = s2[threadIdx.x + w];
        const unsigned long long lo = a1 < b1 ? a1 : b1, hi = a1 < b1 ? b1 : a1;
        const unsigned long long rest = a2 < b2 ? a2 : b2;
        s1[threadIdx.x] = lo;
        s2[threadIdx.x] = hi < rest ? hi : rest;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      winner[j] = static_cast<int32_t>(s1[0] & 0xFFFFFFFFu);
      second[j] = static_cast<int32_t>(s2[0] & 0xFFFFFFFFu);
      d1[j] = __uint_as_float(static_cast<uint32_t>(s1[0] >> 32));
      d2[j] = __uint_as_float(static_cast<uint32_t>(s2[0] >> 32));
    }
    __syncthreads();
  }
}

}  // namespace

// Regions of the caller's grid workspace (offsets from its 256-aligned base).
static void grid_layout(int64_t cells, int32_t n_max, int32_t m_max, size_t* off) {
  size_t o = 0;
  const size_t sz[7] = {4 * static_cast<size_t>(cells + 1), 4 * static_cast<size_t>(cells + 1),
                        4 * static_cast<size_t>(cells / kBlock + 2),
                        16 * static_cast<size_t>(n_max), 4 * static_cast<size_t>(n_max),
                        4 * static_cast<size_t>(m_max), 256};
  for (int i = 0; i < 7; ++i) {
    off[i] = o;
    o = (o + sz[i] + 255) & ~static_cast<size_t>(255);
  }
  off[7] = o;
}

size_t grid_bytes(int64_t cells, int32_t n_max, int32_t m_max) {
  size_t off[8];
  grid_layout(cells, n_max, m_max, off);
  return off[7];
}

GridBufs carve_grid(void* base, int64_t cells, int32_t n_max, int32_t m_max) {
  size_t off[8];
  grid_layout(cells, n_max, m_max, off);
  char* b = static_cast<char*>(base);
  GridBufs g;
  g.cnt = reinterpret_cast<int32_t*>(b + off[0]);
  g.start = reinterpret_cast<int32_t*>(b + off[1]);
  g.bsum = reinterpret_cast<int32_t*>(b + off[2]);
  g.sorted = reinterpret_cast<float4*>(b + off[3]);
  g.ucell = reinterpret_cast<int32_t*>(b + off[4]);
  g.fb_list = reinterpret_cast<int32_t*>(b + off[5]);
  g.nfb = reinterpret_cast<int32_t*>(b + off[6]);
  return g;
}

hipError_t launch_find_grid(const DevState& s, const GridBufs& gb, const GridSpec& spec,
                            int32_t n, const float* sig, int32_t m, int32_t* winner,
                            int32_t* second, float* d1, float* d2, hipStream_t st) {
  const int32_t cells = static_cast<int32_t>(spec.cells);
  const GridArgs g{spec.lo[0], spec.lo[1], spec.lo[2], spec.inv_h,
                   spec.dims[0], spec.dims[1], spec.dims[2], spec.exact};
  gx_clear<<<std::min(blocks(cells), 1024), kBlock, 0, st>>>(gb.cnt, cells, gb.nfb);
  gx_count<<<blocks(n), kBlock, 0, st>>>(n, s.x, s.y, s.z, g, gb.ucell, gb.cnt);
  const int nb = static_cast<int>((cells + kScanPart - 1) / kScanPart);
  gx_bsum<<<nb, kBlock, 0, st>>>(cells, gb.cnt, gb.bsum);
  if (nb > kFoldBlocks) {
    const hipError_t e = launch_scan_blocks(gb.bsum, nb, INT64_MAX, nullptr, s.status, -1, st);
    if (e != hipSuccess) return e;
  }
  gx_start<<<nb, kBlock, 0, st>>>(cells, n, gb.cnt, gb.bsum, nb, nb <= kFoldBlocks ? 1 : 0,
                                  gb.start);
  gx_scatter<<<blocks(n), kBlock, 0, st>>>(n, s.x, s.y, s.z, gb.ucell, gb.start, gb.cnt,
                                           gb.sorted);
  const int64_t lanes = static_cast<int64_t>(m) * kGroupLanes;
  gx_query<<<static_cast<int>((lanes + kQueryBlock - 1) / kQueryBlock), kQueryBlock, 0, st>>>(
      sig, m, g, gb.start, gb.sorted, winner, second, d1, d2, gb.fb_list, gb.nfb);
  gx_fallback<<<kFallbackBlocks, kBlock, 0, st>>>(sig, m, n, s.x, s.y, s.z, gb.fb_list, gb.nfb,
                                                  winner, second, d1, d2);
  return hipGetLastError();
}

}  // namespace gsn
