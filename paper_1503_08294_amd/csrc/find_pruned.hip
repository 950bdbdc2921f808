// Find Winners over the units in spatial order, with whole blocks of units left out where a
// bound shows that they hold neither of the two nearest (variant 7: the default above 256
// signals, and for smaller batches in a running network).
//
// Order and blocks.  The units are gathered into the staging's spatial order (staging.hip)
// as packed (x, y, z, index) records; every leaf of 32 consecutive records, every top of 512 and
// every sixteen tops have their bounding box (pruned_gather.h, from the present positions, so
// the boxes are exact however old the order is; the order affects speed only).
//
// The bound needs no rounding margin.  With g_a = max(lo_a - s_a, s_a - hi_a, 0), each
// difference rounded, and L = (g_x g_x + g_y g_y) + g_z g_z in the operation order of the
// distance: for a unit w in the box w_a <= hi_a, so s_a - w_a >= s_a - hi_a, and rounding
// to nearest is monotone, so |fl(s_a - w_a)| >= g_a (likewise below lo_a); products and sums
// of non-negative numbers are monotone under rounding too, hence the computed distance of w
// is >= L.  A box is left out only if L > B, B the computed distance of a real unit that is
// at least the second smallest one: every unit that can enter the two nearest, ties by index
// included, is in a box that is visited.  A comparison with NaN or between infinities never
// leaves a box out.
//
// Search.  L lanes of a wave per signal.  The leaf around the signal's cell gives B; the lanes
// test the outermost boxes, then the tops and the leaves of those that pass, each list
// compacted in LDS, and evaluate the units of the leaves that pass (about six of 32 units on a
// surface).  The kernel is bound by the vector unit for many signals (554 instructions a wave of
// two signals at 100,000 units and 65,536 signals, 83% of the issue cycles) and by the chain of
// seven dependent loads for few (waves wait 64% of their cycles at 37,501 and 2,999).  At 200,000
// units and 16,384 signals an iteration's search takes 16.5 us with its claims (and 3.7 more in
// the rewrite that gathers for it), where staging, the exhaustive screen on the matrix cores and
// its merge took 125; at 100,000 and 65,536, 36.6 us where they took 231.  What it took: boxes in
// three levels with leaves of 32 units (88 us with 64 and two levels), cells in cubes, 64 a side
// (32 a side fitted to the box: a quarter more leaves), and the tries below, without which the few
// signals with a poor first bound (one unit in their cell, the next in Morton order far off) held
// up four launches in ten by 12 to 40 us.  16 lanes a signal measured 26.3 and 43.6 us (when 32
// measured 20.6 and 42.1), 8 and 4 lanes more.
#include <type_traits>

#include "pruned_gather.h"

namespace gsn {
namespace {

constexpr int kLeaf = kPrunedLeaf;
constexpr int kTop = kPrunedTop;
constexpr int kFan = kTop / kLeaf;   // leaves of a top
constexpr int32_t kWideBatch = 8192;    // signals up to which a signal gets a whole wave

// minimum over the L lanes of a group, in every lane
template <int L>
__device__ __forceinline__ unsigned long long min_group(unsigned long long v) {
  v = min(v, row_move<0xB1>(v));
  v = min(v, row_move<0x4E>(v));
  v = min(v, row_move<0x141>(v));
  v = min(v, row_move<0x140>(v));
#pragma unroll
  for (int off = 16; off < L; off <<= 1) v = min(v, __shfl_xor(v, off));
  return v;
}

__device__ __forceinline__ float gap(float s, float lo, float hi) {
  return fmaxf(fmaxf(lo - s, s - hi), 0.0f);
}

__device__ __forceinline__ float box_bound(float sx, float sy, float sz, float4 lo, float4 hi) {
  const float gx = gap(sx, lo.x, hi.x), gy = gap(sy, lo.y, hi.y), gz = gap(sz, lo.z, hi.z);
  return (gx * gx + gy * gy) + gz * gz;
}

// ------------------------------------------------------------------- gather ----

__global__ __launch_bounds__(kBlock) void pr_gather(GatherArgs g) {
  __shared__ float red[kGatherRed];
  gather_top(g, blockIdx.x, red);
}

// ------------------------------------------------------------------- search ----

template <int CTRL>
__device__ __forceinline__ float row_float(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

__device__ __forceinline__ void second_step(float& a1, float& a2, float b1, float b2) {
  const float hi = fmaxf(a1, b1);
  a1 = fminf(a1, b1);
  a2 = fminf(hi, fminf(a2, b2));
}

// second smallest of the values of a group's lanes (two per lane, d1 <= d2; NaN left out)
template <int L>
__device__ __forceinline__ float second_of_group(float d1, float d2) {
  const float inf = __builtin_huge_valf();
  d1 = fminf(d1, inf);   // (a NaN in a maximum would hide the other value)
  d2 = fminf(d2, inf);
  second_step(d1, d2, row_float<0xB1>(d1), row_float<0xB1>(d2));
  second_step(d1, d2, row_float<0x4E>(d1), row_float<0x4E>(d2));
  second_step(d1, d2, row_float<0x141>(d1), row_float<0x141>(d2));
  second_step(d1, d2, row_float<0x140>(d1), row_float<0x140>(d2));
#pragma unroll
  for (int off = 16; off < L; off <<= 1)
    second_step(d1, d2, __shfl_xor(d1, off), __shfl_xor(d2, off));
  return d2;
}

struct PrunedArgs {
  const float4* pq;
  const float4* leaf;
  const float4* top;
  const int32_t* sup;
  int32_t nleaf, ntop;
  const int32_t* off_u;
  const float* bb;
  const float* sig;
  int32_t m;
  int32_t *winner, *second;
  float *d1, *d2;
  ClaimArgs claim;
  int do_claim;
  int32_t* mail;
};

constexpr int kFewUnits = 3;     // a cell with fewer leaves the first bound to a larger one
// A signal with more passing leaves than this has a poor bound: the nearest of those leaves
// improve it and the boxes are tested again, up to kTries times in all; on the last try up to
// kMostLeaves will do.
constexpr int kFewLeaves = 40;
constexpr int kMostLeaves = 64;
constexpr int kNearFrom = 8;     // passing leaves before the nearest is looked for (first try)
constexpr int kNearLeaves = 8;   // nearest leaves evaluated before another try
constexpr int kMostTops = 32;
constexpr int kTries = 4;

// (With more than 80 scalar registers fewer waves run side by side: 8,192 signals on 50,000 units
// 14.4 us instead of 13.2.)
template <int L>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_num_sgpr(80))) void pr_search(
    PrunedArgs a) {
  static_assert(L == 32 || L == 64, "two or four rows of 16 lanes");
  static_assert(kFan == 16, "one row of lanes tests the boxes of a node");
  constexpr int kGroups = kBlock / L;
  constexpr int kRows = L / 16;                     // nodes tested side by side
  constexpr int kSide = L > kLeaf ? L / kLeaf : 1;  // leaves evaluated side by side
  constexpr int kPer = kLeaf * kSide / L;           // units per lane
  constexpr int kUnroll = 2;                        // nodes per row and step
  __shared__ int32_t tops[kGroups][kMostTops + kUnroll * L];
  __shared__ int32_t leaves[kGroups][kMostLeaves];
  const int g = threadIdx.x / L, q = threadIdx.x % L;
  const int row = q / 16, c = q % 16;
  const int32_t j = blockIdx.x * kGroups + g;
  if (j >= a.m) return;   // whole groups; nothing below spans groups
  const float sx = a.sig[j], sy = a.sig[a.m + j], sz = a.sig[2 * a.m + j];
  const int32_t nsup = (a.ntop + kFan - 1) / kFan;
  const int sh = (threadIdx.x & 63) / L * L;     // first lane of the group in its wave
  // a group's part of a ballot, its set bits and those before this lane's
  using Bits = std::conditional_t<L == 64, unsigned long long, uint32_t>;
  const Bits before = static_cast<Bits>((1ull << q) - 1);
  auto bits = [&](bool p) -> Bits {
    const unsigned long long b = __ballot(p);
    if constexpr (L == 64) return b;
    else {
      return static_cast<uint32_t>(sh == 0 ? b : b >> 32);
    }
  };
  auto count = [](Bits b) {
    if constexpr (L == 64) return static_cast<int32_t>(__popcll(b));
    else return static_cast<int32_t>(__popc(b));
  };
  auto first = [](Bits b) {
    if constexpr (L == 64) return static_cast<int32_t>(__builtin_ctzll(b));
    else return static_cast<int32_t>(__builtin_ctz(b));
  };
  auto below = [&](Bits b) { return count(b & before); };
  unsigned long long k1 = kNone, k2 = kNone;
  float bound = __builtin_huge_valf();
  struct Units { float4 w[kPer]; };
  // the group's units of leaf lf (with kSide > 1, lanes from kLeaf on take leaf lf2)
  auto load_leaf = [&](int32_t lf, int32_t lf2) {
    const int32_t l = kSide > 1 && q >= kLeaf ? lf2 : lf;
    Units u;
#pragma unroll
    for (int i = 0; i < kPer; ++i) u.w[i] = a.pq[l * kLeaf + (i * L + q) % kLeaf];
    return u;
  };
  auto eval = [&](const Units& u, bool both) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const float dx = sx - u.w[i].x, dy = sy - u.w[i].y, dz = sz - u.w[i].z;
      const float d = (dx * dx + dy * dy) + dz * dz;
      if (!(d > bound) && (kSide == 1 || both || q < kLeaf)) {
        const unsigned long long k = pack_key(d, __float_as_int(u.w[i].w));
        k2 = min(k2, max(k1, k));
        k1 = min(k1, k);
      }
    }
  };
  // The second smallest distance of the group's units so far as the bound (the words of an
  // empty place read as NaN, which the minima leave out).
  auto tighten = [&]() {
    float d1 = __uint_as_float(static_cast<uint32_t>(k1 >> 32));
    float d2 = __uint_as_float(static_cast<uint32_t>(k2 >> 32));
    bound = fminf(bound, second_of_group<L>(d1, d2));
  };
  auto box = [&](const float4* b, int32_t i) {
    return box_bound(sx, sy, sz, b[2 * i], b[2 * i + 1]);
  };
  auto sup_box = [&](int32_t s) {
    const int4 u = *reinterpret_cast<const int4*>(a.sup + kSupWords * s);
    const int2 v = *reinterpret_cast<const int2*>(a.sup + kSupWords * s + 4);
    return box_bound(sx, sy, sz, make_float4(unord(u.x), unord(u.y), unord(u.z), 0.0f),
                     make_float4(unord(u.w), unord(v.x), unord(v.y), 0.0f));
  };

  // (the first supers' boxes are read beside the chain that gives the first bound)
  const float first_sup = sup_box(min(q, nsup - 1));
  // The leaf at the middle of the signal's cell gives the first bound; with few units in the
  // cell, of the eight or 64 cells it is one of (consecutive in Morton order).
  const int32_t key = stage_bucket(sx, sy, sz, a.bb);
  int32_t r0 = a.off_u[key], r1 = a.off_u[key + 1];
  {
    const int32_t p0 = a.off_u[key & ~7], p1 = a.off_u[(key | 7) + 1];
    const int32_t g0 = a.off_u[key & ~63], g1 = a.off_u[(key | 63) + 1];
    if (r1 - r0 < kFewUnits) {
      const bool parent = p1 - p0 >= kFewUnits;
      r0 = parent ? p0 : g0;
      r1 = parent ? p1 : g1;
    }
  }
  const int32_t home = min(max((r0 + r1) / 2 / kLeaf, 0), a.nleaf - 1);
  eval(load_leaf(home, home), false);
  tighten();

  int32_t nl = 0, skip = home, tried = -1;
  bool many;
  for (int attempt = 1;; ++attempt) {
    // the tops that pass, through the boxes of kFan of them
    int32_t nt = 0;
    for (int32_t s0 = 0; s0 < nsup && nt <= kMostTops; s0 += L) {
      const int32_t s = s0 + q;
      const float ls = s0 == 0 ? first_sup : sup_box(min(s, nsup - 1));
      Bits sm = bits(s < nsup && !(ls > bound));
      while (sm != 0 && nt <= kMostTops) {
        // kUnroll supers per row at a time
        int32_t t[kUnroll];
        bool have[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          t[u] = 0;
          have[u] = false;
#pragma unroll
          for (int r = 0; r < kRows; ++r) {
            if (r == row) {
              have[u] = sm != 0;
              t[u] = (s0 + (sm != 0 ? first(sm) : 0)) * kFan + c;
            }
            sm &= sm - 1;
          }
          have[u] = have[u] && t[u] < a.ntop;
        }
        float lb[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) lb[u] = box(a.top, min(t[u], a.ntop - 1));
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const bool pass = have[u] && !(lb[u] > bound);
          const Bits b = bits(pass);
          if (pass) tops[g][nt + below(b)] = t[u];
          nt += count(b);
        }
      }
    }
    wave_lds_fence();
    const int32_t mt = min(nt, kMostTops);

    // their leaves that pass, and the nearest of them
    nl = 0;
    unsigned long long near = kNone;
    for (int32_t k = row; k < mt + row; k += kUnroll * kRows) {
      int32_t f[kUnroll];
      float lb[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) f[u] = tops[g][min(k + u * kRows, mt - 1)] * kFan + c;
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) lb[u] = box(a.leaf, min(f[u], a.nleaf - 1));
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const bool pass = k + u * kRows < mt && f[u] < a.nleaf && f[u] != skip &&
                          !(lb[u] > bound);
        // (of the first few there is no need: most signals have no more)
        if ((nl > kNearFrom || attempt > 1) && pass && f[u] != tried)
          near = min(near, pack_key(lb[u], f[u]));
        const Bits b = bits(pass);
        const int32_t at = nl + below(b);
        if (pass && at < kMostLeaves) leaves[g][at] = f[u];
        nl += count(b);
      }
    }
    wave_lds_fence();
    many = nt > kMostTops || nl > kMostLeaves;
    if (attempt == kTries || (!many && nl <= kFewLeaves)) break;

    // Nearest first, each lane's nearest leaf in turn, while one is nearer than the bound: boxes
    // that span a jump of the order hold many signals and few units near them.  (With each try
    // the lists start again from nothing: a unit enters them once.)
    for (int i = 0; i < kNearLeaves; ++i) {
      const unsigned long long best = min_group<L>(near);
      if (best == kNone || __uint_as_float(static_cast<uint32_t>(best >> 32)) > bound) break;
      if (near == best) near = kNone;
      tried = static_cast<int32_t>(static_cast<uint32_t>(best));
      k1 = k2 = kNone;
      eval(load_leaf(tried, tried), false);
      tighten();
    }
    k1 = k2 = kNone;
    skip = -1;
  }
  if (!many && nl > 0) {
    Units u = load_leaf(leaves[g][0], leaves[g][min(1, nl - 1)]);
    int32_t e = kSide;
    for (; e < nl; e += kSide) {
      const Units v = load_leaf(leaves[g][e], leaves[g][min(e + 1, nl - 1)]);
      eval(u, true);
      u = v;
    }
    eval(u, e <= nl);
  }
  // A hard signal (near the centre of a closed surface, or so far away that distances round alike,
  // no box can be left out): a top per lane, then the leaves of a row's tops, then the units of
  // those that pass, eight leaves on their way at a time.  Bound by that chain of loads when few
  // signals are hard, by the vector unit and the cache when all are: on 200,000 units of a
  // sphere, 16,384 signals at its centre take 1.8 ms a find (one leaf after another took 2.1, and
  // the scan of every pair, whose screen passes them all too, takes 2.8), one among others on the
  // surface 0.73 (1.4 and 1.2).
  if (many) {
    for (int32_t t0 = 0; t0 < a.ntop; t0 += L) {
      const int32_t t = t0 + q;
      Bits tm = bits(t < a.ntop && !(box(a.top, min(t, a.ntop - 1)) > bound));
      while (tm != 0) {
        int32_t f = a.nleaf;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          if (r == row && tm != 0) f = (t0 + first(tm)) * kFan + c;
          tm &= tm - 1;
        }
        const bool pass = f < a.nleaf && !(box(a.leaf, min(f, a.nleaf - 1)) > bound);
        const Bits lm = bits(pass);
        const int32_t n = count(lm);
        if (pass) leaves[g][below(lm)] = f;
        wave_lds_fence();
        const unsigned long long was = k2;
        constexpr int kAhead = 8 / kSide;
        for (int32_t e0 = 0; e0 < n; e0 += kAhead * kSide) {
          Units u[kAhead];
#pragma unroll
          for (int i = 0; i < kAhead; ++i) {
            const int32_t e = e0 + i * kSide;
            u[i] = load_leaf(leaves[g][min(e, n - 1)], leaves[g][min(e + 1, n - 1)]);
          }
#pragma unroll
          for (int i = 0; i < kAhead; ++i)
            if (e0 + i * kSide < n) eval(u[i], e0 + i * kSide + 1 < n);
        }
        wave_lds_fence();
        if (bits(k2 < was) != 0) tighten();
      }
    }
    if (q == 0 && a.m <= kSmallM)   // (the host goes back to the scan for a while)
      __hip_atomic_store(a.mail, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  // the least key of the group, then the least of the others
  const unsigned long long best1 = min_group<L>(k1);
  k2 = min_group<L>(k1 == best1 ? k2 : k1);
  k1 = best1;
  // Fewer than two distances are numbers (their keys are above all others): as in the scans, a
  // small batch has no such unit for an answer, and in a larger one a signal that is no number
  // has the two of lowest index.
  constexpr unsigned long long kInfinite = 0x7f800000ffffffffull;
  if (k2 > kInfinite) {
    const bool none = k1 > kInfinite;
    if (a.m <= kSmallM) {
      k2 = kNone;
      if (none) k1 = kNone;
    } else if (none) {
      k1 &= ~0xffffffffull;
      k2 = k1 | 1u;
    }
  }

  const int32_t bw = static_cast<int32_t>(static_cast<uint32_t>(k1));
  const int32_t sw = static_cast<int32_t>(static_cast<uint32_t>(k2));
  const float dw = __uint_as_float(static_cast<uint32_t>(k1 >> 32));
  if (q == 0) {
    a.winner[j] = bw;
    a.second[j] = sw;
    a.d1[j] = dw;
    a.d2[j] = __uint_as_float(static_cast<uint32_t>(k2 >> 32));
  }
  if (!a.do_claim) return;
  const bool ok = pair_ok(bw, sw, a.claim.n);
  if (a.claim.pend && q == 0) a.claim.pend[j] = ok ? 1 : 0;
  if (!ok) {
    if (q == 0) raise_error(a.claim.status, GSN_E_INVAL);
    return;
  }
  const unsigned long long ck = signal_key(dw, j, a.claim.key_mode);
  if (q == 0) {
    atomicMin(&a.claim.lock[bw], ck);
    if (!a.claim.winner_only) atomicMin(&a.claim.lock[sw], ck);
  }
  if (a.claim.winner_only) return;
  for (int32_t k = a.claim.rp[bw] + q; k < a.claim.rp[bw + 1]; k += L)
    atomicMin(&a.claim.lock[a.claim.col[k]], ck);
}

}  // namespace

GatherArgs pruned_gather_args(const DevState& s, const StageBufs& b, int32_t n, int32_t slots,
                              int32_t n_max, int par) {
  const int32_t words = sup_words(n_max);
  return GatherArgs{s.x, s.y, s.z, b.pidx, b.pq, b.leaf, b.top, b.sup + par * words,
                    b.sup + stage_next(par) * words, n, slots, (slots + kTop - 1) / kTop, words};
}

hipError_t launch_pruned_gather(const GatherArgs& g, hipStream_t st) {
  pr_gather<<<g.tops, kBlock, 0, st>>>(g);
  return hipGetLastError();
}

hipError_t launch_pruned_search(const StageBufs& b, int32_t n, int32_t slots, int32_t n_max,
                                int par, const float* sig, int32_t m, int32_t* winner,
                                int32_t* second, float* d1, float* d2, const ClaimArgs* claim,
                                int32_t* mail, hipStream_t st, LaunchEvents ev) {
  if (n < 2 || m < 1) return hipErrorInvalidValue;
  const PrunedArgs a{b.pq, b.leaf, b.top, b.sup + par * sup_words(n_max),
                     (slots + kLeaf - 1) / kLeaf, (slots + kTop - 1) / kTop, b.off_u, b.bb, sig, m,
                     winner, second, d1, d2, claim ? *claim : ClaimArgs{}, claim ? 1 : 0, mail};
  auto go = [&](auto k, int lanes) {
    const int per = kBlock / lanes;
    launch_with(k, dim3((m + per - 1) / per), dim3(kBlock), st, ev, a);
  };
  // A wave per signal while the batch leaves waves free (2,048 signals on 50,000 units 5.8 us
  // against 6.2 with two signals a wave, on 100,000 6.5 against 9.2; 4,096 on 200,000 7.5 against
  // 7.8), two signals a wave beyond (16,384 on 200,000 15.9 against 12.8, 65,536 on 100,000 48.4
  // against 31.4).  Between the two it depends on the units: 8,192 on 50,000 take 9.9 against 8.9
  // at rest, 13.2 against 13.7 in a network that is pruned and grows.
  if (m <= kWideBatch) go(pr_search<64>, 64);
  else go(pr_search<32>, 32);
  return hipGetLastError();
}

}  // namespace gsn
