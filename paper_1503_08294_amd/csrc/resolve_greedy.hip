// Greedy lock-set resolve (lock_mode 2): the lock sets L_j = {b_j, s_j} + N(b_j) of the
// lock-set reading of Sec. 2.2, with the signals taken in key order: j is accepted iff L_j
// is disjoint from the lock sets accepted before it.  Computed in rounds.  In a round every
// pending signal with a unit of L_j taken by an accepted signal is rejected, the others claim
// L_j with a 64-bit atomic minimum of their key, and one that holds all of L_j is accepted and
// marks its units taken.  (An accepted signal held every unit it shares with a pending one, so
// its key is the smaller.)  A signal is settled once every signal of smaller key whose lock set
// meets L_j is settled, exactly as in the sequential greedy order, so the result is that
// order's; the pending signal of smallest key is always settled, so every round makes
// progress.  The first rounds are grid-wide launches, the rest run in one workgroup.
//
// These kernels wait on chains of dependent loads.  Rejecting at the claim instead of at the
// check settles in the second round nearly all that the first leaves (of 16,001 signals on
// 99,991 units about half are pending after the first check, 1,100 claim again, 300 are
// pending after the second), where a check that both rejects and accepts took twice the
// rounds.  With that, eight lanes per signal in the grid-wide rounds, one pass over the
// signal states in the last workgroup, and the acceptance written by the update, a resolve
// takes six launches and 22 us where it took eight and 53 (65,536 signals on 100,000 units:
// 33.5 us).
#include "gsn_internal.h"

namespace gsn {
namespace {

constexpr int kRoundBlock = 256;
constexpr int kTailBlock = 1024;

inline int blocks(int64_t n) { return static_cast<int>((n + kBlock - 1) / kBlock); }

struct GreedyArgs {
  int32_t m, n;
  const int32_t* winner;
  const int32_t* second;
  const float* d1;
  int key_mode;
  const int32_t* rp;
  const int32_t* col;
  unsigned long long* lock;
  int32_t* taken;      // 1: unit of an accepted lock set
  uint8_t* state;      // 0 rejected, 1 pending, 2 accepted
  int32_t* list;
  int32_t* status;
  unsigned long long* acc64;
};

// Rows of up to this many entries (nearly all of them) are read in one batch of loads
// (indices past the row's end repeat its last entry and are ignored).
constexpr int kShortRow = 8;
constexpr int kGroup = 8;    // lanes per signal in the grid-wide rounds

// whether a predicate holds in any lane of the calling thread's group
__device__ __forceinline__ bool any_of_group(bool p) {
  const int base = static_cast<int>(threadIdx.x & 63) & ~(kGroup - 1);
  return (static_cast<uint32_t>(__ballot(p) >> base) & ((1u << kGroup) - 1)) != 0;
}

// A signal of the single-workgroup rounds, one thread each: false if a unit of L_j is taken,
// else the claims.
__device__ bool t_claim(const GreedyArgs& a, int32_t j) {
  const int32_t b = a.winner[j], s = a.second[j];
  const unsigned long long key = signal_key(a.d1[j], j, a.key_mode);
  const int32_t r0 = a.rp[b], r1 = a.rp[b + 1];
  bool blocked = a.taken[b] != 0 || a.taken[s] != 0;
  for (int32_t k0 = r0; k0 < r1; k0 += kShortRow) {
    int32_t c[kShortRow], t[kShortRow];
#pragma unroll
    for (int k = 0; k < kShortRow; ++k) c[k] = a.col[min(k0 + k, r1 - 1)];
#pragma unroll
    for (int k = 0; k < kShortRow; ++k) t[k] = a.taken[c[k]];
#pragma unroll
    for (int k = 0; k < kShortRow; ++k) blocked |= t[k] != 0;
  }
  if (blocked) return false;
  atomicMin(&a.lock[b], key);
  atomicMin(&a.lock[s], key);
  claim_row(a.lock, a.col, r0, r1 - r0, key);
  return true;
}

// Whether j holds all of L_j; it releases what it holds, and marks L_j taken if it does.  The
// claims were made in the same launch, so the words are read at device scope, where the minima
// are made.
__device__ bool t_check(const GreedyArgs& a, int32_t j) {
  const int32_t b = a.winner[j], s = a.second[j];
  const unsigned long long key = signal_key(a.d1[j], j, a.key_mode);
  bool holds = true;
  auto read = [&](int32_t u) {
    return __hip_atomic_load(&a.lock[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto visit = [&](int32_t u, unsigned long long w) {
    if (w == key)
      __hip_atomic_store(&a.lock[u], ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      holds = false;
  };
  const int32_t r0 = a.rp[b], r1 = a.rp[b + 1];
  const unsigned long long wb = read(b), ws = read(s);
  bool s_nb = false;
  for (int32_t k0 = r0; k0 < r1; k0 += kShortRow) {
    int32_t c[kShortRow];
    unsigned long long w[kShortRow];
#pragma unroll
    for (int k = 0; k < kShortRow; ++k) c[k] = a.col[min(k0 + k, r1 - 1)];
#pragma unroll
    for (int k = 0; k < kShortRow; ++k) w[k] = read(c[k]);
#pragma unroll
    for (int k = 0; k < kShortRow; ++k)
      if (k0 + k < r1) {
        s_nb |= c[k] == s;
        visit(c[k], w[k]);
      }
  }
  visit(b, wb);
  if (!s_nb) visit(s, ws);
  if (!holds) return false;
  a.taken[b] = 1;
  a.taken[s] = 1;
  for (int32_t k = r0; k < r1; ++k) a.taken[a.col[k]] = 1;
  return true;
}

__global__ void rg_init(GreedyArgs a) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < a.n) {
    a.lock[i] = ~0ull;
    a.taken[i] = 0;
  }
  if (i < a.m) {
    const bool ok = pair_ok(a.winner[i], a.second[i], a.n);
    if (!ok) raise_error(a.status, GSN_E_INVAL);
    a.state[i] = ok ? 1 : 0;
  }
}

// A grid-wide round, eight lanes per signal: lane q takes the neighbours q, q + 8, ... of b,
// lane 0 also b and s.
__global__ __launch_bounds__(kRoundBlock) void rg_claim(GreedyArgs a) {
  const int32_t gt = blockIdx.x * kRoundBlock + threadIdx.x;
  const int32_t j = gt / kGroup;
  const int q = gt % kGroup;
  if (j >= a.m || a.state[j] != 1) return;   // whole groups
  const int32_t b = a.winner[j], s = a.second[j];
  const float dj = a.d1[j];
  const int32_t r0 = a.rp[b], r1 = a.rp[b + 1];
  bool blocked = q == 0 && (a.taken[b] != 0 || a.taken[s] != 0);
  const int32_t v0 = r0 + q < r1 ? a.col[r0 + q] : -1;
  if (v0 >= 0) blocked |= a.taken[v0] != 0;
  for (int32_t k = r0 + q + kGroup; k < r1; k += kGroup) blocked |= a.taken[a.col[k]] != 0;
  if (any_of_group(blocked)) {
    if (q == 0) a.state[j] = 0;
    return;
  }
  const unsigned long long key = signal_key(dj, j, a.key_mode);
  if (q == 0) {
    atomicMin(&a.lock[b], key);
    atomicMin(&a.lock[s], key);
  }
  if (v0 >= 0) atomicMin(&a.lock[v0], key);
  for (int32_t k = r0 + q + kGroup; k < r1; k += kGroup) atomicMin(&a.lock[a.col[k]], key);
}

// The words were claimed by an earlier launch (kernel boundaries make the minima visible to
// plain loads) while the only writes are releases by the holders, so plain loads and stores
// serve here: a stale word reads as its claimed key or as all ones, and only the signal that
// held it at the end of the claims sees its own key.
__global__ __launch_bounds__(kRoundBlock) void rg_check(GreedyArgs a) {
  const int32_t gt = blockIdx.x * kRoundBlock + threadIdx.x;
  const int32_t j = gt / kGroup;
  const int q = gt % kGroup;
  if (j >= a.m || a.state[j] != 1) return;   // whole groups
  const int32_t b = a.winner[j], s = a.second[j];
  const unsigned long long key = signal_key(a.d1[j], j, a.key_mode);
  const int32_t r0 = a.rp[b], r1 = a.rp[b + 1];
  unsigned long long lb = 0, ls = 0;
  if (q == 0) {
    lb = a.lock[b];
    ls = a.lock[s];
  }
  const int32_t v0 = r0 + q < r1 ? a.col[r0 + q] : -1;
  const unsigned long long l0 = v0 >= 0 ? a.lock[v0] : 0;
  bool holds = true, is_s = v0 == s;
  auto visit = [&](int32_t u, unsigned long long w) {
    if (w == key) a.lock[u] = ~0ull; else holds = false;
  };
  if (v0 >= 0) visit(v0, l0);
  for (int32_t k = r0 + q + kGroup; k < r1; k += kGroup) {
    const int32_t v = a.col[k];
    is_s |= v == s;
    visit(v, a.lock[v]);
  }
  const bool s_nb = any_of_group(is_s);
  if (q == 0) {
    visit(b, lb);
    if (!s_nb) visit(s, ls);
  }
  if (any_of_group(!holds)) return;
  if (q == 0) {
    a.state[j] = 2;
    a.taken[b] = 1;
    a.taken[s] = 1;
  }
  if (v0 >= 0) a.taken[v0] = 1;
  for (int32_t k = r0 + q + kGroup; k < r1; k += kGroup) a.taken[a.col[k]] = 1;
}

// The remaining rounds in one workgroup; with accepted not null (the separate resolve call)
// then the acceptance flags of all signals and their counts in the statistics.
__global__ __launch_bounds__(kTailBlock) void rg_tail(GreedyArgs a, uint8_t* accepted) {
  constexpr int kNear = 4096;   // a list of up to so many pending signals is held in LDS
  __shared__ int32_t near[2][kNear];
  __shared__ int32_t s_n, s_next;
  const int tid = threadIdx.x;
  if (tid == 0) {
    s_n = 0;
    s_next = 0;
  }
  __syncthreads();
  // sixteen states per load (they start on a 256-byte boundary, in a region padded to one)
  const int32_t words = (a.m + 15) / 16;
  for (int32_t i = tid; i < words; i += kTailBlock) {
    const uint4 w = reinterpret_cast<const uint4*>(a.state)[i];
    const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (((v[k / 4] >> (8 * (k % 4))) & 0xffu) == 1u && 16 * i + k < a.m) {
        const int32_t at = atomicAdd(&s_n, 1);
        if (at < kNear) near[0][at] = 16 * i + k;
        a.list[at] = 16 * i + k;
      }
  }
  __syncthreads();
  const bool lds = s_n <= kNear;
  int32_t* cur = lds ? near[0] : a.list;
  int32_t* nxt = lds ? near[1] : a.list + a.m;
  for (;;) {
    const int32_t n = s_n;
    if (n == 0) break;
    for (int32_t i = tid; i < n; i += kTailBlock)
      if (!t_claim(a, cur[i])) {
        a.state[cur[i]] = 0;
        cur[i] = -1;
      }
    __syncthreads();
    for (int32_t i = tid; i < n; i += kTailBlock) {
      const int32_t j = cur[i];
      if (j < 0) continue;
      if (t_check(a, j)) a.state[j] = 2;
      else nxt[atomicAdd(&s_next, 1)] = j;
    }
    __syncthreads();
    if (tid == 0) {
      if (s_next == n) {  // no progress: the lock words were not cleared on entry
        raise_error(a.status, GSN_E_STATE);
        s_next = 0;
      }
      s_n = s_next;
      s_next = 0;
    }
    __syncthreads();
    int32_t* t = cur;
    cur = nxt;
    nxt = t;
  }
  if (accepted == nullptr) return;
  // the counts with one atomic each (hundreds of same-address atomics would queue at the
  // cache)
  __shared__ int32_t s_acc;
  if (tid == 0) s_acc = 0;
  __syncthreads();
  int32_t mine = 0;
  for (int32_t j = tid; j < a.m; j += kTailBlock) {
    const bool acc = a.state[j] == 2;
    accepted[j] = acc ? 1 : 0;
    mine += acc;
  }
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
  if ((tid & 63) == 0 && mine != 0) atomicAdd(&s_acc, mine);
  __syncthreads();
  if (tid == 0) {
    atomicAdd(&a.acc64[kA64Resolved], static_cast<unsigned long long>(a.m));
    if (s_acc != 0) atomicAdd(&a.acc64[kA64Accepted], static_cast<unsigned long long>(s_acc));
  }
}

}  // namespace

hipError_t launch_resolve_greedy(const DevState& s, int cur, int32_t n, int32_t m,
                                 const int32_t* winner, const int32_t* second, const float* d1,
                                 uint8_t* accepted, int key_mode, int grid_rounds,
                                 hipStream_t st, bool claimed) {
  GreedyArgs a{m, n, winner, second, d1, key_mode, s.rp[cur], s.col[cur], s.lock,
               s.extra, s.pend, s.list, s.status, s.acc64};
  if (!claimed) rg_init<<<blocks(std::max(n, m)), kBlock, 0, st>>>(a);
  const int g = static_cast<int>((static_cast<int64_t>(m) * kGroup + kRoundBlock - 1) /
                                 kRoundBlock);
  for (int32_t t = 0; t < grid_rounds; ++t) {
    // (round 0's claims may come from the find)
    if (t > 0 || !claimed) rg_claim<<<g, kRoundBlock, 0, st>>>(a);
    rg_check<<<g, kRoundBlock, 0, st>>>(a);
  }
  rg_tail<<<1, kTailBlock, 0, st>>>(a, accepted);
  return hipGetLastError();
}

}  // namespace gsn
