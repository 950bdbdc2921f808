// Host side of the C ABI declared in include/gsn.h: argument validation, workspace
// carving, launch configuration, call ordering and event timing.  All device memory is the
// caller's; this file allocates only the handle (and short-lived host vectors in the
// synchronous export/import calls).
#include <stdlib.h>
#include <string.h>

#include <cmath>
#include <cstddef>
#include <mutex>
#include <new>
#include <vector>

#include "gsn_internal.h"

// The grid workspace of gsn_find_winners_grid_noalloc, for callers that cannot allocate:
// one fixed array per GPU, held from the library's load until the process ends.  In host
// code the name only stands for the symbol; its device address on each GPU comes from
// hipGetSymbolAddress (noalloc_scratch below), and only that address is used.
static __device__ __align__(256) unsigned char scratch[GSN_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device with that
// device current; nullptr if the lookup fails.
void* noalloc_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_dev[dev] = ptr;
  }
  return g_scratch_dev[dev];
}

}  // namespace

namespace gsn {

Layout layout_for(const gsn_params& p) {
  Layout L{};
  size_t o = 0;
  int i = 0;
  auto add = [&](size_t bytes) {
    o = (o + 255) & ~static_cast<size_t>(255);
    L.off[i++] = o;
    o += bytes;
  };
  const size_t nm = static_cast<size_t>(p.n_max);
  const size_t mm = static_cast<size_t>(p.m_max);
  // the winner-lock update works on a copy of the adjacency with room for one insertion
  // per survivor at its winner and one at its second
  const size_t hc = 2 * (static_cast<size_t>(p.e_max) + (p.lock_mode == 1 ? mm : 0)) + 2;
  add(4 * nm);                 // 0 x
  add(4 * nm);                 // 1 y
  add(4 * nm);                 // 2 z
  add(4 * nm);                 // 3 err
  add(4 * (nm + 2));           // 4 rp0
  add(4 * (nm + 2));           // 5 rp1
  add(4 * hc);                 // 6 col0
  add(4 * hc);                 // 7 col1
  add(4 * hc);                 // 8 age0
  add(4 * hc);                 // 9 age1
  add(8 * nm);                 // 10 lock
  add(4 * nm);                 // 11 ins
  add(4 * nm);                 // 12 orphan
  add(4 * nm);                 // 13 cnt
  add(4 * (nm / kBlock + 2));  // 14 bsum
  add(16 * nm);                // 15 tmp
  add(4 * kStSlots);           // 16 status
  add(8 * static_cast<size_t>(kMaxSplit) * 2 * mm);  // 17 part
  add(stage_bytes(p.n_max, p.m_max));                 // 18 screened staging
  add(mm);                     // 19 pend
  add(4 * nm);                 // 20 len
  add(4 * nm);                 // 21 extra
  add(4 * kRmWords);           // 22 rem
  add(8 * mm);                 // 23 list
  add(12 * mm);                // 24 schedule signals
  add(4 * mm);                 // 25 schedule winners
  add(4 * mm);                 // 26 schedule seconds
  add(4 * mm);                 // 27 schedule d1
  add(4 * mm);                 // 28 schedule d2
  add(mm);                     // 29 schedule acceptance
  add(8 * kA64Slots);          // 30 64-bit accumulators
  add(4 * (mm / 32 + 2));      // 31 accepted signals per workgroup of the fused check
  add(8 * small_part_keys(p.m_max));  // 32 partial keys of the small-batch scan
  add(4 * (nm / kBlock + 2));  // 33 per-block half-edge changes, set 0
  add(4 * (nm / kBlock + 2));  // 34 per-block half-edge changes, set 1
  const bool wl = p.lock_mode == 1;
  add(wl ? 32 * nm : 0);       // 35 survivor records (key, second), two parities
  add(wl ? 2 * nm : 0);        // 36 survivor flags, two parities
  add(wl ? 8 * nm : 0);        // 37 heads of the second lists, two parities
  add(wl ? 8 * mm : 0);        // 38 links of the second lists
  add(wl ? 8 : 0);             // 39 table bounds
  L.total = (o + 255) & ~static_cast<size_t>(255);
  return L;
}

void carve(const gsn_params& p, void* base, DevState* s) {
  const Layout L = layout_for(p);
  char* b = static_cast<char*>(base);
  s->x = reinterpret_cast<float*>(b + L.off[0]);
  s->y = reinterpret_cast<float*>(b + L.off[1]);
  s->z = reinterpret_cast<float*>(b + L.off[2]);
  s->err = reinterpret_cast<float*>(b + L.off[3]);
  s->rp[0] = reinterpret_cast<int32_t*>(b + L.off[4]);
  s->rp[1] = reinterpret_cast<int32_t*>(b + L.off[5]);
  s->col[0] = reinterpret_cast<int32_t*>(b + L.off[6]);
  s->col[1] = reinterpret_cast<int32_t*>(b + L.off[7]);
  s->age[0] = reinterpret_cast<int32_t*>(b + L.off[8]);
  s->age[1] = reinterpret_cast<int32_t*>(b + L.off[9]);
  s->lock = reinterpret_cast<unsigned long long*>(b + L.off[10]);
  s->ins = reinterpret_cast<int32_t*>(b + L.off[11]);
  s->orphan = reinterpret_cast<int32_t*>(b + L.off[12]);
  s->cnt = reinterpret_cast<int32_t*>(b + L.off[13]);
  s->bsum = reinterpret_cast<int32_t*>(b + L.off[14]);
  s->tmp = reinterpret_cast<float*>(b + L.off[15]);
  s->status = reinterpret_cast<int32_t*>(b + L.off[16]);
  s->part = reinterpret_cast<unsigned long long*>(b + L.off[17]);
  s->scr = b + L.off[18];
  s->pend = reinterpret_cast<uint8_t*>(b + L.off[19]);
  s->len = reinterpret_cast<int32_t*>(b + L.off[20]);
  s->extra = reinterpret_cast<int32_t*>(b + L.off[21]);
  s->rem = reinterpret_cast<int32_t*>(b + L.off[22]);
  s->list = reinterpret_cast<int32_t*>(b + L.off[23]);
  s->ssig = reinterpret_cast<float*>(b + L.off[24]);
  s->swin = reinterpret_cast<int32_t*>(b + L.off[25]);
  s->ssec = reinterpret_cast<int32_t*>(b + L.off[26]);
  s->sd1 = reinterpret_cast<float*>(b + L.off[27]);
  s->sd2 = reinterpret_cast<float*>(b + L.off[28]);
  s->sacc = reinterpret_cast<uint8_t*>(b + L.off[29]);
  s->acc64 = reinterpret_cast<unsigned long long*>(b + L.off[30]);
  s->apart = reinterpret_cast<int32_t*>(b + L.off[31]);
  s->spart = reinterpret_cast<unsigned long long*>(b + L.off[32]);
  s->bdelta[0] = reinterpret_cast<int32_t*>(b + L.off[33]);
  s->bdelta[1] = reinterpret_cast<int32_t*>(b + L.off[34]);
  const bool wl = p.lock_mode == 1;
  s->wkey = wl ? reinterpret_cast<unsigned long long*>(b + L.off[35]) : nullptr;
  s->wflag = wl ? reinterpret_cast<uint8_t*>(b + L.off[36]) : nullptr;
  s->rhead = wl ? reinterpret_cast<int32_t*>(b + L.off[37]) : nullptr;
  s->rlink = wl ? reinterpret_cast<int2*>(b + L.off[38]) : nullptr;
  s->whi = wl ? reinterpret_cast<int32_t*>(b + L.off[39]) : nullptr;
}

}  // namespace gsn

using gsn::DevState;

enum Phase { kReady = 0, kFound = 1, kResolved = 2, kAdapted = 3 };
constexpr int kRebucketEvery = 64;     // default calls between rebuilds of the unit order
// Iterations of small batches on the same units, or finds alone on units at rest, after which
// they take the pruned search: its order and records cost about 60 us once, and then an iteration
// of a recorded loop takes less (64 signals on 100,000 units 18.3 us against 24.6, 256 19.4
// against 41.9, one 15.1 against 15.7; 256 on 1,000 units 16.4 against 18.0).
constexpr int32_t kSmallRun = 8;
// A new order is due once more than one unit in this many joined at its end (a growing run of 1.5 M
// signals: the search 8.7 us an iteration, new orders 0.7; 20.8 with one every 64 finds), or more
// than kAppendedMost.  Their leaves span the network, so nearly every signal visits them all: 32
// leaves still fit its lists without another try, 160 took the search from 11 to 73 us (a run from
// 2 to 116,080 units 0.274 s without this bound, 0.263 with 2,048, 0.243 with 1,024 and with 512).
constexpr int kAppendedPart = 16;
constexpr int32_t kAppendedMost = 1024;
// The search leaves out little for a hard signal (find_pruned.hip), and the few workgroups of a
// small batch take long over one: once a search has reported one, the next kScanRun small finds
// take the scan, whose time does not depend on the signals; then the search is tried again.  (64
// signals at the centre of 100,000 units on a sphere: 227 us a search, 15 a scan.)
constexpr int32_t kScanRun = 64;
constexpr int kDefaultGrab = 4;        // batches per grab of the dynamic scan
constexpr int kDefaultGridRounds = 6;  // before any update has reported back
// Grid-wide rounds of the greedy lock-set resolve: one while the last workgroup has a thread per
// signal (300 signals on 20,000 units: 11.4 us a resolve, 15.3 with three), else three (16,001
// on 99,991: 22.3 us, 23.1 with two and 25.1 with four; 65,536 on 100,000: 33.5, 90.6, 34.3).
constexpr int kGreedyGridRounds = 3;
constexpr int32_t kGreedyOneRound = 1024;

struct gsn_net {
  gsn_params p;
  DevState s;
  int32_t n;        // live units (host copy, changed only by grow/import)
  int cur;          // current CSR buffer
  int dpar;         // which per-block delta array the next lock-set edge update uses
  int wpar;         // which survivor tables the next one-pass winner-lock update uses
  int phase;
  int cus;          // compute units of the device
  int tune_split;
  int tune_variant;
  int tune_grab;    // list entries per atomic of the dynamic scan
  int tune_rebucket;  // staged find calls between rebuilds of the spatial unit order
  int stage_parity;  // which set of signal histogram and cursors the next call uses
  // the pruned search's records: which set of outer boxes the last gather wrote, whether that
  // gather saw the present positions in the present unit order, and whether growth changed the
  // units since the last update (then the next update does not gather ahead)
  int sup_parity;
  bool staged;
  bool grew;
  bool searched;     // the last find took the pruned search
  int32_t scan_left; // small finds that take the scan instead of it
  bool foreign;      // a caller recorded a staged find or an update: its graph may run at any
                     // time and rewrite the records or move the units, so each find makes its
                     // own records (the unit order stays: a recorded find has its own)
  // the order that the finds of a caller's recording share: which recording, on which stream,
  // for how many units, the finds since it was made, and their sets of counts and boxes
  unsigned long long rec_id;
  hipStream_t rec_stream;
  int32_t rec_n, rec_finds;
  int rec_hist, rec_sup;
  bool timing;
  uint32_t timing_mask;  // timers that record while timing is on (bit GSN_T_*)
  int32_t bucket_n;            // units in the spatial order (-1: none, or not these units)
  int32_t slots;               // its places: more than units after a removal
  int32_t appended;            // of these, units that joined at its end
  int32_t finds_since_bucket;  // staged finds of more than kSmallM signals since it was made
  int64_t small_signals;       // signals of the smaller ones
  int32_t small_run;           // smaller iterations since the units were last replaced or grew
  int32_t still;               // finds alone of small batches since the units last moved
  int grid_rounds;             // grid-wide rounds of the winner-lock update (0: automatic)
  int32_t* feedback;           // pinned host word: the last update's grid rounds used
  int32_t* feedback_dev;       // its device address, stored by the update's last kernel
  gsn::GrowMail* mail;         // pinned too, beside it: what growth waits for
  gsn::GrowMail* mail_dev;
  void* scratch_dev;           // device address of the no-allocation grid workspace
  std::vector<hipEvent_t> pool;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> rec[GSN_T_COUNT];
  // gsn_iterate_loop: recorded loops, the stream they are recorded on, and the recording
  // state (event timers off; the unit-order rule of the first staged find overridden)
  struct LoopGraph {
    // what the recorded launches depend on
    const float* sigs;
    int32_t m, count;
    int32_t *winner, *second;
    float *d1, *d2;
    uint8_t* accepted;
    int32_t n;
    int cur, dpar, wpar, stage_parity, sup_parity;
    bool rebuild_first, staged, grew, scan;
    int32_t slots, appended, small_run;
    int tune_split, tune_variant, tune_grab, tune_rebucket, grid_rounds;
    // the host state the loop leaves
    bool staged_after;
    int32_t slots_after, appended_after;
    int64_t small_after, small_delta;
    bool rebuilt;   // the first find rebuilt the unit order (else finds_delta counts finds)
    int cur_after, dpar_after, wpar_after, stage_parity_after, sup_parity_after;
    int32_t finds_after, finds_delta, bucket_n_after;
    hipGraphExec_t exec;
    uint64_t used;
  };
  std::vector<LoopGraph> graphs;
  uint64_t graph_clock;
  int64_t loop_records;   // loop calls that recorded a graph
  hipStream_t cap_stream;
  bool capturing;
  int loop_rebuild;   // -1, or the unit-order decision (0/1) of the next staged find
  bool loop_scan;     // its small finds take the scan
};

namespace {

bool params_ok(const gsn_params* p) {
  if (!p) return false;
  if (!(p->eps_b >= 0.0f && p->eps_b <= 1.0f)) return false;
  if (!(p->eps_n >= 0.0f && p->eps_n <= 1.0f)) return false;
  // errors stay >= +0 and only shrink under the two factors (the argmax keys rely on it)
  if (!(p->err_alpha >= 0.0f && p->err_alpha <= 1.0f)) return false;
  if (!(p->err_beta >= 0.0f && p->err_beta <= 1.0f)) return false;
  if (p->max_age < 0) return false;
  if (p->n_max < 2 || p->e_max < 0 || p->m_max < 1) return false;
  if (p->lock_mode < 0 || p->lock_mode > 2 || p->key_mode < 0 || p->key_mode > 1) return false;
  // keep every derived index inside int32
  const int64_t slack = p->lock_mode == 1 ? p->m_max : 0;
  if ((static_cast<int64_t>(p->e_max) + slack) * 2 + 2 > INT32_MAX) return false;
  if (static_cast<int64_t>(p->n_max) + 2 > INT32_MAX / 4) return false;
  if (static_cast<int64_t>(p->m_max) * 2 * gsn::kMaxSplit > INT32_MAX) return false;
  return true;
}

inline hipStream_t as_stream(void* st) { return static_cast<hipStream_t>(st); }

bool grid_ok(const gsn_grid* g, int64_t* cells) {
  if (!g) return false;
  if (!(g->h > 0.0f) || !std::isfinite(g->h)) return false;
  if (!std::isfinite(1.0f / g->h)) return false;
  int64_t c = 1;
  for (int a = 0; a < 3; ++a) {
    if (!std::isfinite(g->lo[a]) || g->dims[a] < 1) return false;
    c *= g->dims[a];
    if (c > GSN_MAX_GRID_CELLS) return false;
  }
  if (g->exact != 0 && g->exact != 1) return false;
  *cells = c;
  return true;
}

int greedy_rounds(const gsn_net* net, int32_t m) {
  if (net->grid_rounds) return net->grid_rounds;
  return m <= kGreedyOneRound ? 1 : kGreedyGridRounds;
}

inline int hip_ok(hipError_t e) { return e == hipSuccess ? GSN_OK : GSN_E_HIP; }

hipEvent_t take_event(gsn_net* net) {
  if (!net->pool.empty()) {
    hipEvent_t e = net->pool.back();
    net->pool.pop_back();
    return e;
  }
  // timing only: no system-scope fence at the record (the default one writes back and
  // invalidates the caches, which stalls the stream for several microseconds per record)
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
  return e;
}

// Records an event pair around the launches made between begin() and end().
struct TimedRegion {
  gsn_net* net;
  int which;
  hipStream_t st;
  hipEvent_t a = nullptr;
  TimedRegion(gsn_net* n, int w, hipStream_t s) : net(n), which(w), st(s) {
    if (net->timing && !net->capturing && ((net->timing_mask >> w) & 1u)) {
      a = take_event(net);
      if (a && hipEventRecord(a, st) != hipSuccess) {
        net->pool.push_back(a);
        a = nullptr;
      }
    }
  }
  void end() {
    if (!a) return;
    hipEvent_t b = take_event(net);
    if (!b) {
      net->pool.push_back(a);
      a = nullptr;
      return;
    }
    if (hipEventRecord(b, st) == hipSuccess) {
      net->rec[which].emplace_back(a, b);
    } else {
      net->pool.push_back(a);
      net->pool.push_back(b);
    }
    a = nullptr;
  }
};

// A timer whose event pair is bound to one kernel launch (gsn::LaunchEvents): the pair is
// taken from the pool when the timer records, and end() keeps it only if the launch was made.
struct LaunchTimer {
  gsn_net* net;
  int which;
  gsn::LaunchEvents ev;
  LaunchTimer(gsn_net* n, int w) : net(n), which(w) {
    if (net->timing && !net->capturing && ((net->timing_mask >> w) & 1u)) {
      ev.start = take_event(net);
      ev.stop = ev.start ? take_event(net) : nullptr;
      if (ev.start && !ev.stop) {
        net->pool.push_back(ev.start);
        ev.start = nullptr;
      }
    }
  }
  void end(bool launched) {
    if (!ev.start) return;
    if (launched) {
      net->rec[which].emplace_back(ev.start, ev.stop);
    } else {
      net->pool.push_back(ev.start);
      net->pool.push_back(ev.stop);
    }
    ev = {};
  }
};

int read_status_slot(gsn_net* net, int slot, int32_t* out, hipStream_t st) {
  if (hipMemcpyAsync(out, net->s.status + slot, sizeof(int32_t), hipMemcpyDeviceToHost, st) !=
      hipSuccess)
    return GSN_E_HIP;
  return hip_ok(hipStreamSynchronize(st));
}

int read_acc64(gsn_net* net, int slot, int64_t* out, hipStream_t st) {
  unsigned long long v = 0;
  if (hipMemcpyAsync(&v, net->s.acc64 + slot, sizeof(v), hipMemcpyDeviceToHost, st) !=
      hipSuccess)
    return GSN_E_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return GSN_E_HIP;
  *out = static_cast<int64_t>(v);
  return GSN_OK;
}

// Waits for the stream and for the words growth decides by (in net->mail afterwards).
int read_mail(gsn_net* net, hipStream_t st) {
  if (gsn::launch_grow_report(net->s, net->mail_dev, st) != hipSuccess) return GSN_E_HIP;
  return hip_ok(hipStreamSynchronize(st));
}

int insert_units(gsn_net* net, int32_t count, hipStream_t st) {
  return hip_ok(gsn::launch_insert(net->s, net->cur, net->n, count, net->p.err_alpha,
                                   net->p.n_max, 2 * static_cast<int64_t>(net->p.e_max), st));
}

// Between iterations: remove the units orphaned since the last call, then up to `count` GNG
// insertions one after another (while N < n_max).  Syncs to learn the new unit count: once
// where no unit waits to be removed, which is nearly always so (the insertion is launched
// without knowing, and does nothing if one does).
int grow_step(gsn_net* net, int32_t count, int32_t* inserted_out, hipStream_t st) {
  auto can_insert = [&]() { return count > 0 && net->n >= 1 && net->n < net->p.n_max; };
  bool tried = can_insert();
  int rc = tried ? insert_units(net, count, st) : GSN_OK;
  if (!rc) rc = read_mail(net, st);
  if (rc) return rc;
  if (net->mail->orphans > 0) {
    const bool ordered = net->bucket_n == net->n;
    const gsn::StageBufs sb = gsn::carve_stage(net->s.scr, net->p.n_max, net->p.m_max);
    if (gsn::launch_remove(net->s, net->cur, net->n, net->p.n_max, ordered ? sb.pidx : nullptr,
                           ordered ? net->slots : 0, st) != hipSuccess)
      return GSN_E_HIP;
    net->cur ^= 1;
    if ((rc = read_mail(net, st))) return rc;
    const int32_t kept = net->mail->kept;
    net->n = kept;
    // the order was renumbered with the units; many empty places are worth a new one
    net->bucket_n = ordered && net->slots - kept <= kept / 8 ? kept : -1;
    net->staged = false;
    net->grew = true;
    net->small_run = 0;
    net->still = 0;
    tried = can_insert();
    if (tried && ((rc = insert_units(net, count, st)) || (rc = read_mail(net, st)))) return rc;
  }
  const int32_t inserted = tried ? net->mail->inserted : 0;
  if (inserted) {
    const int32_t n_before = net->n;
    net->n += inserted;
    net->staged = false;
    net->grew = true;
    net->small_run = 0;
    net->still = 0;
    // new units take the next indices: they join the spatial order at its end (the
    // periodic rebucketing restores locality)
    if (net->bucket_n == n_before && net->slots + inserted <= gsn::stage_slots(net->p.n_max)) {
      const gsn::StageBufs sb = gsn::carve_stage(net->s.scr, net->p.n_max, net->p.m_max);
      if (gsn::launch_stage_append(sb, n_before, net->n, net->slots, st) != hipSuccess)
        return GSN_E_HIP;
      net->bucket_n = net->n;
      net->slots += inserted;
      net->appended += inserted;
    } else {
      net->bucket_n = -1;
    }
  }
  if (inserted_out) *inserted_out = inserted;
  return GSN_OK;
}

}  // namespace

extern "C" {

size_t gsn_workspace_bytes(const gsn_params* params) {
  if (!params_ok(params)) return 0;
  return gsn::layout_for(*params).total;
}

int gsn_create(const gsn_params* params, void* workspace, size_t workspace_bytes, int32_t n0,
               const float* init_xyz, void* stream, gsn_net** out) {
  if (!out) return GSN_E_INVAL;
  *out = nullptr;
  if (!params_ok(params) || !workspace || n0 < 0 || n0 > params->n_max) return GSN_E_INVAL;
  if (n0 > 0 && !init_xyz) return GSN_E_INVAL;
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return GSN_E_INVAL;
  if (workspace_bytes < gsn::layout_for(*params).total) return GSN_E_CAPACITY;
  gsn_net* net = new (std::nothrow) gsn_net();
  if (!net) return GSN_E_CAPACITY;
  net->p = *params;
  gsn::carve(*params, workspace, &net->s);
  net->n = n0;
  net->cur = 0;
  net->dpar = 0;
  net->wpar = 0;
  net->phase = kReady;
  net->tune_split = 0;
  net->tune_variant = 0;
  net->tune_grab = kDefaultGrab;
  net->tune_rebucket = kRebucketEvery;
  net->stage_parity = 0;
  net->sup_parity = 0;
  net->staged = false;
  net->grew = false;
  net->searched = false;
  net->scan_left = 0;
  net->foreign = false;
  net->rec_id = 0;
  net->rec_stream = nullptr;
  net->rec_n = 0;
  net->rec_finds = 0;
  net->rec_hist = 0;
  net->rec_sup = 0;
  net->timing = false;
  net->timing_mask = (1u << GSN_T_COUNT) - 1;
  net->bucket_n = -1;
  net->finds_since_bucket = 0;
  net->slots = 0;
  net->appended = 0;
  net->small_signals = 0;
  net->small_run = 0;
  net->still = 0;
  net->grid_rounds = 0;
  net->graph_clock = 0;
  net->loop_records = 0;
  net->cap_stream = nullptr;
  net->capturing = false;
  net->loop_rebuild = -1;
  net->loop_scan = false;
  net->feedback = nullptr;
  // one pinned allocation: the feedback word, then the growth mailbox
  constexpr size_t kMailAt = 64;
  if (hipHostMalloc(reinterpret_cast<void**>(&net->feedback), kMailAt + sizeof(gsn::GrowMail)) !=
      hipSuccess) {
    delete net;
    return GSN_E_HIP;
  }
  net->mail = reinterpret_cast<gsn::GrowMail*>(reinterpret_cast<char*>(net->feedback) + kMailAt);
  *net->mail = gsn::GrowMail{};
  *net->feedback = kDefaultGridRounds - 1;
  net->feedback_dev = nullptr;
  // set-up of the no-allocation entry point on this device (null if the lookup failed;
  // that entry point then tries once more and reports GSN_E_HIP)
  net->scratch_dev = noalloc_scratch();
  if (hipHostGetDevicePointer(reinterpret_cast<void**>(&net->feedback_dev), net->feedback, 0) !=
      hipSuccess) {
    gsn_destroy(net);
    return GSN_E_HIP;
  }
  net->mail_dev = reinterpret_cast<gsn::GrowMail*>(
      reinterpret_cast<char*>(net->feedback_dev) + kMailAt);
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
    net->cus = cus;
  else
    net->cus = 256;
  hipStream_t st = as_stream(stream);
  hipError_t e = gsn::launch_init(net->s, 0, n0, params->n_max, st);
  if (e == hipSuccess)
    e = gsn::launch_stage_init(gsn::carve_stage(net->s.scr, params->n_max, params->m_max),
                               params->n_max, st);
  const size_t bytes = sizeof(float) * static_cast<size_t>(n0);
  if (e == hipSuccess && n0 > 0) {
    e = hipMemcpyAsync(net->s.x, init_xyz, bytes, hipMemcpyDefault, st);
    if (e == hipSuccess)
      e = hipMemcpyAsync(net->s.y, init_xyz + n0, bytes, hipMemcpyDefault, st);
    if (e == hipSuccess)
      e = hipMemcpyAsync(net->s.z, init_xyz + 2 * static_cast<size_t>(n0), bytes,
                         hipMemcpyDefault, st);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    gsn_destroy(net);  // frees the pinned feedback word with the handle
    return GSN_E_HIP;
  }
  *out = net;
  return GSN_OK;
}

}  // extern "C"

namespace {

// Whether a staged find of m signals with this variant, or one of `count` of them in a row, is
// due to rebuild the unit order: when there is none of these units, when it has empty places and
// a scan is to use it (which reads the first n places, unlike the search), every tune_rebucket
// finds, and, for small batches, which move few units, about once for as many signals as units.
bool order_due(const gsn_net* net, int variant, int32_t m, int64_t count) {
  if (net->bucket_n != net->n) return true;
  if (variant >= 2 && variant <= 5 && net->slots != net->n) return true;
  // units appended far from their place are in the way of every signal of the search (a scan
  // visits every unit anyway)
  if (variant >= 6 && (static_cast<int64_t>(net->appended) * kAppendedPart > net->n ||
                       net->appended > kAppendedMost))
    return true;
  if (m > gsn::kSmallM) return net->finds_since_bucket + count > net->tune_rebucket;
  return net->small_signals + m * count > std::max(net->n, 64 * gsn::kSmallM);
}

// Whether the caller, not gsn_iterate_loop, records the launches on st into a graph; id (not
// null) receives which recording it is (0 if that cannot be told).
bool caller_records(const gsn_net* net, hipStream_t st, unsigned long long* id = nullptr) {
  if (net->capturing) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (cs == hipStreamCaptureStatusNone) return false;
  if (id && hipStreamGetCaptureInfo(st, &cs, id) != hipSuccess) {
    (void)hipGetLastError();
    *id = 0;
  }
  return true;
}

// Whether a find that a caller records must make the order of its recording: the launches of one
// recording on one stream run in turn at every replay, so its later finds of as many units use
// the order of the first, for as many finds as an order of the handle's would serve.
bool recorded_order_due(gsn_net* net, unsigned long long id, hipStream_t st) {
  const bool due = id == 0 || id != net->rec_id || st != net->rec_stream ||
                   net->rec_n != net->n || net->rec_finds >= net->tune_rebucket;
  if (due) {
    net->rec_id = id;
    net->rec_stream = st;
    net->rec_n = net->n;
    net->rec_finds = 0;
  }
  ++net->rec_finds;
  return due;
}

// Whether the next small finds take the scan in place of the search (a report that comes late
// only changes which one runs, never the result).
bool scan_due(gsn_net* net) {
  volatile int32_t* hard = &net->mail->hard;
  if (*hard != 0) {
    *hard = 0;
    net->scan_left = kScanRun;
  }
  return net->scan_left > 0;
}

// gsn_find_winners; with claim not null the merge of the staged scans also makes the
// lock-set claims of every signal, and *claimed says whether it did (the direct scan's
// merge does not).
int find_impl(gsn_net* net, const float* sig, int32_t m, int32_t* winner, int32_t* second,
              float* d1, float* d2, void* stream, const gsn::ClaimArgs* claim,
              bool* claimed, const int32_t** order = nullptr) {
  if (claimed) *claimed = false;
  if (order) *order = nullptr;
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kReady && net->phase != kFound) return GSN_E_STATE;
  if (net->n < 2) return GSN_E_INVAL;
  if (m > 0 && (!sig || !winner || !second || !d1 || !d2)) return GSN_E_INVAL;
  net->phase = kFound;
  if (m == 0) return GSN_OK;
  hipStream_t st = as_stream(stream);
  gsn::FindConfig cfg =
      gsn::find_config(net->n, m, net->cus, net->tune_split, net->tune_variant);
  // A small batch takes the search too where its records are at hand, or after enough finds of
  // the same positions or, in an iteration, enough iterations on the same units.
  const bool small = m <= gsn::kSmallM;
  bool may_search = cfg.variant == 6 && net->tune_variant == 0 && !net->foreign;
  if (may_search) may_search = !(net->capturing ? net->loop_scan : scan_due(net));
  if (may_search) {
    int32_t& run = claim ? net->small_run : net->still;
    run = std::min(run + 1, kSmallRun);
    if ((net->staged && net->bucket_n == net->n) || run >= kSmallRun) cfg.variant = 7;
  }
  // Recorded by the caller (not by gsn_iterate_loop, which tracks what its graph leaves): the
  // launches run later and perhaps often, so they may not rely on records or an order that
  // are in place now, and leave the handle's account of them alone: they make an order of their
  // own, in places of their own (the handle's has other units and empty places by then), at
  // each replay (once for the finds of one recording).
  unsigned long long rec_id = 0;
  bool recorded = cfg.variant != 6 && cfg.variant >= 2 && caller_records(net, st, &rec_id);
  if (recorded && may_search) {
    cfg.variant = 6;   // the scan that needs neither
    recorded = false;
  }
  if (recorded) {
    net->staged = false;
    net->foreign = true;
  }
  net->searched = cfg.variant == 7 && !net->foreign;
  if (small && net->scan_left > 0 && !net->capturing) --net->scan_left;
  TimedRegion all(net, GSN_T_FIND, st);
  hipError_t e;
  if (cfg.variant == 6) {
    // a marker pair here: binding a pair to a launch costs the host tens of microseconds,
    // which a launch-bound small batch would show in its step time
    TimedRegion scan(net, GSN_T_FIND_SCAN, st);
    e = gsn::launch_find_small_scan(net->s, net->n, sig, m, st);
    scan.end();
    if (e == hipSuccess) {
      e = gsn::launch_find_small_merge(net->s, net->n, m, winner, second, d1, d2, claim, st);
      if (claimed) *claimed = claim != nullptr;
    }
  } else if (cfg.variant >= 2) {
    gsn::StageBufs sb = gsn::carve_stage(net->s.scr, net->p.n_max, net->p.m_max);
    if (recorded) sb.pidx = sb.rpidx;
    // the unit order is rebuilt when the network changed and every kRebucketEvery calls
    bool rebucket =
        recorded ? recorded_order_due(net, rec_id, st) : order_due(net, cfg.variant, m, 1);
    if (net->loop_rebuild >= 0) {  // the first staged find of a recorded loop
      rebucket = net->loop_rebuild == 1;
      net->loop_rebuild = -1;
    }
    const int32_t slots = rebucket || recorded ? net->n : net->slots;
    const bool gather = cfg.variant == 7 && (rebucket || !net->staged);
    // successive gathers alternate between two sets of boxes (a new order leaves every set empty)
    int& sup = recorded ? net->rec_sup : net->sup_parity;
    if (gather && !rebucket) sup ^= 1;
    const int boxes = recorded ? gsn::kRecordedSet + sup : sup;
    if (cfg.variant == 7) {
      e = rebucket ? gsn::launch_stage_order(net->s, sb, net->n, net->p.n_max, st)
                   : hipSuccess;
      if (e == hipSuccess && gather) {
        e = gsn::launch_pruned_gather(
            gsn::pruned_gather_args(net->s, sb, net->n, slots, net->p.n_max, boxes), st);
        net->staged = e == hipSuccess && !net->foreign;
      }
    } else {
      int& hist = recorded ? net->rec_hist : net->stage_parity;
      e = gsn::launch_stage(net->s, sb, net->n, net->p.n_max, sig, m, rebucket,
                            recorded ? gsn::kRecordedSet + hist : hist, cfg.variant, st);
      hist ^= 1;
      if (rebucket) net->staged = false;   // a new order, gathered for the scans alone
    }
    if (!recorded) {
      if (rebucket) {
        net->bucket_n = net->n;
        net->slots = slots;
        net->finds_since_bucket = 0;
        net->small_signals = 0;
        net->appended = 0;
      }
      if (small) net->small_signals += m;
      else ++net->finds_since_bucket;
    }
    if (e == hipSuccess && cfg.variant == 7) {
      TimedRegion scan(net, GSN_T_FIND_SCAN, st);
      e = gsn::launch_pruned_search(sb, net->n, slots, net->p.n_max, boxes, sig, m, winner,
                                    second, d1, d2, claim, &net->mail_dev->hard, st);
      scan.end();
      if (claimed) *claimed = claim != nullptr;
    } else if (e == hipSuccess) {
      LaunchTimer scan(net, GSN_T_FIND_SCAN);
      e = cfg.variant == 5   ? gsn::launch_scan_f16_dyn(net->s, sb, net->n, m, cfg.split,
                                                    net->tune_grab, st, scan.ev)
          : cfg.variant == 4 ? gsn::launch_scan_f16(net->s, sb, net->n, sig, m, cfg.split, st,
                                                    scan.ev)
          : cfg.variant == 3 ? gsn::launch_scan_mfma(net->s, sb, net->n, sig, m, cfg.split, st,
                                                     scan.ev)
                             : gsn::launch_scan_screened(net->s, sb, net->n, sig, m, cfg.split,
                                                         st, scan.ev);
      scan.end(e == hipSuccess);
    }
    if (e == hipSuccess && cfg.variant != 7) {
      e = gsn::launch_stage_merge(net->s, sb, m, cfg.split, winner, second, d1, d2, claim, st);
      if (claimed) *claimed = claim != nullptr;
      if (order) *order = sb.sperm;  // the signals' spatial order of this call
    }
  } else {
    TimedRegion scan(net, GSN_T_FIND_SCAN, st);
    e = gsn::launch_find_scan(net->s, net->n, sig, m, cfg, winner, second, d1, d2, st);
    scan.end();
    if (e == hipSuccess) e = gsn::launch_find_merge(net->s, m, cfg, winner, second, d1, d2, st);
  }
  all.end();
  return hip_ok(e);
}

// Resolve, adapt and edges after a find, fused where the rule allows (the outputs and state
// of gsn_resolve_conflicts, gsn_adapt and gsn_update_edges in order).  claimed: the find's
// merge made the lock-set claims; order: the signals in the staging's spatial order, or null.
int update_impl(gsn_net* net, const float* sig, int32_t m, const int32_t* winner,
                const int32_t* second, const float* d1, uint8_t* accepted, void* stream,
                bool claimed, const int32_t* order) {
  hipStream_t st = as_stream(stream);
  const int64_t half_cap = 2 * static_cast<int64_t>(net->p.e_max);
  if (caller_records(net, st)) {   // its graph may move the units at any time
    net->staged = false;
    net->foreign = true;
  }
  // The update moves units.  Its last launch gathers them for the next search if this find took
  // the search and the next one is due to use the same units in the same order.
  const bool ahead = net->searched && net->staged && !net->grew && m > 0 &&
                     gsn::update_gathers(net->n) &&
                     (net->capturing || !order_due(net, 7, m, 1));
  net->staged = false;
  net->still = 0;
  net->grew = false;
  gsn::GatherArgs ga{};
  if (ahead)
    ga = gsn::pruned_gather_args(
        net->s, gsn::carve_stage(net->s.scr, net->p.n_max, net->p.m_max), net->n, net->slots,
        net->p.n_max, net->sup_parity ^ 1);
  const gsn::GatherArgs* gather = ahead ? &ga : nullptr;
  auto gathered = [&]() {
    if (!ahead) return;
    net->sup_parity ^= 1;
    net->staged = true;
  };
  if (net->p.lock_mode == 1) {
    if (m == 0) {
      int rc = gsn_resolve_conflicts(net, m, winner, second, d1, accepted, stream);
      if (!rc) rc = gsn_adapt(net, sig, m, winner, second, d1, accepted, stream);
      if (!rc) rc = gsn_update_edges(net, m, winner, second, accepted, stream);
      return rc;
    }
    // the resolve leaves one survivor per winner: the update in one pass, no rounds (the
    // resolve's check fills the survivor tables)
    const gsn::WinnerTables tab = gsn::winner_tables(net->s, net->wpar, net->p.n_max);
    {
      TimedRegion tr(net, GSN_T_RESOLVE, st);
      const hipError_t e = gsn::launch_resolve(net->s, net->cur, net->n, m, winner, second, d1,
                                               accepted, 1, net->p.key_mode, st, &tab,
                                               claimed);
      tr.end();
      if (e != hipSuccess) return GSN_E_HIP;
    }
    TimedRegion t(net, GSN_T_UPDATE, st);
    const gsn::WinnerStep w{sig, m, winner, second, d1, accepted, net->p.key_mode,
                            net->p.eps_b, net->p.eps_n, net->p.err_beta, net->p.max_age, 0, 0,
                            half_cap, nullptr, net->p.n_max};
    const hipError_t e =
        gsn::launch_winner_local(net->s, net->cur, net->wpar, net->n, w, st, gather);
    t.end();
    if (e != hipSuccess) return GSN_E_HIP;
    gathered();
    net->cur ^= 1;
    net->wpar ^= 1;
    net->phase = kReady;
    return GSN_OK;
  }
  // the lock sets: the fused check and update; greedy: the resolve's rounds decide, and the
  // same update applies the accepted signals (disjoint lock sets) without claims or check
  const bool greedy = net->p.lock_mode == 2;
  if (greedy && m > 0) {
    // (with claimed the find's merge made the first round's claims and the signal states)
    TimedRegion tr(net, GSN_T_RESOLVE, st);
    const hipError_t e = gsn::launch_resolve_greedy(
        net->s, net->cur, net->n, m, winner, second, d1, nullptr, net->p.key_mode,
        greedy_rounds(net, m), st, claimed);
    tr.end();
    if (e != hipSuccess) return GSN_E_HIP;
  }
  TimedRegion t(net, GSN_T_UPDATE, st);
  const hipError_t e = gsn::launch_iterate_set(
      net->s, net->cur, net->dpar, net->n, sig, m, winner, second, d1, accepted,
      net->p.key_mode, net->p.eps_b, net->p.eps_n, net->p.err_beta, net->p.max_age, half_cap,
      greedy || claimed, order, st, greedy ? net->s.pend : nullptr, gather);
  t.end();
  if (e != hipSuccess) return GSN_E_HIP;
  gathered();
  net->cur ^= 1;
  net->dpar ^= 1;
  net->phase = kReady;
  return GSN_OK;
}

}  // namespace

extern "C" {

int gsn_find_winners(gsn_net* net, const float* sig, int32_t m, int32_t* winner,
                     int32_t* second, float* d1, float* d2, void* stream) {
  return find_impl(net, sig, m, winner, second, d1, d2, stream, nullptr, nullptr);
}

size_t gsn_grid_workspace_bytes(const gsn_grid* grid, int32_t n_max, int32_t m_max) {
  int64_t cells = 0;
  if (!grid_ok(grid, &cells) || n_max < 2 || m_max < 1) return 0;
  return gsn::grid_bytes(cells, n_max, m_max);
}

}  // extern "C"

namespace {

int find_grid_impl(gsn_net* net, const gsn_grid* grid, void* grid_ws, size_t grid_ws_bytes,
                   const float* sig, int32_t m, int32_t* winner, int32_t* second, float* d1,
                   float* d2, void* stream, bool timed) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kReady && net->phase != kFound) return GSN_E_STATE;
  int64_t cells = 0;
  if (!grid_ok(grid, &cells) || !grid_ws) return GSN_E_INVAL;
  if (reinterpret_cast<uintptr_t>(grid_ws) % 256 != 0) return GSN_E_INVAL;
  if (grid_ws_bytes < gsn::grid_bytes(cells, net->p.n_max, net->p.m_max)) return GSN_E_CAPACITY;
  if (net->n < 2) return GSN_E_INVAL;
  if (m > 0 && (!sig || !winner || !second || !d1 || !d2)) return GSN_E_INVAL;
  net->phase = kFound;
  if (m == 0) return GSN_OK;
  net->searched = false;
  hipStream_t st = as_stream(stream);
  gsn::GridSpec spec{};
  for (int a = 0; a < 3; ++a) {
    spec.lo[a] = grid->lo[a];
    spec.dims[a] = grid->dims[a];
  }
  spec.inv_h = 1.0f / grid->h;
  spec.cells = cells;
  spec.exact = grid->exact;
  const gsn::GridBufs gb = gsn::carve_grid(grid_ws, cells, net->p.n_max, net->p.m_max);
  hipError_t e;
  if (timed) {
    TimedRegion t(net, GSN_T_FIND, st);
    e = gsn::launch_find_grid(net->s, gb, spec, net->n, sig, m, winner, second, d1, d2, st);
    t.end();
  } else {
    e = gsn::launch_find_grid(net->s, gb, spec, net->n, sig, m, winner, second, d1, d2, st);
  }
  return hip_ok(e);
}

}  // namespace

extern "C" {

int gsn_find_winners_grid(gsn_net* net, const gsn_grid* grid, void* grid_ws,
                          size_t grid_ws_bytes, const float* sig, int32_t m, int32_t* winner,
                          int32_t* second, float* d1, float* d2, void* stream) {
  return find_grid_impl(net, grid, grid_ws, grid_ws_bytes, sig, m, winner, second, d1, d2,
                        stream, true);
}

int gsn_find_winners_grid_noalloc(gsn_net* net, const gsn_grid* grid, const float* sig,
                                  int32_t m, int32_t* winner, int32_t* second, float* d1,
                                  float* d2, void* stream) {
  if (!net) return GSN_E_INVAL;
  int64_t cells = 0;
  if (!grid_ok(grid, &cells)) return GSN_E_INVAL;
  if (gsn::grid_bytes(cells, net->p.n_max, net->p.m_max) > GSN_NOALLOC_SCRATCH_BYTES)
    return GSN_E_CAPACITY;
  if (!net->scratch_dev) net->scratch_dev = noalloc_scratch();
  if (!net->scratch_dev) return GSN_E_HIP;
  // no event timing here: a first event record would create (allocate) an event
  return find_grid_impl(net, grid, net->scratch_dev, GSN_NOALLOC_SCRATCH_BYTES, sig, m, winner,
                        second, d1, d2, stream, false);
}

int gsn_resolve_conflicts(gsn_net* net, int32_t m, const int32_t* winner,
                          const int32_t* second, const float* d1, uint8_t* accepted,
                          void* stream) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kFound && net->phase != kResolved) return GSN_E_STATE;
  if (m > 0 && (!winner || !second || !d1 || !accepted)) return GSN_E_INVAL;
  net->phase = kResolved;
  if (m == 0) return GSN_OK;
  hipStream_t st = as_stream(stream);
  TimedRegion t(net, GSN_T_RESOLVE, st);
  hipError_t e =
      net->p.lock_mode == 2
          ? gsn::launch_resolve_greedy(net->s, net->cur, net->n, m, winner, second, d1,
                                       accepted, net->p.key_mode,
                                       greedy_rounds(net, m), st)
          : gsn::launch_resolve(net->s, net->cur, net->n, m, winner, second, d1, accepted,
                                net->p.lock_mode, net->p.key_mode, st);
  t.end();
  return hip_ok(e);
}

int gsn_adapt(gsn_net* net, const float* sig, int32_t m, const int32_t* winner,
              const int32_t* second, const float* d1, const uint8_t* accepted, void* stream) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kResolved) return GSN_E_STATE;
  if (m > 0 && (!sig || !winner || !second || !d1 || !accepted)) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  net->phase = kAdapted;
  if (caller_records(net, st)) net->foreign = true;   // its graph may move the units at any time
  net->staged = false;
  net->still = 0;
  TimedRegion t(net, GSN_T_ADAPT, st);
  hipError_t e;
  if (net->p.lock_mode == 1 && m > 0 && net->n > 0) {
    // automatic: from the grid rounds the last update could use (read from the pinned copy
    // of its count; a stale value only changes the split, never the result)
    int g = net->grid_rounds;
    if (g == 0) {
      // a quarter more than the last update could use grid-wide: the single-workgroup tail
      // is the slow part, and a recorded loop keeps this count for all its iterations while
      // the network (and the rounds its updates need) grows
      const int used = *static_cast<volatile int32_t*>(net->feedback) + 1;
      g = std::clamp(used + used / 4, 1, gsn::kMaxGridRounds);
    }
    gsn::WinnerStep w{sig, m, winner, second, d1, accepted, net->p.key_mode, net->p.eps_b,
                      net->p.eps_n, net->p.err_beta, net->p.max_age, g,
                      2 * (static_cast<int64_t>(net->p.e_max) + net->p.m_max),
                      2 * static_cast<int64_t>(net->p.e_max), net->feedback_dev};
    e = gsn::launch_winner_update(net->s, net->cur, net->n, w, st);
  } else {
    e = gsn::launch_adapt(net->s, net->cur, net->n, sig, m, winner, second, d1, accepted,
                          net->p.eps_b, net->p.eps_n, net->p.err_beta, st);
  }
  t.end();
  return hip_ok(e);
}

int gsn_update_edges(gsn_net* net, int32_t m, const int32_t* winner, const int32_t* second,
                     const uint8_t* accepted, void* stream) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kAdapted) return GSN_E_STATE;
  if (m > 0 && (!winner || !second || !accepted)) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  if (net->p.lock_mode == 1) {  // gsn_adapt has updated the edges
    net->phase = kReady;
    return GSN_OK;
  }
  TimedRegion t(net, GSN_T_EDGES, st);
  hipError_t e = gsn::launch_edges(net->s, net->cur, net->dpar, net->n, m, winner, second,
                                   accepted,
                                   net->p.max_age, 2 * static_cast<int64_t>(net->p.e_max), st,
                                   net->p.lock_mode == 2 ? net->s.extra : nullptr);
  t.end();
  if (e != hipSuccess) return GSN_E_HIP;
  net->cur ^= 1;
  net->dpar ^= 1;
  net->phase = kReady;
  return GSN_OK;
}

int gsn_iterate(gsn_net* net, const float* sig, int32_t m, int32_t* winner, int32_t* second,
                float* d1, float* d2, uint8_t* accepted, void* stream) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kReady && net->phase != kFound) return GSN_E_STATE;
  if (m > 0 && !accepted) return GSN_E_INVAL;
  // with the lock-set and winner-lock rules the find's merge makes the claims where it can
  const gsn::ClaimArgs claim{net->n, net->s.rp[net->cur], net->s.col[net->cur], net->s.lock,
                             net->s.status, net->p.key_mode, net->p.lock_mode == 1 ? 1 : 0,
                             net->p.lock_mode == 2 ? net->s.pend : nullptr};
  bool claimed = false;
  const int32_t* order = nullptr;
  const int rc = find_impl(net, sig, m, winner, second, d1, d2, stream, &claim, &claimed,
                           &order);
  if (rc) return rc;
  return update_impl(net, sig, m, winner, second, d1, accepted, stream, claimed, order);
}

int gsn_update(gsn_net* net, const float* sig, int32_t m, const int32_t* winner,
               const int32_t* second, const float* d1, uint8_t* accepted, void* stream) {
  if (!net || m < 0 || m > net->p.m_max) return GSN_E_INVAL;
  if (net->phase != kFound && net->phase != kResolved) return GSN_E_STATE;
  if (m > 0 && (!sig || !winner || !second || !d1 || !accepted)) return GSN_E_INVAL;
  return update_impl(net, sig, m, winner, second, d1, accepted, stream, false, nullptr);
}

int gsn_iterate_loop(gsn_net* net, const float* sigs, int32_t m, int32_t count,
                     int32_t* winner, int32_t* second, float* d1, float* d2,
                     uint8_t* accepted, void* stream) {
  if (!net || count < 1 || count > GSN_MAX_LOOP || m < 0 || m > net->p.m_max)
    return GSN_E_INVAL;
  if (net->phase != kReady && net->phase != kFound) return GSN_E_STATE;
  if (net->n < 2) return GSN_E_INVAL;
  if (m > 0 && (!sigs || !winner || !second || !d1 || !d2 || !accepted)) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  const bool scan = m <= gsn::kSmallM && scan_due(net);
  // the unit order is rebuilt at the first iteration if the usual rule would rebuild it
  // anywhere inside the loop (after that the usual rule applies, from a fresh count)
  const int variant =
      m > 0 ? gsn::find_config(net->n, m, net->cus, net->tune_split, net->tune_variant).variant
            : 0;
  const bool rebuild_first = order_due(net, variant, m, count);
  // (small batches decide at the first iteration whether they take the search; the iterations
  // count once, whether they are recorded now or replayed)
  const int32_t small_run0 = net->small_run;
  if (m > 0 && m <= gsn::kSmallM)
    net->small_run = std::min<int32_t>(net->small_run + count, kSmallRun);
  const int32_t small_run = net->small_run;
  using LoopGraph = gsn_net::LoopGraph;
  auto same = [&](const LoopGraph& g) {
    return g.sigs == sigs && g.m == m && g.count == count && g.winner == winner &&
           g.second == second && g.d1 == d1 && g.d2 == d2 && g.accepted == accepted &&
           g.n == net->n && g.cur == net->cur && g.dpar == net->dpar && g.wpar == net->wpar &&
           g.stage_parity == net->stage_parity && g.sup_parity == net->sup_parity &&
           g.rebuild_first == rebuild_first && g.staged == net->staged &&
           g.grew == net->grew && g.scan == scan && g.slots == net->slots &&
           g.appended == net->appended && g.small_run == small_run &&
           g.tune_split == net->tune_split && g.tune_variant == net->tune_variant &&
           g.tune_grab == net->tune_grab && g.tune_rebucket == net->tune_rebucket &&
           g.grid_rounds == net->grid_rounds;
  };
  LoopGraph* hit = nullptr;
  for (auto& g : net->graphs)
    if (same(g)) hit = &g;
  if (!hit) {
    if (!net->cap_stream &&
        hipStreamCreateWithFlags(&net->cap_stream, hipStreamNonBlocking) != hipSuccess) {
      net->cap_stream = nullptr;
      return GSN_E_HIP;
    }
    LoopGraph g{};
    g.sigs = sigs; g.m = m; g.count = count;
    g.winner = winner; g.second = second; g.d1 = d1; g.d2 = d2; g.accepted = accepted;
    g.n = net->n; g.cur = net->cur; g.dpar = net->dpar; g.wpar = net->wpar;
    g.stage_parity = net->stage_parity;
    g.sup_parity = net->sup_parity;
    g.rebuild_first = rebuild_first;
    g.staged = net->staged;
    g.grew = net->grew;
    g.scan = scan;
    g.slots = net->slots;
    g.appended = net->appended;
    g.small_run = small_run;
    g.tune_split = net->tune_split; g.tune_variant = net->tune_variant;
    g.tune_grab = net->tune_grab; g.tune_rebucket = net->tune_rebucket;
    g.grid_rounds = net->grid_rounds;
    // record the loop: the calls run on the host as usual (argument checks, state), their
    // launches go into the graph
    const int cur0 = net->cur, dpar0 = net->dpar, wpar0 = net->wpar, sp0 = net->stage_parity;
    const int up0 = net->sup_parity;
    const bool staged0 = net->staged, grew0 = net->grew, searched0 = net->searched;
    const int32_t slots0 = net->slots, appended0 = net->appended, still0 = net->still;
    const int64_t small0 = net->small_signals;
    const int phase0 = net->phase;
    const int32_t bn0 = net->bucket_n, f0 = net->finds_since_bucket;
    (void)hipGetLastError();
    if (hipStreamBeginCapture(net->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
      net->small_run = small_run0;
      return GSN_E_HIP;
    }
    net->capturing = true;
    net->loop_scan = scan;
    net->loop_rebuild = rebuild_first ? 1 : 0;
    int rc = GSN_OK;
    for (int32_t k = 0; k < count && rc == GSN_OK; ++k)
      rc = gsn_iterate(net, sigs ? sigs + 3 * static_cast<size_t>(m) * k : nullptr, m, winner,
                       second, d1, d2, accepted, net->cap_stream);
    net->capturing = false;
    // a staged find consumed the unit-order decision; other finds leave the order alone
    const bool rebuilt = rebuild_first && net->loop_rebuild == -1;
    net->loop_rebuild = -1;
    hipGraph_t graph = nullptr;
    const hipError_t ec = hipStreamEndCapture(net->cap_stream, &graph);
    hipGraphExec_t exec = nullptr;
    if (rc == GSN_OK && ec == hipSuccess && graph &&
        hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
      exec = nullptr;
    }
    if (graph) (void)hipGraphDestroy(graph);
    if (rc != GSN_OK || !exec) {
      // nothing ran: the handle is as before the call
      net->cur = cur0; net->dpar = dpar0; net->wpar = wpar0; net->stage_parity = sp0;
      net->sup_parity = up0;
      net->staged = staged0;
      net->grew = grew0;
      net->searched = searched0;
      net->slots = slots0;
      net->appended = appended0;
      net->small_signals = small0;
      net->small_run = small_run0;
      net->still = still0;
      net->phase = phase0;
      net->bucket_n = bn0; net->finds_since_bucket = f0;
      (void)hipGetLastError();
      return rc != GSN_OK ? rc : GSN_E_HIP;
    }
    g.exec = exec;
    g.rebuilt = rebuilt;
    g.cur_after = net->cur; g.dpar_after = net->dpar; g.wpar_after = net->wpar;
    g.stage_parity_after = net->stage_parity;
    g.sup_parity_after = net->sup_parity;
    g.staged_after = net->staged;
    g.slots_after = net->slots;
    g.appended_after = net->appended;
    g.small_after = net->small_signals;
    g.small_delta = net->small_signals - small0;
    g.finds_after = net->finds_since_bucket;
    g.finds_delta = net->finds_since_bucket - f0;
    g.bucket_n_after = net->bucket_n;
    // the host state is back at the start until the graph is launched below
    net->cur = cur0; net->dpar = dpar0; net->wpar = wpar0; net->stage_parity = sp0;
    net->sup_parity = up0;
    net->staged = staged0;
    net->grew = grew0;
    net->searched = searched0;
    net->slots = slots0;
    net->appended = appended0;
    net->small_signals = small0;
    net->small_run = small_run;
    net->still = still0;
    net->bucket_n = bn0; net->finds_since_bucket = f0;
    if (net->graphs.size() >= GSN_GRAPH_CACHE) {
      size_t old = 0;
      for (size_t i = 1; i < net->graphs.size(); ++i)
        if (net->graphs[i].used < net->graphs[old].used) old = i;
      (void)hipGraphExecDestroy(net->graphs[old].exec);
      net->graphs.erase(net->graphs.begin() + static_cast<std::ptrdiff_t>(old));
    }
    net->graphs.push_back(g);
    hit = &net->graphs.back();
    ++net->loop_records;
  }
  hit->used = ++net->graph_clock;
  if (hipGraphLaunch(hit->exec, st) != hipSuccess) {
    net->small_run = small_run0;
    return GSN_E_HIP;
  }
  if (scan) net->scan_left = std::max(net->scan_left - count, 0);
  net->cur = hit->cur_after;
  net->dpar = hit->dpar_after;
  net->wpar = hit->wpar_after;
  net->stage_parity = hit->stage_parity_after;
  net->sup_parity = hit->sup_parity_after;
  net->staged = hit->staged_after && !net->foreign;
  net->grew = false;
  net->still = 0;
  net->slots = hit->slots_after;
  net->appended = hit->appended_after;
  net->small_signals = hit->rebuilt ? hit->small_after : net->small_signals + hit->small_delta;
  if (hit->rebuilt) {
    net->finds_since_bucket = hit->finds_after;
    net->bucket_n = hit->bucket_n_after;
  } else {
    net->finds_since_bucket += hit->finds_delta;
  }
  net->phase = kReady;
  return GSN_OK;
}

int gsn_grow(gsn_net* net, int32_t iteration, int32_t insert_every, void* stream) {
  if (!net || insert_every < 0) return GSN_E_INVAL;
  if (net->phase != kReady) return GSN_E_STATE;
  const bool insert = insert_every > 0 && iteration > 0 && iteration % insert_every == 0;
  return grow_step(net, insert ? 1 : 0, nullptr, as_stream(stream));
}

int gsn_run_schedule(gsn_net* net, const float* cloud, int64_t n_points,
                     const gsn_schedule* sc, gsn_schedule_result* res, void* stream) {
  if (!net || !cloud || !sc || !res) return GSN_E_INVAL;
  if (n_points < 1 || n_points > static_cast<int64_t>(UINT32_MAX)) return GSN_E_INVAL;
  if (sc->m_cap < 1 || sc->m_cap > net->p.m_max || sc->fixed_m < 0 ||
      sc->fixed_m > net->p.m_max)
    return GSN_E_INVAL;
  if (sc->insert_every < 0 || sc->qe_window < 1 || sc->max_signals < 1) return GSN_E_INVAL;
  const int32_t m_big = sc->fixed_m > 0 ? sc->fixed_m : sc->m_cap;
  if (sc->qe_window + m_big > (int64_t{1} << 19)) return GSN_E_INVAL;
  if (net->phase != kReady || net->n < 2) return GSN_E_STATE;
  hipStream_t st = as_stream(stream);
  const gsn::DevState& s = net->s;
  *res = gsn_schedule_result{};
  int64_t accepted0 = 0, accepted1 = 0;
  int rc = read_acc64(net, gsn::kA64Accepted, &accepted0, st);
  if (rc) return rc;
  if (hipMemsetAsync(s.acc64 + gsn::kA64Window, 0, 8, st) != hipSuccess) return GSN_E_HIP;
  int64_t wcount = 0;
  bool have_qe = false;
  for (;;) {
    if (net->n < 2) return GSN_E_STATE;
    int32_t m = sc->fixed_m;
    if (m == 0) {
      int64_t p2 = 1;
      while (p2 <= net->n) p2 *= 2;  // the smallest power of two greater than N
      m = static_cast<int32_t>(std::min<int64_t>(p2, sc->m_cap));
    }
    if (gsn::launch_draw(cloud, n_points, sc->seed, res->signals, m, s.ssig, st) != hipSuccess)
      return GSN_E_HIP;
    if ((rc = gsn_iterate(net, s.ssig, m, s.swin, s.ssec, s.sd1, s.sd2, s.sacc, stream)))
      return rc;
    if (gsn::launch_qe(s.sd1, m, s.acc64 + gsn::kA64Window, st) != hipSuccess) return GSN_E_HIP;
    res->signals += m;
    res->iterations += 1;
    wcount += m;
    const int64_t k = sc->insert_every > 0 ? res->signals / sc->insert_every -
                                                 (res->signals - m) / sc->insert_every
                                           : 0;
    int32_t inserted = 0;
    if ((rc = grow_step(net, static_cast<int32_t>(std::min<int64_t>(k, INT32_MAX)), &inserted,
                        st)))
      return rc;
    res->inserted += inserted;
    if (wcount >= sc->qe_window) {
      // (growth's wait brought the sum of this iteration's window)
      const uint64_t sum = net->mail->window;
      if (hipMemsetAsync(s.acc64 + gsn::kA64Window, 0, 8, st) != hipSuccess) return GSN_E_HIP;
      res->qe = static_cast<double>(sum) * 0x1p-32 /
                static_cast<double>(wcount);
      have_qe = true;
      wcount = 0;
      if (res->qe < static_cast<double>(sc->qe_threshold)) {
        res->converged = 1;
        break;
      }
    }
    if (res->signals >= sc->max_signals) break;
  }
  if (!have_qe && wcount > 0) {
    res->qe = static_cast<double>(static_cast<uint64_t>(net->mail->window)) * 0x1p-32 /
              static_cast<double>(wcount);
  }
  if ((rc = read_acc64(net, gsn::kA64Accepted, &accepted1, st))) return rc;
  res->accepted = accepted1 - accepted0;
  int32_t nu = 0, ne = 0;
  if ((rc = gsn_sizes(net, &nu, &ne, stream))) return rc;
  res->n_units = nu;
  res->n_edges = ne;
  return GSN_OK;
}

int gsn_sizes(gsn_net* net, int32_t* n_units, int32_t* n_edges, void* stream) {
  if (!net) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  int32_t half = 0;
  if (hipMemcpyAsync(&half, net->s.rp[net->cur] + net->n, sizeof(int32_t),
                     hipMemcpyDeviceToHost, st) != hipSuccess)
    return GSN_E_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return GSN_E_HIP;
  if (n_units) *n_units = net->n;
  if (n_edges) *n_edges = half / 2;
  return GSN_OK;
}

int gsn_export(gsn_net* net, float* xyz, float* err, int32_t* edges, void* stream) {
  if (!net) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  const size_t n = static_cast<size_t>(net->n);
  // every copy is ordered on the caller's stream, each group followed by its sync
  auto copy = [&](void* dst, const void* src, size_t bytes) {
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDefault, st) == hipSuccess;
  };
  // the edges are listed on the device, in the adjacency buffer that is not current (the next
  // update overwrites it); the host needs their number for the copies
  int32_t half = 0;
  if (edges && !copy(&half, net->s.rp[net->cur] + n, sizeof(int32_t))) return GSN_E_HIP;
  if (edges && hipStreamSynchronize(st) != hipSuccess) return GSN_E_HIP;
  const int32_t e = std::min(half / 2, net->p.e_max);
  if (e > 0 && gsn::launch_export_edges(net->s, net->cur, net->n, e, st) != hipSuccess)
    return GSN_E_HIP;
  bool ok = true;
  if (xyz && n > 0)
    ok = copy(xyz, net->s.x, 4 * n) && copy(xyz + n, net->s.y, 4 * n) &&
         copy(xyz + 2 * n, net->s.z, 4 * n);
  if (ok && err && n > 0) ok = copy(err, net->s.err, 4 * n);
  if (ok && e > 0) {
    const size_t ne = static_cast<size_t>(e);
    const int32_t* uv = net->s.col[net->cur ^ 1];
    ok = copy(edges, uv, 8 * ne) && copy(edges + 2 * ne, net->s.age[net->cur ^ 1], 4 * ne);
  }
  return hip_ok(hipStreamSynchronize(st)) == GSN_OK && ok ? GSN_OK : GSN_E_HIP;
}

int gsn_import(gsn_net* net, int32_t n, const float* xyz, const float* err, int32_t n_edges,
               const int32_t* edges, void* stream) {
  if (!net || n < 0 || n > net->p.n_max || n_edges < 0) return GSN_E_INVAL;
  if (n_edges > net->p.e_max) return GSN_E_CAPACITY;
  if ((n > 0 && !xyz) || (n_edges > 0 && !edges)) return GSN_E_INVAL;
  hipStream_t st = as_stream(stream);
  try {
    if (hipStreamSynchronize(st) != hipSuccess) return GSN_E_HIP;
    const size_t nn = static_cast<size_t>(n), ne = static_cast<size_t>(n_edges);
    std::vector<int32_t> ed(3 * ne);
    if (ne > 0 && (hipMemcpyAsync(ed.data(), edges, 4 * 3 * ne, hipMemcpyDefault, st) !=
                       hipSuccess ||
                   hipStreamSynchronize(st) != hipSuccess))
      return GSN_E_HIP;
    std::vector<int32_t> deg(nn + 1, 0);
    for (size_t k = 0; k < ne; ++k) {
      const int32_t u = ed[k], v = ed[ne + k], a = ed[2 * ne + k];
      if (u < 0 || v < 0 || u >= n || v >= n || u == v || a < 0) return GSN_E_INVAL;
      ++deg[u];
      ++deg[v];
    }
    std::vector<int32_t> rp(nn + 1, 0);
    for (size_t u = 0; u < nn; ++u) rp[u + 1] = rp[u] + deg[u];
    std::vector<int32_t> fill(rp.begin(), rp.end() - 1);
    std::vector<std::pair<int32_t, int32_t>> half(2 * ne);
    for (size_t k = 0; k < ne; ++k) {
      const int32_t u = ed[k], v = ed[ne + k], a = ed[2 * ne + k];
      half[fill[u]++] = {v, a};
      half[fill[v]++] = {u, a};
    }
    std::vector<int32_t> col(2 * ne), age(2 * ne);
    for (size_t u = 0; u < nn; ++u) {
      std::sort(half.begin() + rp[u], half.begin() + rp[u + 1]);
      for (int32_t k = rp[u]; k < rp[u + 1]; ++k) {
        if (k > rp[u] && half[k].first == half[k - 1].first) return GSN_E_INVAL;
        col[k] = half[k].first;
        age[k] = half[k].second;
      }
    }
    // everything below is ordered on the caller's stream; the host vectors stay alive
    // until the stream synchronization at the end
    net->cur = 0;
    const DevState& s = net->s;
    bool ok = true;
    auto copy = [&](void* dst, const void* src, size_t bytes) {
      ok = ok && hipMemcpyAsync(dst, src, bytes, hipMemcpyDefault, st) == hipSuccess;
    };
    auto fill_bytes = [&](void* dst, int value, size_t bytes) {
      ok = ok && hipMemsetAsync(dst, value, bytes, st) == hipSuccess;
    };
    if (n > 0) {
      copy(s.x, xyz, 4 * nn);
      copy(s.y, xyz + nn, 4 * nn);
      copy(s.z, xyz + 2 * nn, 4 * nn);
      if (err)
        copy(s.err, err, 4 * nn);
      else
        fill_bytes(s.err, 0, 4 * nn);
    }
    copy(s.rp[0], rp.data(), 4 * (nn + 1));
    if (ne > 0) {
      copy(s.col[0], col.data(), 8 * ne);
      copy(s.age[0], age.data(), 8 * ne);
    }
    const size_t nm = static_cast<size_t>(net->p.n_max);
    fill_bytes(s.ins, 0xff, 4 * nm);
    fill_bytes(s.orphan, 0, 4 * nm);
    fill_bytes(s.lock, 0xff, 8 * nm);
    fill_bytes(s.extra, 0, 4 * nm);
    fill_bytes(s.rem, 0, 4 * gsn::kRmWords);
    fill_bytes(s.status, 0, 4 * gsn::kStSlots);
    fill_bytes(s.bdelta[0], 0, 4 * (nm / gsn::kBlock + 2));
    fill_bytes(s.bdelta[1], 0, 4 * (nm / gsn::kBlock + 2));
    if (s.wkey) {
      fill_bytes(s.wkey, 0xff, 32 * nm);
      fill_bytes(s.wflag, 0, 2 * nm);
      fill_bytes(s.rhead, 0xff, 8 * nm);
      fill_bytes(s.whi, 0, 8);
    }
    ok = ok && gsn::launch_stage_init(gsn::carve_stage(s.scr, net->p.n_max, net->p.m_max),
                                      net->p.n_max, st) == hipSuccess;
    ok = hipStreamSynchronize(st) == hipSuccess && ok;
    if (!ok) return GSN_E_HIP;
    net->n = n;
    net->dpar = 0;
    net->wpar = 0;
    net->stage_parity = 0;   // every histogram set was cleared above
    net->sup_parity = 0;     // and every set of outer boxes
    net->phase = kReady;
    net->bucket_n = -1;
    net->slots = 0;
    net->appended = 0;
    net->staged = false;
    net->grew = false;
    net->small_run = 0;
    net->still = 0;
    net->mail->hard = 0;
    net->scan_left = 0;
  } catch (const std::bad_alloc&) {
    return GSN_E_CAPACITY;
  }
  return GSN_OK;
}

int gsn_check(gsn_net* net, void* stream) {
  if (!net) return GSN_E_INVAL;
  int32_t code = 0;
  int rc = read_status_slot(net, gsn::kStError, &code, as_stream(stream));
  if (rc) return rc;
  return code;
}

void gsn_destroy(gsn_net* net) {
  if (!net) return;
  for (auto& g : net->graphs) (void)hipGraphExecDestroy(g.exec);
  if (net->cap_stream) (void)hipStreamDestroy(net->cap_stream);
  for (auto& v : net->rec)
    for (auto& pr : v) {
      (void)hipEventDestroy(pr.first);
      (void)hipEventDestroy(pr.second);
    }
  for (hipEvent_t e : net->pool) (void)hipEventDestroy(e);
  if (net->feedback) (void)hipHostFree(net->feedback);
  delete net;
}

int gsn_tune(gsn_net* net, int32_t key, int32_t value) {
  if (!net) return GSN_E_INVAL;
  switch (key) {
    case GSN_TUNE_SPLIT:
      if (value < 0 || value > GSN_MAX_SPLIT) return GSN_E_INVAL;
      net->tune_split = value;
      return GSN_OK;
    case GSN_TUNE_VARIANT:
      if (value < 0 || value > 6) return GSN_E_INVAL;
      net->tune_variant = value;
      return GSN_OK;
    case GSN_TUNE_GRAB:
      if (value < 0 || value > 1024) return GSN_E_INVAL;
      net->tune_grab = value ? value : kDefaultGrab;
      return GSN_OK;
    case GSN_TUNE_REBUCKET:
      if (value < 0 || value > 4096) return GSN_E_INVAL;
      net->tune_rebucket = value ? value : kRebucketEvery;
      return GSN_OK;
    case GSN_TUNE_GRID_ROUNDS:
      if (value < 0 || value > gsn::kMaxGridRounds) return GSN_E_INVAL;  // 0: automatic
      net->grid_rounds = value;
      return GSN_OK;
    default:
      return GSN_E_INVAL;
  }
}

int gsn_stat(gsn_net* net, int32_t key, int64_t* value, void* stream) {
  if (!net || key < 0 || key > GSN_STAT_LOOP_RECORDS) return GSN_E_INVAL;
  if (key != GSN_STAT_CLEAR && !value) return GSN_E_INVAL;
  if (key == GSN_STAT_LOOP_RECORDS) {
    *value = net->loop_records;
    return GSN_OK;
  }
  hipStream_t st = as_stream(stream);
  int32_t* slots = net->s.rem + gsn::kRmRounds;
  if (key == GSN_STAT_CLEAR) {
    net->loop_records = 0;
    const int32_t zero[3] = {0, 0, 0};
    const unsigned long long zero64[2] = {0, 0};
    if (hipMemcpyAsync(slots, zero, sizeof(zero), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(net->s.acc64 + gsn::kA64Resolved, zero64, sizeof(zero64),
                       hipMemcpyHostToDevice, st) != hipSuccess)
      return GSN_E_HIP;
    return hip_ok(hipStreamSynchronize(st));
  }
  if (key == GSN_STAT_RESOLVED)
    return read_acc64(net, gsn::kA64Resolved, value, st);
  if (key == GSN_STAT_ACCEPTED)
    return read_acc64(net, gsn::kA64Accepted, value, st);
  int32_t h[3];
  if (hipMemcpyAsync(h, slots, sizeof(h), hipMemcpyDeviceToHost, st) != hipSuccess)
    return GSN_E_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return GSN_E_HIP;
  *value = key == GSN_STAT_ROUNDS ? h[0] : key == GSN_STAT_ROUNDS_MAX ? h[1] : h[2];
  return GSN_OK;
}

int gsn_timing_enable(gsn_net* net, int32_t enable) {
  if (!net) return GSN_E_INVAL;
  net->timing = enable != 0;
  return GSN_OK;
}

int gsn_timing_select(gsn_net* net, uint32_t mask) {
  if (!net || (mask >> GSN_T_COUNT) != 0) return GSN_E_INVAL;
  net->timing_mask = mask;
  return GSN_OK;
}

int gsn_timing_read(gsn_net* net, int32_t which, double* total_ms, int32_t* launches) {
  if (!net || which < 0 || which >= GSN_T_COUNT) return GSN_E_INVAL;
  double sum = 0.0;
  int32_t cnt = 0;
  int rc = GSN_OK;
  for (auto& pr : net->rec[which]) {
    float ms = 0.0f;
    if (hipEventSynchronize(pr.second) != hipSuccess ||
        hipEventElapsedTime(&ms, pr.first, pr.second) != hipSuccess)
      rc = GSN_E_HIP;
    sum += ms;
    ++cnt;
    net->pool.push_back(pr.first);
    net->pool.push_back(pr.second);
  }
  net->rec[which].clear();
  if (total_ms) *total_ms = sum;
  if (launches) *launches = cnt;
  return rc;
}

}  // extern "C"
