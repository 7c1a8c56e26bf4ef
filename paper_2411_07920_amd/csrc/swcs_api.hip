// C ABI of libswcs: argument validation, device memory, and the host
// orchestration of the kernels in k_state / k_sigma / k_sort / k_screener.
// Declarations and the contract of every call are in include/swcs.h.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/swcs.h"
#include "conn_ops.h"
#include "gate_ops.h"
#include "rdm_ops.h"
#include "swcs_internal.h"

using namespace swcs;

namespace {

thread_local std::string g_create_error;

// Device memory routines of a context: the caller's (swcs_set_allocator)
// or, when none is set, hipMalloc / hipFree.  `cached` counts the bytes the
// library has handed back to the caller's allocator and not taken again, an
// estimate of what a caching allocator holds for it beyond hipMemGetInfo's
// free figure.
struct Allocator {
  swcs_alloc_fn alloc = nullptr;
  swcs_free_fn free = nullptr;
  void* user = nullptr;
  size_t cached = 0;
  // before an allocation fails: gives back what holds nothing, false if there is
  // nothing of the kind
  bool (*reclaim)(swcs_ctx*) = nullptr;
  swcs_ctx* ctx = nullptr;
};

// Device buffer that grows on demand (contents are not preserved on growth).
// It is freed by the routines that allocated it, even if the context's
// allocator has been replaced since.
struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  Allocator* cur = nullptr;             // allocator of the next allocation
  swcs_free_fn owner_free = nullptr;    // how p is freed (null: hipFree)
  void* owner_user = nullptr;
  Allocator* owner = nullptr;
  hipError_t ensure(size_t want) {
    if (want <= bytes && p) return hipSuccess;
    release();
    if (want == 0) want = 8;
    hipError_t e = take(want);
    if (e == hipErrorOutOfMemory && cur && cur->reclaim && cur->reclaim(cur->ctx)) e = take(want);
    return e;
  }
  hipError_t take(size_t want) {
    if (cur && cur->alloc) {
      p = cur->alloc(want, cur->user);
      if (!p) return hipErrorOutOfMemory;
      owner_free = cur->free;
      owner_user = cur->user;
      owner = cur;
      cur->cached = cur->cached > want ? cur->cached - want : 0;
    } else {
      hipError_t e = hipMalloc(&p, want);
      if (e != hipSuccess) {
        (void)hipGetLastError();  // or the next launch would report it as its own
        p = nullptr;
        return e;
      }
      owner_free = nullptr;
      owner = nullptr;
    }
    bytes = want;
    return hipSuccess;
  }
  void release() {
    if (p) {
      if (owner_free) {
        owner_free(p, owner_user);
        if (owner) owner->cached += bytes;
      } else {
        (void)hipFree(p);
      }
    }
    p = nullptr;
    bytes = 0;
    owner_free = nullptr;
    owner = nullptr;
  }
  template <class T> T* as() const { return (T*)p; }
};

// C(m, k) for m <= 64 by Pascal's rule (no intermediate overflow).
u64 binomial_u64(int m, int k) {
  if (k < 0 || k > m) return 0;
  std::vector<u64> row((size_t)m + 1, 0);
  row[0] = 1;
  for (int i = 1; i <= m; ++i)
    for (int j = std::min(i, k); j >= 1; --j) row[(size_t)j] += row[(size_t)j - 1];
  return row[(size_t)k];
}

u64 next_pow2(u64 x) {
  u64 p = 1;
  while (p < x) p <<= 1;
  return p;
}

double binom(int n, int k) {
  if (k < 0 || k > n) return 0.0;
  double r = 1.0;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

}  // namespace

struct swcs_ctx {
  int n = 0, na = 0, nb = 0, nso = 0, device = 0, num_cu = 1;
  hipStream_t stream = nullptr;
  std::string err;
  Allocator alloc;          // device memory routines (swcs_set_allocator)
  int64_t max_dets = 0;
  bool allow_regrow = true;  // false: state arrays reserved once at max_dets
  int64_t table_budget = 0;  // bytes for one sigma accumulation table (0 = from free memory)
  u64 sector = 0;
  ExcSpace exc;

  // integrals
  bool have_ints = false;
  double ecore = 0.0;
  DevBuf h, eri, eri8, J, K, fock;

  // reference and pool
  bool have_ref = false;
  u64 ref = 0;
  bool have_pool = false;
  int64_t K_pool = 0;
  std::vector<OpDesc> ops_host;
  std::vector<int32_t> pool_rows;
  DevBuf ops, opmap;  // pool rows; generator table (P, Q, R, S) -> pool index

  // state
  DevBuf keys, amps, hash, ctr, filt;
  u64 filt_bits_alloc = 0;
  DeviceState st;
  Counters hc;            // host copy of the device counters
  bool hc_valid = false;  // true while no launch may have changed them
  bool have_state = false;
  u64 peak_n = 0;

  // last ansatz (for parameter gradients)
  bool ansatz_valid = false;
  std::vector<int32_t> a_ops;           // per unitary: pool row (row 1 of a star gate)
  std::vector<double> a_theta, a_c, a_s;  // parameters; cos / sin of each unitary's angle
  std::vector<int> a_kind;              // per unitary: 0 one row, 1 overlapping generator
  std::vector<GenGate> a_gen;           // per unitary (kind 1)
  std::vector<int64_t> a_owner;         // per unitary: its parameter
  std::vector<double> a_factor;         // d(angle) / d(parameter)
  bool a_has_star = false;
  double a_eps = 0.0;
  int64_t a_ncut = 0;
  int seg = 1;
  std::vector<DevBuf> ckpt;
  DevBuf ckpt_n;      // u64 per checkpoint
  DevBuf ckpt_ptrs;   // double* per checkpoint (device table)
  std::vector<double*> ckpt_ptrs_host;  // last uploaded contents of ckpt_ptrs
  std::vector<GateDesc> gate_tab_host;  // source of the last gate-table upload
  DevBuf gate_tab;    // GateDesc per gate of the last apply call
  DevBuf gate_n_in;   // u64 per gate of the last apply call
  DevBuf gen_tab;     // GenGate and kind per gate, for adjoint replays of overlapping generators
  DevBuf gate_n_act;  // u64 per gate: stored entries the gate's operator acts on
  int64_t last_M = 0;

  // kernel timer: HIP events around every launch of one kernel
  int timer_kernel = 0;
  std::vector<hipEvent_t> ev_start, ev_stop;
  size_t ev_used = 0;

  // scratch
  DevBuf gacc, selected, ncut_state, ncut_cand, qfilt;
  DevBuf partial, partial2, sigma, mu, work, seg_states, acc_tab, gbuf, subset_buf, scalars,
      exp_keys, exp_amps, exp_tmp_k, exp_tmp_v, sort_scratch, ctr_r, occ, sel_scratch, mlp_partial, mse_partial, hp_key, hp_val, hp_tk, hp_tv, diag, join_src,
      join_w, rdm_g3, rdm_g2, rdm_vtab, rdm_part, rdm_bs, rdm_mem,
      str_rec, str_key, str_val, str_oth, str_tab;
  int sigma_method = SWCS_SIGMA_AUTO;
  int pool_method = SWCS_POOL_AUTO;
  // distinct external keys of the last whole-pool join or table pass (a density-matrix
  // pass has no count of them: the screened estimate then rests on an older state,
  // scaled by the alive entries, and corrects itself)
  double ext_count = 0.0, ext_alive = 0.0;
  // the last pool-gradient pass (swcs_pool_stats): keys the table was sized
  // for (distinct external keys after a full pass), slots, batches, passes
  double ps_keys = 0.0;
  u64 ps_slots = 0;
  int ps_batches = 0, ps_passes = 0, ps_screened = 0;
  // The state (and integrals) version, bumped by every call that may change
  // them; the diagonal elements and <psi|psi> on the device are reused while
  // they were computed for the current version.
  // rdm_declined: the version whose determinants were found too crowded for the
  // density matrix.
  u64 state_version = 1, diag_version = 0, norm_version = 0, rdm_declined = 0;

  template <class F> void for_each_buf(F&& f) {
    DevBuf* all[] = {&h, &eri, &eri8, &J, &K, &fock, &ops, &opmap, &gacc, &selected, &ncut_state, &ncut_cand, &filt, &keys, &amps, &hash, &ctr, &ckpt_n, &ckpt_ptrs,
                     &gate_tab, &gen_tab, &gate_n_in, &gate_n_act,
                     &partial, &partial2, &sigma, &mu, &work, &seg_states, &acc_tab, &gbuf,
                     &subset_buf, &scalars, &exp_keys, &exp_amps, &exp_tmp_k, &exp_tmp_v,
                     &sort_scratch, &ctr_r, &occ, &sel_scratch, &mlp_partial, &mse_partial,
                     &hp_key, &hp_val, &hp_tk, &hp_tv, &diag, &qfilt, &join_src, &join_w,
                     &rdm_g3, &rdm_g2, &rdm_vtab, &rdm_part, &rdm_bs, &rdm_mem, &str_rec, &str_key,
                     &str_val, &str_oth, &str_tab};
    for (DevBuf* b : all) f(*b);
    for (auto& b : ckpt) f(b);
  }
  // A pass that uses the density matrix's, the strings' or the adjoint's scratch is
  // under way; between passes this scratch holds nothing.
  bool matrix_busy = false, strings_busy = false, adjoint_busy = false;

  // Point every buffer's next allocation at the context's allocator.
  void bind_buffers() {
    for_each_buf([this](DevBuf& b) { b.cur = &alloc; });
  }

  ~swcs_ctx() {
    for_each_buf([](DevBuf& b) { b.release(); });
    for (hipEvent_t e : ev_start) (void)hipEventDestroy(e);
    for (hipEvent_t e : ev_stop) (void)hipEventDestroy(e);
  }
};

namespace {

int fail(swcs_ctx* c, int code, const std::string& msg) {
  c->err = msg;
  return code;
}

int hip_fail(swcs_ctx* c, hipError_t e, const char* where) {
  int code = (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) ? SWCS_E_OOM : SWCS_E_DEVICE;
  c->err = std::string(where) + ": " + hipGetErrorString(e);
  return code;
}

#define HIP_TRY(ctx, expr, where)                       \
  do {                                                  \
    hipError_t _e = (expr);                             \
    if (_e != hipSuccess) return hip_fail(ctx, _e, where); \
  } while (0)

// Event pair around a launch of the kernel selected by swcs_timer_start.
hipError_t timer_mark(swcs_ctx* c, int kid, bool start) {
  if (c->timer_kernel != kid) return hipSuccess;
  if (start) {
    if (c->ev_used == c->ev_start.size()) {
      hipEvent_t a, b;
      hipError_t e = hipEventCreate(&a);
      if (e != hipSuccess) return e;
      e = hipEventCreate(&b);
      if (e != hipSuccess) return e;
      c->ev_start.push_back(a);
      c->ev_stop.push_back(b);
    }
    return hipEventRecord(c->ev_start[c->ev_used], c->stream);
  }
  hipError_t e = hipEventRecord(c->ev_stop[c->ev_used], c->stream);
  ++c->ev_used;
  return e;
}

#define TIMED(ctx, kid, expr, where)                             \
  do {                                                           \
    HIP_TRY(ctx, timer_mark(ctx, kid, true), "timer");           \
    HIP_TRY(ctx, expr, where);                                   \
    HIP_TRY(ctx, timer_mark(ctx, kid, false), "timer");          \
  } while (0)

int grid_blocks(swcs_ctx* c, u64 work_items, int per_block) {
  u64 g = (work_items + per_block - 1) / per_block;
  u64 maxg = (u64)c->num_cu * 16;
  if (g > maxg) g = maxg;
  if (g < 1) g = 1;
  return (int)g;
}

// Grid of the tiled gate kernels: one block per tile, up to 2,048 resident
// threads per compute unit.
int gate_grid(swcs_ctx* c, u64 n_entries, int tile) {
  u64 g = (n_entries + tile - 1) / tile;
  const u64 maxg = (u64)c->num_cu * (2048 / kGateThreads);
  if (g > maxg) g = maxg;
  if (g < 1) g = 1;
  return (int)g;
}

int sigma_grid(swcs_ctx* c, u64 n) {
  u64 g = n;
  u64 maxg = (u64)c->num_cu * 32;
  if (g > maxg) g = maxg;
  if (g < 1) g = 1;
  return (int)g;
}

Ints ints_view(swcs_ctx* c) {
  Ints I;
  I.h = c->h.as<double>();
  I.eri = c->eri8.as<double>();
  I.J = c->J.as<double>();
  I.K = c->K.as<double>();
  I.ecore = c->ecore;
  I.n = c->n;
  return I;
}

Counters read_counters(swcs_ctx* c, hipError_t* e) {
  Counters h;
  std::memset(&h, 0, sizeof(h));
  *e = hipMemcpyAsync(&h, c->ctr.p, sizeof(Counters), hipMemcpyDeviceToHost, c->stream);
  if (*e == hipSuccess) *e = hipStreamSynchronize(c->stream);
  if (*e == hipSuccess) {
    c->hc = h;
    c->hc_valid = true;
  }
  return h;
}

// Counters without a round trip when nothing has changed them since the
// last read (state sizes only change in apply / set_state).
Counters get_counters(swcs_ctx* c, hipError_t* e) {
  if (c->hc_valid) {
    *e = hipSuccess;
    return c->hc;
  }
  return read_counters(c, e);
}

// Device memory the context may still claim: hipMemGetInfo's free bytes plus
// what it has given back to a caching allocator of the caller.
size_t avail_bytes(swcs_ctx* c) {
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) free_b = 0;
  return free_b + c->alloc.cached;
}

// Buffers that hold nothing from one call to the next (the external sigma
// table, hole-pair records, sort and export scratch): given back to the device
// when the state needs the memory, and allocated again on their next use.
void release_scratch(swcs_ctx* c) {
  DevBuf* bufs[] = {&c->acc_tab, &c->hp_key, &c->hp_val, &c->hp_tk, &c->hp_tv, &c->sort_scratch,
                    &c->exp_keys, &c->exp_amps, &c->exp_tmp_k, &c->exp_tmp_v, &c->qfilt, &c->join_src, &c->join_w,
                    &c->rdm_g3, &c->rdm_part, &c->rdm_mem, &c->seg_states, &c->work, &c->str_rec, &c->str_key,
                    &c->str_val, &c->str_oth, &c->str_tab};
  for (DevBuf* b : bufs) b->release();
}

// The sort-and-join pool pass keeps its records, sort buffers and source
// table between calls (they hold nothing); a table pass that sizes itself
// from free memory gives them back first when they are large, so that the
// join of a smaller state earlier does not shrink (and split into batches)
// the table of a larger one.
void release_join_scratch(swcs_ctx* c) {
  DevBuf* bufs[] = {&c->hp_key, &c->hp_tk, &c->join_src, &c->sort_scratch, &c->join_w};
  size_t held = 0;
  for (DevBuf* b : bufs) held += b->bytes;
  if (held < ((size_t)1 << 30)) return;
  for (DevBuf* b : bufs) b->release();
}

// What the density-matrix and spin-string passes keep between calls (it holds
// nothing): given back where another pass needs the room.  Returns its size.
size_t matrix_scratch(swcs_ctx* c, bool release) {
  DevBuf* bufs[] = {&c->rdm_g3, &c->rdm_part, &c->rdm_mem, &c->str_rec, &c->str_key, &c->str_val, &c->str_oth, &c->str_tab};
  size_t held = 0;
  for (DevBuf* b : bufs) {
    held += b->bytes;
    if (release) b->release();
  }
  return held;
}

// Marks a pass that is under way (swcs_ctx::*_busy).
struct Busy {
  bool& flag;
  explicit Busy(bool& f) : flag(f) { flag = true; }
  ~Busy() { flag = false; }
};

// Last resort of an allocation: the scratch of passes that are not under way.  A
// call fits where it did before such a pass had run.
bool reclaim_idle(swcs_ctx* c) {
  size_t held = 0;
  auto give = [&](bool busy, std::initializer_list<DevBuf*> bufs) {
    for (DevBuf* b : bufs) {
      if (busy) continue;
      held += b->bytes;
      b->release();
    }
  };
  give(c->matrix_busy, {&c->rdm_g3, &c->rdm_part, &c->rdm_mem});
  give(c->strings_busy, {&c->str_rec, &c->str_key, &c->str_val, &c->str_oth, &c->str_tab});
  give(c->adjoint_busy, {&c->seg_states, &c->work});
  return held > 0;
}

// Whether the whole-pool join is taken for a state of `alive` entries: a
// forced join always, AUTO up to kJoinAutoMaxRecords records.
bool join_fits_state(swcs_ctx* c, u64 alive) {
  if (c->pool_method == SWCS_POOL_TABLE) return false;
  if (c->pool_method == SWCS_POOL_JOIN) return true;
  return alive * (u64)(c->exc.total + 1) <= kJoinAutoMaxRecords;
}

// Budget for a table sized from free memory: 40 % of what is free (blocks
// cached by the allocator included) plus the table's own allocation.  The
// join's scratch is given back first only when a table of `need` bytes would
// not fit that budget otherwise, and the density matrix's and the strings' when
// it still does not and they are an eighth of the rest: giving them back on every
// call makes a caching allocator split and regrow its blocks from one call to the
// next.
double free_table_budget(swcs_ctx* c, double need) {
  auto budget = [&]() {
    return std::max<double>(64.0 * 1024 * 1024, 0.4 * (double)(avail_bytes(c) + c->acc_tab.bytes));
  };
  double b = budget();
  if (need > b) {
    release_join_scratch(c);
    b = budget();
  }
  if (need > b && 8 * matrix_scratch(c, false) >= avail_bytes(c)) {
    (void)matrix_scratch(c, true);
    b = budget();
  }
  return b;
}

u64 max_capacity(swcs_ctx* c) {
  u64 cap = c->sector;
  if (c->max_dets > 0 && (u64)c->max_dets < cap) cap = (u64)c->max_dets;
  if (c->max_dets <= 0) {
    u64 lim = (u64)(avail_bytes(c) / 96);  // keys + amps + 2 hash slots + headroom
    if (lim < cap) cap = lim;
  }
  if (cap < 16) cap = 16;
  return cap;
}

// Capacity of the state arrays when they may not be regrown: the configured
// maximum (never more than the sector).
u64 fixed_capacity(swcs_ctx* c) {
  return std::max<u64>(16, std::min<u64>(c->sector, (u64)c->max_dets));
}

// (Re)allocate the state arrays with capacity `cap`, preserving the first
// n_keep entries, and rebuild the hash index.  Without room for keys and
// amplitudes the old arrays stay; without room for the index or the filter
// behind them (the old index goes first, it is the largest block) there is no
// state, and the next call that sets one allocates all of it.
int state_reserve(swcs_ctx* c, u64 cap, u64 n_keep) {
  const u64 hslots = next_pow2(2 * cap);
  DevBuf nk, na;
  nk.cur = &c->alloc;
  na.cur = &c->alloc;
  HIP_TRY(c, nk.ensure(cap * sizeof(u64)), "alloc keys");
  hipError_t e = na.ensure(cap * sizeof(double));
  if (e == hipSuccess && n_keep > 0) {
    e = hipMemcpyAsync(nk.p, c->keys.p, n_keep * sizeof(u64), hipMemcpyDeviceToDevice, c->stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync(na.p, c->amps.p, n_keep * sizeof(double), hipMemcpyDeviceToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  }
  if (e != hipSuccess) {
    nk.release();
    na.release();
    return hip_fail(c, e, "alloc amps");
  }
  c->keys.release();
  c->amps.release();
  c->keys = nk;
  c->amps = na;
  nk.p = nullptr;
  na.p = nullptr;
  const bool had_state = c->have_state;
  c->have_state = false;
  c->ansatz_valid = false;
  c->st.cap = 0;
  if (c->hash.bytes < hslots * sizeof(HashSlot)) {
    c->hash.release();
    HIP_TRY(c, c->hash.ensure(hslots * sizeof(HashSlot)), "alloc hash");
  }
  const u64 fbits = next_pow2(std::max<u64>(4096, 16 * cap));
  HIP_TRY(c, c->filt.ensure(fbits / 8), "alloc filter");
  c->filt_bits_alloc = fbits;
  c->st.keys = c->keys.as<u64>();
  c->st.amps = c->amps.as<double>();
  c->st.hash = c->hash.as<HashSlot>();
  c->st.hmask = hslots - 1;
  c->st.filt = c->filt.as<unsigned>();
  c->st.fmask = fbits - 1;
  c->st.ctr = c->ctr.as<Counters>();
  HIP_TRY(c, launch_hash_clear(c->st.hash, hslots, c->stream), "hash clear");
  if (n_keep > 0) HIP_TRY(c, launch_hash_build(c->st, n_keep, c->stream), "hash build");
  c->st.cap = cap;
  c->have_state = had_state && n_keep > 0;
  return SWCS_OK;
}

// Presence filter of the alive keys, about 16 bits per key (bounded by the
// allocation) so that it stays cache-resident.
int build_filter(swcs_ctx* c, u64 n, u64 alive) {
  const u64 want = next_pow2(std::max<u64>(4096, 16 * alive));
  c->st.fmask = std::min<u64>(want, c->filt_bits_alloc) - 1;
  HIP_TRY(c, launch_filter_build(c->st, n, grid_blocks(c, n, 256), c->stream), "filter");
  return SWCS_OK;
}

// Rebuild of the state without its pruned entries (tombstones): the alive
// entries are moved, in storage order, to the front of the arrays and the
// index is rebuilt over them.  Storage positions change, so a gate record
// that refers to them (the checkpoints of a chain applied from the
// reference) no longer matches the state: callers compact only states that
// carry no such record, or drop it.  *h is updated to the new counters.
int state_compact(swcs_ctx* c, Counters* h) {
  const u64 n = h->n, alive = h->alive;
  if (alive >= n) return SWCS_OK;
  HIP_TRY(c, c->exp_keys.ensure(std::max<u64>(1, alive) * 8), "alloc");
  HIP_TRY(c, c->exp_amps.ensure(std::max<u64>(1, alive) * 8), "alloc");
  const u64 scr = compact_scratch_elems(n);
  HIP_TRY(c, c->sort_scratch.ensure(scr * 8), "alloc");
  HIP_TRY(c, launch_compact_alive(c->st, n, nullptr, c->exp_keys.as<u64>(), c->exp_amps.as<double>(),
                                  c->scalars.as<u64>() + 8, c->sort_scratch.as<u64>(), scr, c->stream), "compact");
  if (alive > 0) {
    HIP_TRY(c, hipMemcpyAsync(c->st.keys, c->exp_keys.p, alive * 8, hipMemcpyDeviceToDevice, c->stream), "copy keys");
    HIP_TRY(c, hipMemcpyAsync(c->st.amps, c->exp_amps.p, alive * 8, hipMemcpyDeviceToDevice, c->stream), "copy amps");
  }
  HIP_TRY(c, launch_hash_clear(c->st.hash, c->st.hmask + 1, c->stream), "hash clear");
  if (alive > 0) HIP_TRY(c, launch_hash_build(c->st, alive, c->stream), "hash build");
  h->n = alive;
  HIP_TRY(c, launch_store_counters(c->st.ctr, *h, c->stream), "counters");
  c->hc = *h;
  c->hc_valid = true;
  ++c->state_version;
  return SWCS_OK;
}

// Tombstones are reclaimed once they outnumber the alive entries (and are
// at least kCompactMin), so a scan over the stored entries costs at most
// twice one over the alive ones.
constexpr u64 kCompactMin = 4096;
bool compact_due(const Counters& h) {
  const u64 dead = h.n - h.alive;
  return dead >= kCompactMin && dead > h.alive;
}

// Whether a chain of M gates starts in the single-workgroup kernel.  The arrays
// have to hold what it may write back: the LDS capacity, or a whole sector smaller
// than that (12 spin-orbitals: 225 determinants, 30 gates 163 us in HBM, 32 here).
bool chain_in_lds(swcs_ctx* c, u64 n_start, int64_t M) {
  return M > 0 && n_start <= (u64)lds_chain_capacity() &&
         c->st.cap >= std::min((u64)lds_chain_capacity(), c->sector) && M <= (int64_t)1 << 30;
}

// Reset the state to the single reference determinant, for a chain of M gates.
int state_reset_to_reference(swcs_ctx* c, int64_t M) {
  u64 cap;
  if (!c->allow_regrow) {
    cap = fixed_capacity(c);
  } else {
    cap = next_pow2(std::max<u64>(4096, 4 * c->peak_n));
    if (cap > c->st.cap && cap > max_capacity(c)) release_scratch(c);
    cap = std::min<u64>(cap, max_capacity(c));
  }
  if (cap < 2) cap = 2;
  if (!c->keys.p || c->st.cap != cap) {
    int r = state_reserve(c, cap, 0);
    if (r) return r;
  } else if (!chain_in_lds(c, 1, M)) {
    HIP_TRY(c, launch_hash_clear(c->st.hash, c->st.hmask + 1, c->stream), "hash clear");
  }
  HIP_TRY(c, launch_reset_reference(c->st, c->ref, c->stream), "reset");
  // the single-workgroup kernel has an index of its own, and this one is built
  // from its result
  if (!chain_in_lds(c, 1, M)) HIP_TRY(c, launch_hash_build(c->st, 1, c->stream), "hash build");
  std::memset(&c->hc, 0, sizeof(c->hc));
  c->hc.n = 1;
  c->hc.alive = 1;
  c->hc_valid = true;
  c->have_state = true;
  return SWCS_OK;
}

int check_ready(swcs_ctx* c) {
  if (!c->have_ints) return fail(c, SWCS_E_STATE, "integrals not set");
  if (!c->have_ref) return fail(c, SWCS_E_STATE, "reference not set");
  if (!c->have_pool) return fail(c, SWCS_E_STATE, "pool not set");
  return SWCS_OK;
}

int validate_gates(swcs_ctx* c, const int32_t* op_idx, const double* theta, int64_t M, double eps,
                   int64_t ncut) {
  if (M < 0) return fail(c, SWCS_E_INVALID, "M < 0");
  if (M > 0 && (!op_idx || !theta)) return fail(c, SWCS_E_INVALID, "null op_idx/theta");
  if (!(eps >= 0.0) || !std::isfinite(eps)) return fail(c, SWCS_E_INVALID, "eps must be finite and >= 0");
  if (ncut < 0) return fail(c, SWCS_E_INVALID, "ncut < 0");
  if (ncut > 0x7fffffffLL) return fail(c, SWCS_E_INVALID, "ncut too large");
  for (int64_t i = 0; i < M; ++i) {
    if (op_idx[i] < 0 || op_idx[i] >= c->K_pool) return fail(c, SWCS_E_INVALID, "op index out of range");
    if (!std::isfinite(theta[i])) return fail(c, SWCS_E_INVALID, "non-finite theta");
  }
  return SWCS_OK;
}

// Upload the checkpoint pointer table (device array of double*).
int upload_ckpt_table(swcs_ctx* c, int nck) {
  std::vector<double*> ptrs((size_t)nck);
  for (int j = 0; j < nck; ++j) ptrs[(size_t)j] = c->ckpt[(size_t)j].as<double>();
  if (ptrs == c->ckpt_ptrs_host && c->ckpt_ptrs.bytes >= (size_t)nck * sizeof(double*))
    return SWCS_OK;  // device table already current
  // The previous upload may still be reading the host copy: wait for it.
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  c->ckpt_ptrs_host = ptrs;
  HIP_TRY(c, c->ckpt_ptrs.ensure((size_t)nck * sizeof(double*)), "alloc ckpt table");
  HIP_TRY(c, hipMemcpyAsync(c->ckpt_ptrs.p, c->ckpt_ptrs_host.data(), (size_t)nck * sizeof(double*),
                            hipMemcpyHostToDevice, c->stream), "copy ckpt table");
  return SWCS_OK;
}

// Buffers of the N_CUT selection for `states` arrays of at most n entries; the
// select states are zeroed.
int ncut_reserve(swcs_ctx* c, int states, u64 n) {
  HIP_TRY(c, c->ncut_state.ensure((size_t)states * ncut_select_bytes()), "alloc ncut state");
  HIP_TRY(c, c->ncut_cand.ensure((size_t)states * n * 4), "alloc ncut candidates");
  HIP_TRY(c, launch_fill_u32(c->ncut_state.p, 0u, (u64)states * ncut_select_bytes() / 4, c->stream), "zero ncut state");
  return SWCS_OK;
}

// Generators and kinds of a chain with overlapping generators, in device memory.
int upload_generators(swcs_ctx* c, const GenGate* gen, const int* kind, int64_t M, const GenGate** d_gens,
                      const int** d_kinds) {
  HIP_TRY(c, c->gen_tab.ensure((size_t)M * (sizeof(GenGate) + sizeof(int))), "alloc generator table");
  int* kinds = (int*)((char*)c->gen_tab.p + (size_t)M * sizeof(GenGate));
  HIP_TRY(c, hipMemcpyAsync(c->gen_tab.p, gen, (size_t)M * sizeof(GenGate), hipMemcpyHostToDevice, c->stream),
          "copy generators");
  HIP_TRY(c, hipMemcpyAsync(kinds, kind, (size_t)M * sizeof(int), hipMemcpyHostToDevice, c->stream), "copy generators");
  *d_gens = c->gen_tab.as<GenGate>();
  *d_kinds = kinds;
  return SWCS_OK;
}

// Apply gates [0, M) of (ops, c, s) to the current state, with checkpoints
// every `seg` gates when ckpt is requested.  A state that starts with at
// most lds_chain_capacity() entries runs in one single-workgroup launch
// (LDS-resident) for as long as it fits; the rest runs one multi-block
// launch per gate in HBM, growing the arrays when a gate would not fit.
int run_chain(swcs_ctx* c, const int32_t* op_idx, const double* cs, const double* sn, int64_t M,
              double eps, unsigned ncut, bool ckpt, u64 n_start, Counters* out,
              const int* kind = nullptr, const GenGate* gen = nullptr) {
  bool has_star = false;
  for (int64_t g = 0; kind && g < M; ++g) has_star |= kind[g] != 0;
  // With N_CUT the gates keep everything and the selection prunes.
  if (ncut) eps = 0.0;
  int64_t g0 = 0;
  c->hc_valid = false;
  if (M == 0) {
    hipError_t e;
    *out = read_counters(c, &e);
    if (e != hipSuccess) return hip_fail(c, e, "read counters");
    return SWCS_OK;
  }
  // The previous upload from gate_tab_host must be complete before it is
  // rewritten.
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  std::vector<GateDesc>& gt = c->gate_tab_host;
  gt.resize((size_t)M);
  for (int64_t g = 0; g < M; ++g) {
    gt[(size_t)g].op = c->ops_host[op_idx[g]];
    gt[(size_t)g].c = cs[g];
    gt[(size_t)g].s = sn[g];
  }
  HIP_TRY(c, c->gate_tab.ensure((size_t)M * sizeof(GateDesc)), "alloc gate table");
  HIP_TRY(c, hipMemcpyAsync(c->gate_tab.p, gt.data(), (size_t)M * sizeof(GateDesc),
                            hipMemcpyHostToDevice, c->stream), "copy gate table");
  if (ckpt) {
    const int nck = (int)((M + c->seg - 1) / c->seg);
    for (int j = 0; j < nck; ++j)
      HIP_TRY(c, c->ckpt[(size_t)j].ensure(c->st.cap * sizeof(double)), "alloc checkpoint");
    int r = upload_ckpt_table(c, nck);
    if (r) return r;
  }
  const GenGate* gens = nullptr;
  const int* kinds = nullptr;
  if (has_star) {
    int r = upload_generators(c, gen, kind, M, &gens, &kinds);
    if (r) return r;
  }
  if (chain_in_lds(c, n_start, M)) {
    // counted where the chain would run in HBM but for its small sector or its
    // overlapping generators
    const bool count = has_star || c->st.cap < (u64)lds_chain_capacity();
    TIMED(c, SWCS_K_CHAIN_LDS, launch_chain_lds(c->st, c->gate_tab.as<GateDesc>(), kinds, gens, 0, (int)M, eps, eps > 0.0 ? 1 : 0,
                                ckpt ? c->ckpt_ptrs.as<double*>() : nullptr, c->ckpt_n.as<u64>(),
                                c->seg, c->gate_n_in.as<u64>(), count ? c->gate_n_act.as<u64>() : nullptr, c->sector, ncut,
                                c->stream), "chain");
    HIP_TRY(c, launch_hash_clear(c->st.hash, c->st.hmask + 1, c->stream), "hash clear");
    HIP_TRY(c, launch_hash_build_dev(c->st, grid_blocks(c, lds_chain_capacity(), 256), c->stream), "hash build");
    hipError_t e;
    Counters h = read_counters(c, &e);
    if (e != hipSuccess) return hip_fail(c, e, "read counters");
    if (!(h.flags & kFlagStopped)) {
      *out = h;
      return SWCS_OK;
    }
    // Continue in HBM from the gate that did not fit in LDS.
    g0 = (int64_t)h.stop_gate;
    h.flags &= ~kFlagStopped;
    h.stop_gate = 0;
    HIP_TRY(c, launch_store_counters(c->st.ctr, h, c->stream), "counters");
  }
  // From its first gate on, a chain that cannot be brought to its end leaves no
  // state: the counts of gates under way are in the rotating slots, and the
  // filter is built behind the last gate.
  bool begun = g0 > 0;
  auto part_way = [&](int r) {
    if (begun) c->have_state = false;
    return r;
  };
  // A checkpoint is allocated ahead of its gate, while the gates before it run
  // (in a new context these allocations are a tenth of the chain's time).
  auto enqueue = [&]() -> int {
    if (ncut) {
      int r = ncut_reserve(c, 1, c->st.cap);
      if (r) return r;
    }
    HIP_TRY(c, launch_live_begin(c->st, (unsigned)g0, c->stream), "counters");
    for (int64_t g = g0; g < M; ++g) {
      if (ckpt && g % c->seg == 0) {
        const int j = (int)(g / c->seg);
        HIP_TRY(c, c->ckpt[j].ensure(c->st.cap * sizeof(double)), "alloc checkpoint");
        HIP_TRY(c, launch_ckpt_save(c->st, (unsigned)g, c->ckpt[j].as<double>(), c->ckpt_n.as<u64>() + j,
                                    grid_blocks(c, c->st.cap / 4, 256), c->stream), "checkpoint");
      }
      begun = true;
      const OpDesc& op = c->ops_host[op_idx[g]];
      if (kind && kind[g])
        HIP_TRY(c, launch_gen_gate(c->st, gen[g], eps, c->gate_n_in.as<u64>() + g, (unsigned)g, c->sector,
                                   grid_blocks(c, c->st.cap / 2, 256), c->stream, c->gate_n_act.as<u64>() + g),
                "generator gate");
      else
        TIMED(c, SWCS_K_GATE, launch_gate(c->st, op, cs[g], sn[g], eps, c->gate_n_in.as<u64>() + g,
                               (unsigned)g, c->sector, gate_grid(c, c->st.cap / 2, gate_scan_tile(c->st.cap)), c->stream,
                               c->gate_n_act.as<u64>() + g),
                "gate");
      // The gates only test the entries they touch; entries of a starting
      // state that were never tested against eps are pruned once, after the
      // first gate, so every later state is exactly P(U psi).
      if (g == 0 && eps > 0.0)
        HIP_TRY(c, launch_prune_all(c->st, eps, (unsigned)g, grid_blocks(c, c->st.cap / 2, 256), c->stream), "prune");
      if (ncut)
        HIP_TRY(c, launch_ncut(c->st.amps, 0, c->st.keys, 0, c->st.ctr, (unsigned)g, c->st.cap, c->ncut_state.p, c->ncut_cand.as<unsigned>(), 0,
                               ncut, c->st.cap, 1, c->stream), "ncut");
    }
    HIP_TRY(c, launch_live_end(c->st, (unsigned)M, c->stream), "counters");
    return SWCS_OK;
  };
  for (int attempt = 0; attempt < 64; ++attempt) {
    int r = enqueue();
    if (r) return part_way(r);
    hipError_t e;
    Counters h = read_counters(c, &e);
    if (e != hipSuccess) return part_way(hip_fail(c, e, "read counters"));
    if (h.flags & kFlagOverflow) {
      h.flags &= ~(kFlagOverflow | kFlagStopped);
      HIP_TRY(c, launch_store_counters(c->st.ctr, h, c->stream), "counters");
      c->hc_valid = false;
      return part_way(fail(c, SWCS_E_DEVICE, "internal overflow in gate chain"));
    }
    if (!(h.flags & kFlagStopped)) {
      // a chain without checkpoints leaves no record of storage positions
      if (!ckpt && compact_due(h)) {
        r = state_compact(c, &h);
        if (r) return part_way(r);
      }
      *out = h;
      return SWCS_OK;
    }
    g0 = (int64_t)h.stop_gate;
    h.flags &= ~kFlagStopped;
    h.stop_gate = 0;
    // A stopped gate changed nothing.  Without checkpoints, tombstones are
    // reclaimed first when they are a quarter of the alive entries or more,
    // and the arrays grow only if the gate still does not fit.
    const bool star_stop = kind && kind[g0];
    if (!ckpt && h.n - h.alive >= kCompactMin && 4 * (h.n - h.alive) >= h.alive) {
      r = state_compact(c, &h);
      if (r) return part_way(r);
      const u64 room = c->sector > h.n ? c->sector - h.n : 0;
      const u64 grow_c = star_stop ? 2 * h.alive : h.alive;
      if (h.n + std::min<u64>(grow_c, room) <= c->st.cap) continue;
    }
    HIP_TRY(c, launch_store_counters(c->st.ctr, h, c->stream), "counters");
    if (!c->allow_regrow) {
      c->have_state = false;  // the chain stopped part way
      return fail(c, SWCS_E_CAPACITY, "state exceeds the fixed capacity (regrowth disabled)");
    }
    // Grow so that the stopped gate (and a few more) fit, then resume (a star
    // gate appends up to two entries per alive one).
    const u64 grow = star_stop ? 2 * h.alive : h.alive;
    const u64 need = h.n + std::min<u64>(grow, c->sector > h.n ? c->sector - h.n : 0);
    u64 cap = next_pow2(std::max<u64>(2 * c->st.cap, 2 * need));
    u64 maxc = max_capacity(c);
    if (maxc < cap) {
      release_scratch(c);
      maxc = max_capacity(c);
    }
    if (cap > maxc) cap = maxc;
    if (cap < need) return fail(c, SWCS_E_CAPACITY, "state exceeds the maximum capacity");
    r = state_reserve(c, cap, h.n);
    if (r) return part_way(r);
    // Checkpoint of the gate where the chain resumes was skipped if it lies
    // on a segment boundary: the loop above re-enqueues it.
  }
  return part_way(fail(c, SWCS_E_CAPACITY, "capacity growth did not converge"));
}

}  // namespace

// ---- energy without allocation ----
// Scratch of the allocation-free energy: the library's own device array,
// 32 MiB on every device the library runs on, held until the process ends.
// Layout in doubles: 2 x 8,192 per-block partial sums, 64 result slots, then
// the diagonal elements and sigma_P of up to kNoAllocMaxEntries stored
// entries.  Host code never passes `scratch` itself to a kernel: it resolves
// the array's device address once per device (noalloc_scratch).
constexpr size_t kNoAllocBytes = (size_t)32 << 20;
constexpr size_t kNoAllocPartials = 2 * 8192;
constexpr size_t kNoAllocHead = kNoAllocPartials + 64;
constexpr u64 kNoAllocMaxEntries = (kNoAllocBytes / 8 - kNoAllocHead) / 2;

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_dev[64] = {};  // device address of `scratch` per device index

// Device address of `scratch` on the context's device (which must be
// current), resolved on the first call for that device.
hipError_t noalloc_scratch(int device, double** out) {
  if (device < 0 || device >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_dev[device] = p;
  }
  *out = (double*)g_scratch_dev[device];
  return hipSuccess;
}
}  // namespace

extern "C" {

const char* swcs_version(void) { return "swcs-mi355x 0.1 (gfx950)"; }

int swcs_create(int n_spatial, int n_alpha, int n_beta, int device, swcs_ctx** out) {
  if (!out) {
    g_create_error = "out is NULL";
    return SWCS_E_INVALID;
  }
  *out = nullptr;
  if (n_spatial < 1 || 2 * n_spatial > 64 || n_alpha < 0 || n_beta < 0 || n_alpha > n_spatial ||
      n_beta > n_spatial || n_alpha + n_beta < 1) {
    g_create_error = "invalid orbital / electron counts (need 1 <= 2n <= 64, 0 <= n_a, n_b <= n)";
    return SWCS_E_INVALID;
  }
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count < 1) {
    g_create_error = "no HIP device available";
    return SWCS_E_UNSUPPORTED;
  }
  if (device < 0 || device >= count) {
    g_create_error = "device index out of range";
    return SWCS_E_INVALID;
  }
  if (hipSetDevice(device) != hipSuccess) {
    g_create_error = "hipSetDevice failed";
    return SWCS_E_DEVICE;
  }
  swcs_ctx* c = new swcs_ctx;
  c->n = n_spatial;
  c->na = n_alpha;
  c->nb = n_beta;
  c->nso = 2 * n_spatial;
  c->device = device;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) == hipSuccess) c->num_cu = prop.multiProcessorCount;
  double sec = binom(n_spatial, n_alpha) * binom(n_spatial, n_beta);
  c->sector = sec > 1e18 ? (u64)1e18 : (u64)sec;
  c->exc = make_exc_space(n_spatial, n_alpha, n_beta);
  c->alloc.reclaim = reclaim_idle;
  c->alloc.ctx = c;
  c->bind_buffers();
  if (c->ctr.ensure(sizeof(Counters)) != hipSuccess || c->scalars.ensure(64 * sizeof(double)) != hipSuccess) {
    g_create_error = "device allocation failed";
    delete c;
    return SWCS_E_OOM;
  }
  if (hipMemset(c->ctr.p, 0, sizeof(Counters)) != hipSuccess) {
    g_create_error = "device memset failed";
    delete c;
    return SWCS_E_DEVICE;
  }
  c->st.ctr = c->ctr.as<Counters>();
  // device address of the allocation-free energy's scratch, once per device
  // (a failure here is reported by that entry point, which retries)
  double* scr = nullptr;
  (void)noalloc_scratch(device, &scr);
  *out = c;
  return SWCS_OK;
}

void swcs_destroy(swcs_ctx* ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  else (void)hipDeviceSynchronize();
  delete ctx;
}

const char* swcs_last_error(const swcs_ctx* ctx) {
  if (!ctx) return g_create_error.c_str();
  return ctx->err.c_str();
}

int swcs_set_stream(swcs_ctx* c, void* hip_stream) {
  if (!c) return SWCS_E_INVALID;
  ++c->state_version;  // cached device results belong to the old stream's order
  c->stream = (hipStream_t)hip_stream;
  return SWCS_OK;
}

int swcs_set_capacity(swcs_ctx* c, int64_t max_dets, int allow_regrow) {
  if (!c) return SWCS_E_INVALID;
  if (max_dets < 0) return fail(c, SWCS_E_INVALID, "max_dets < 0");
  if (!allow_regrow && max_dets == 0) return fail(c, SWCS_E_INVALID, "a fixed capacity needs max_dets > 0");
  c->max_dets = max_dets;
  c->allow_regrow = allow_regrow != 0;
  return SWCS_OK;
}

int swcs_set_allocator(swcs_ctx* c, swcs_alloc_fn alloc_fn, swcs_free_fn free_fn, void* user) {
  if (!c) return SWCS_E_INVALID;
  if ((alloc_fn == nullptr) != (free_fn == nullptr))
    return fail(c, SWCS_E_INVALID, "alloc_fn and free_fn must both be set or both be NULL");
  c->alloc.alloc = alloc_fn;
  c->alloc.free = free_fn;
  c->alloc.user = user;
  c->alloc.cached = 0;
  return SWCS_OK;
}

int swcs_set_table_budget(swcs_ctx* c, int64_t bytes) {
  if (!c) return SWCS_E_INVALID;
  if (bytes < 0) return fail(c, SWCS_E_INVALID, "bytes < 0");
  if (bytes > 0 && bytes < 4096) return fail(c, SWCS_E_INVALID, "table budget below 4096 bytes");
  c->table_budget = bytes;
  return SWCS_OK;
}

int swcs_set_sigma_method(swcs_ctx* c, int method) {
  if (!c) return SWCS_E_INVALID;
  if (method != SWCS_SIGMA_AUTO && method != SWCS_SIGMA_ENUMERATE && method != SWCS_SIGMA_HOLE_PAIRS &&
      method != SWCS_SIGMA_PAIRS)
    return fail(c, SWCS_E_INVALID, "unknown sigma method");
  c->sigma_method = method;
  return SWCS_OK;
}

int swcs_set_pool_method(swcs_ctx* c, int method) {
  if (!c) return SWCS_E_INVALID;
  if (method != SWCS_POOL_AUTO && method != SWCS_POOL_TABLE && method != SWCS_POOL_JOIN)
    return fail(c, SWCS_E_INVALID, "unknown pool method");
  c->pool_method = method;
  return SWCS_OK;
}

int swcs_set_integrals(swcs_ctx* c, const double* h, const double* eri, double e_core) {
  if (!c) return SWCS_E_INVALID;
  ++c->state_version;
  if (!h || !eri) return fail(c, SWCS_E_INVALID, "null integrals");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  const int n = c->n;
  const size_t n2 = (size_t)n * n, n4 = n2 * n2;
  if (!std::isfinite(e_core)) return fail(c, SWCS_E_INVALID, "non-finite e_core");
  for (size_t i = 0; i < n2; ++i)
    if (!std::isfinite(h[i])) return fail(c, SWCS_E_INVALID, "non-finite h");
  for (size_t i = 0; i < n4; ++i)
    if (!std::isfinite(eri[i])) return fail(c, SWCS_E_INVALID, "non-finite eri");
  for (int p = 0; p < n; ++p)
    for (int q = 0; q < n; ++q)
      if (std::fabs(h[p * n + q] - h[q * n + p]) > 1e-12) return fail(c, SWCS_E_INVALID, "h not symmetric");
  auto E = [&](int p, int q, int r, int s) { return eri[((size_t)(p * n + q) * n + r) * n + s]; };
  for (int p = 0; p < n; ++p)
    for (int q = 0; q < n; ++q)
      for (int r = 0; r < n; ++r)
        for (int s = 0; s < n; ++s) {
          const double v = E(p, q, r, s);
          if (std::fabs(v - E(q, p, r, s)) > 1e-12 || std::fabs(v - E(p, q, s, r)) > 1e-12 ||
              std::fabs(v - E(r, s, p, q)) > 1e-12)
            return fail(c, SWCS_E_INVALID, "eri lacks 8-fold symmetry");
        }
  // (pq|rs) packed by symmetry, the element at p >= q, r >= s, pq >= rs
  const size_t m = (size_t)n * (n + 1) / 2;
  std::vector<double> e8(m * (m + 1) / 2);
  for (int p = 0; p < n; ++p)
    for (int q = 0; q <= p; ++q)
      for (int r = 0; r < n; ++r)
        for (int s = 0; s <= r; ++s)
          if (p * (p + 1) / 2 + q >= r * (r + 1) / 2 + s) e8[eri_packed_index(p, q, r, s)] = E(p, q, r, s);
  std::vector<double> Jh(n2), Kh(n2);
  for (int p = 0; p < n; ++p)
    for (int q = 0; q < n; ++q) {
      Jh[p * n + q] = E(p, p, q, q);
      Kh[p * n + q] = E(p, q, q, p);
    }
  HIP_TRY(c, c->h.ensure(n2 * 8), "alloc h");
  HIP_TRY(c, c->eri.ensure(n4 * 8), "alloc eri");
  HIP_TRY(c, c->eri8.ensure(e8.size() * 8), "alloc packed eri");
  HIP_TRY(c, c->J.ensure(n2 * 8), "alloc J");
  HIP_TRY(c, c->K.ensure(n2 * 8), "alloc K");
  HIP_TRY(c, c->fock.ensure(n2 * 8), "alloc fock");
  HIP_TRY(c, hipMemcpyAsync(c->h.p, h, n2 * 8, hipMemcpyHostToDevice, c->stream), "copy h");
  HIP_TRY(c, hipMemcpyAsync(c->eri.p, eri, n4 * 8, hipMemcpyHostToDevice, c->stream), "copy eri");
  HIP_TRY(c, hipMemcpyAsync(c->eri8.p, e8.data(), e8.size() * 8, hipMemcpyHostToDevice, c->stream), "copy eri");
  HIP_TRY(c, hipMemcpyAsync(c->J.p, Jh.data(), n2 * 8, hipMemcpyHostToDevice, c->stream), "copy J");
  HIP_TRY(c, hipMemcpyAsync(c->K.p, Kh.data(), n2 * 8, hipMemcpyHostToDevice, c->stream), "copy K");
  HIP_TRY(c, launch_fock(c->h.as<double>(), c->eri.as<double>(), n, c->na, c->fock.as<double>(),
                         c->stream), "fock");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  c->ecore = e_core;
  c->have_ints = true;
  c->ansatz_valid = false;
  return SWCS_OK;
}

int swcs_set_reference(swcs_ctx* c, uint64_t det) {
  if (!c) return SWCS_E_INVALID;
  if (c->nso < 64 && (det >> c->nso) != 0) return fail(c, SWCS_E_INVALID, "reference has bits beyond 2n");
  const int a = __builtin_popcountll(det & 0x5555555555555555ULL);
  const int b = __builtin_popcountll(det & 0xAAAAAAAAAAAAAAAAULL);
  if (a != c->na || b != c->nb) return fail(c, SWCS_E_INVALID, "reference electron counts differ from n_alpha/n_beta");
  c->ref = det;
  c->have_ref = true;
  c->ansatz_valid = false;
  return SWCS_OK;
}

int swcs_set_pool(swcs_ctx* c, const int32_t* rows, int64_t K) {
  if (!c) return SWCS_E_INVALID;
  if (K < 0 || (K > 0 && !rows)) return fail(c, SWCS_E_INVALID, "bad pool arguments");
  if (K > (int64_t)1 << 30) return fail(c, SWCS_E_INVALID, "pool too large");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  std::vector<OpDesc> ops((size_t)K);
  const int N = c->nso;
  for (int64_t k = 0; k < K; ++k) {
    const int32_t* r = rows + 4 * k;
    OpDesc o;
    o.P = r[0]; o.Q = r[1]; o.R = r[2]; o.S = r[3];
    const bool single = (o.R == -1 && o.S == -1);
    if (o.P < 0 || o.P >= N || o.Q < 0 || o.Q >= N || o.P <= o.Q)
      return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": need 2n > P > Q >= 0");
    if (single) {
      if ((o.P & 1) != (o.Q & 1)) return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": single changes spin");
      o.cre = 1ULL << o.P;
      o.ann = 1ULL << o.Q;
    } else {
      if (o.R < 0 || o.R >= N || o.S < 0 || o.S >= N || o.R <= o.S)
        return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": need 2n > R > S >= 0");
      if (o.P == o.R || o.P == o.S || o.Q == o.R || o.Q == o.S)
        return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": index sets overlap");
      if (((o.P & 1) + (o.Q & 1)) != ((o.R & 1) + (o.S & 1)))
        return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": double changes spin");
      if (!(o.P > o.R || (o.P == o.R && o.Q > o.S)))
        return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + ": need (P, Q) > (R, S)");
      o.cre = (1ULL << o.P) | (1ULL << o.Q);
      o.ann = (1ULL << o.R) | (1ULL << o.S);
    }
    ops[(size_t)k] = o;
  }
  // Generator table (P, Q, R, S) -> pool index in the layout of
  // optab_double_slot (conn_ops.h); -1 where the pool has no operator.
  // Rejects duplicate rows.
  std::vector<int> optab((size_t)optab_size(c->n), -1);
  for (int64_t k = 0; k < K; ++k) {
    const OpDesc& o = ops[(size_t)k];
    const int64_t slot = o.R < 0 ? pair_index(o.P, o.Q) : optab_double_slot(c->n, o.P, o.Q, o.R, o.S);
    if (optab[(size_t)slot] >= 0)
      return fail(c, SWCS_E_INVALID, "pool row " + std::to_string(k) + " duplicates an earlier row");
    optab[(size_t)slot] = (int)k;
  }
  // earlier work of the stream may still read the old tables
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  HIP_TRY(c, c->opmap.ensure(optab.size() * sizeof(int)), "alloc generator table");
  HIP_TRY(c, hipMemcpyAsync(c->opmap.p, optab.data(), optab.size() * sizeof(int), hipMemcpyHostToDevice, c->stream),
          "copy generator table");
  HIP_TRY(c, c->ops.ensure(std::max<size_t>(1, (size_t)K) * sizeof(OpDesc)), "alloc pool");
  if (K > 0)
    HIP_TRY(c, hipMemcpyAsync(c->ops.p, ops.data(), (size_t)K * sizeof(OpDesc), hipMemcpyHostToDevice, c->stream),
            "copy pool");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  c->ops_host.swap(ops);
  c->pool_rows.assign(rows, rows + 4 * K);
  c->K_pool = K;
  c->have_pool = true;
  c->ansatz_valid = false;
  return SWCS_OK;
}

// The unitaries of one apply call and the parameters they depend on.
struct ChainSpec {
  std::vector<int32_t> ops;    // pool row (row 1 of a star gate)
  std::vector<double> cs, sn;  // cos and sin of each unitary's angle
  std::vector<int> kind;       // 0 one row, 1 overlapping generator
  std::vector<GenGate> gen;    // kind 1
  std::vector<int64_t> owner;  // parameter of each unitary
  std::vector<double> factor;  // d(angle) / d(parameter)
  std::vector<double> theta;   // the parameters
  bool has_star = false;
};

static void spec_plain(const int32_t* op_idx, const double* theta, int64_t M, ChainSpec* sp) {
  sp->ops.assign(op_idx, op_idx + M);
  sp->theta.assign(theta, theta + M);
  sp->cs.resize((size_t)M);
  sp->sn.resize((size_t)M);
  for (int64_t i = 0; i < M; ++i) {
    sp->cs[(size_t)i] = std::cos(theta[i]);
    sp->sn[(size_t)i] = std::sin(theta[i]);
  }
  sp->kind.assign((size_t)M, 0);
  sp->gen.assign((size_t)M, GenGate{});
  sp->owner.resize((size_t)M);
  for (int64_t i = 0; i < M; ++i) sp->owner[(size_t)i] = i;
  sp->factor.assign((size_t)M, 1.0);
}

static int apply_common(swcs_ctx* c, ChainSpec& sp, double eps, int64_t ncut, int64_t* n_det_out,
                        bool from_reference) {
  const int64_t M = (int64_t)sp.ops.size();
  if (!from_reference && !c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  ++c->state_version;
  HIP_TRY(c, c->gate_n_in.ensure(std::max<int64_t>(1, M) * sizeof(u64)), "alloc stats");
  HIP_TRY(c, c->gate_n_act.ensure(std::max<int64_t>(1, M) * sizeof(u64)), "alloc stats");
  HIP_TRY(c, launch_fill_u32(c->gate_n_act.p, 0u, (u64)std::max<int64_t>(1, M) * 2, c->stream), "zero stats");
  c->ansatz_valid = false;
  if (from_reference) {
    c->seg = std::max<int>(1, (int)std::ceil(std::sqrt((double)std::max<int64_t>(1, M))));
    const int nck = (int)((M + c->seg - 1) / c->seg) + 1;
    if ((int)c->ckpt.size() < nck) {
      c->ckpt.resize(nck);
      c->bind_buffers();
    }
    HIP_TRY(c, c->ckpt_n.ensure((size_t)nck * sizeof(u64)), "alloc ckpt sizes");
    int r = state_reset_to_reference(c, M);
    if (r) return r;
  }
  Counters h;
  u64 n_start = 1;
  if (!from_reference) {
    hipError_t e;
    Counters h0 = get_counters(c, &e);
    if (e != hipSuccess) return hip_fail(c, e, "read counters");
    n_start = h0.n;
  }
  int r = run_chain(c, sp.ops.data(), sp.cs.data(), sp.sn.data(), M, eps, (unsigned)ncut, from_reference,
                    n_start, &h, sp.kind.data(), sp.gen.data());
  if (r && c->have_state) {
    // the state in front of the gate that did not fit, or the one before the first:
    // its index, where the chain failed before the one it would have left was
    // built, and its filter
    const std::string err = c->err;
    hipError_t e;
    const Counters h1 = read_counters(c, &e);
    if (e == hipSuccess && from_reference && chain_in_lds(c, 1, M)) {
      e = launch_hash_clear(c->st.hash, c->st.hmask + 1, c->stream);
      if (e == hipSuccess) e = launch_hash_build_dev(c->st, grid_blocks(c, c->st.cap, 256), c->stream);
    }
    if (e != hipSuccess || build_filter(c, h1.n, h1.alive) != SWCS_OK) c->have_state = false;
    c->err = err;
  }
  if (r) return r;
  r = build_filter(c, h.n, h.alive);
  if (r) return r;
  c->peak_n = std::max<u64>(c->peak_n, h.n);
  c->last_M = M;
  if (from_reference) {
    c->a_ops = sp.ops;
    c->a_theta = sp.theta;
    c->a_c = sp.cs;
    c->a_s = sp.sn;
    c->a_kind = sp.kind;
    c->a_gen = sp.gen;
    c->a_owner = sp.owner;
    c->a_factor = sp.factor;
    c->a_has_star = sp.has_star;
    c->a_eps = eps;
    c->a_ncut = ncut;
    c->ansatz_valid = true;
  }
  if (n_det_out) *n_det_out = (int64_t)h.alive;
  return SWCS_OK;
}

int swcs_apply_ansatz(swcs_ctx* c, const int32_t* op_idx, const double* theta, int64_t M,
                      double eps, int64_t ncut, int64_t* n_det_out) {
  if (!c) return SWCS_E_INVALID;
  int r = check_ready(c);
  if (r) return r;
  r = validate_gates(c, op_idx, theta, M, eps, ncut);
  if (r) return r;
  ChainSpec sp;
  spec_plain(op_idx, theta, M, &sp);
  return apply_common(c, sp, eps, ncut, n_det_out, true);
}

// Row k2 is the spin flip of row k1 (every spin-orbital P -> P ^ 1, in the
// same or the adjoint orientation).
static bool is_spin_flip(const OpDesc& a, const OpDesc& b) {
  auto flip = [](u64 m) { return ((m & 0x5555555555555555ULL) << 1) | ((m >> 1) & 0x5555555555555555ULL); };
  return (flip(a.cre) == b.cre && flip(a.ann) == b.ann) || (flip(a.cre) == b.ann && flip(a.ann) == b.cre);
}

int swcs_apply_generators(swcs_ctx* c, const int32_t* gens, const double* theta, int64_t M, double eps,
                          int64_t ncut, int64_t* n_det_out) {
  if (!c) return SWCS_E_INVALID;
  int r = check_ready(c);
  if (r) return r;
  if (M < 0) return fail(c, SWCS_E_INVALID, "M < 0");
  if (M > 0 && (!gens || !theta)) return fail(c, SWCS_E_INVALID, "null gens/theta");
  if (!(eps >= 0.0) || !std::isfinite(eps)) return fail(c, SWCS_E_INVALID, "eps must be finite and >= 0");
  if (ncut < 0 || ncut > 0x7fffffffLL) return fail(c, SWCS_E_INVALID, "ncut out of range");
  ChainSpec sp;
  const double rt = 1.0 / std::sqrt(2.0);
  for (int64_t i = 0; i < M; ++i) {
    const int32_t k1 = gens[3 * i], k2 = gens[3 * i + 1], sg = gens[3 * i + 2];
    const std::string at = "generator " + std::to_string(i) + ": ";
    if (k1 < 0 || k1 >= c->K_pool) return fail(c, SWCS_E_INVALID, at + "row 1 out of range");
    if (k2 < -1 || k2 >= c->K_pool || k2 == k1) return fail(c, SWCS_E_INVALID, at + "bad row 2");
    if (k2 >= 0 && sg != 1 && sg != -1) return fail(c, SWCS_E_INVALID, at + "sign must be +1 or -1");
    if (!std::isfinite(theta[i])) return fail(c, SWCS_E_INVALID, at + "non-finite theta");
    const double cth = std::cos(theta[i]), sth = std::sin(theta[i]);
    auto push = [&](int32_t k, double sn_u, double factor, int kd, const GenGate& g) {
      sp.ops.push_back(k);
      sp.cs.push_back(cth);
      sp.sn.push_back(sn_u);
      sp.kind.push_back(kd);
      sp.gen.push_back(g);
      sp.owner.push_back(i);
      sp.factor.push_back(factor);
    };
    if (k2 < 0) {
      push(k1, sth, 1.0, 0, GenGate{});
    } else {
      const OpDesc& o1 = c->ops_host[k1];
      const OpDesc& o2 = c->ops_host[k2];
      const bool overlap = ((o1.ann | o1.cre) & (o2.ann | o2.cre)) != 0;
      if (!overlap) {
        // commuting parts: two unitaries, row 2 at s theta
        push(k1, sth, 1.0, 0, GenGate{});
        push(k2, (double)sg * sth, (double)sg, 0, GenGate{});
      } else {
        if (o1.R < 0 || o2.R < 0 || !is_spin_flip(o1, o2))
          return fail(c, SWCS_E_UNSUPPORTED, at + "overlapping rows must be a double and its spin flip");
        GenGate g;
        g.op1 = o1;
        g.op2 = o2;
        g.c = cth;
        g.sn = sth;
        g.sn2 = (double)sg * sth;
        const double w = std::sqrt(2.0) * theta[i];
        g.c2 = std::cos(w);
        g.s2 = std::sin(w);
        g.rt = rt;
        g.sg = (double)sg;
        push(k1, sth, 1.0, 1, g);
        sp.has_star = true;
      }
    }
  }
  sp.theta.assign(theta, theta + M);
  return apply_common(c, sp, eps, ncut, n_det_out, true);
}

int swcs_apply_gates(swcs_ctx* c, const int32_t* op_idx, const double* theta, int64_t M,
                     double eps, int64_t ncut, int64_t* n_det_out) {
  if (!c) return SWCS_E_INVALID;
  int r = check_ready(c);
  if (r) return r;
  r = validate_gates(c, op_idx, theta, M, eps, ncut);
  if (r) return r;
  ChainSpec sp;
  spec_plain(op_idx, theta, M, &sp);
  return apply_common(c, sp, eps, ncut, n_det_out, false);
}

int swcs_set_state(swcs_ctx* c, const uint64_t* keys, const double* amps, int64_t n) {
  if (!c) return SWCS_E_INVALID;
  ++c->state_version;
  if (n < 0 || (n > 0 && (!keys || !amps))) return fail(c, SWCS_E_INVALID, "bad state arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  std::vector<u64> sorted(keys, keys + n);
  std::sort(sorted.begin(), sorted.end());
  for (int64_t i = 0; i < n; ++i) {
    const u64 k = keys[i];
    if (c->nso < 64 && (k >> c->nso) != 0) return fail(c, SWCS_E_INVALID, "key has bits beyond 2n");
    if (__builtin_popcountll(k & 0x5555555555555555ULL) != c->na ||
        __builtin_popcountll(k & 0xAAAAAAAAAAAAAAAAULL) != c->nb)
      return fail(c, SWCS_E_INVALID, "key outside the (n_alpha, n_beta) sector");
    if (!std::isfinite(amps[i])) return fail(c, SWCS_E_INVALID, "non-finite amplitude");
    if (i > 0 && sorted[(size_t)i] == sorted[(size_t)i - 1]) return fail(c, SWCS_E_INVALID, "duplicate key");
  }
  u64 cap = next_pow2(std::max<u64>(4096, 2 * (u64)n));
  cap = c->allow_regrow ? std::min<u64>(cap, max_capacity(c)) : fixed_capacity(c);
  if (cap < (u64)n) return fail(c, SWCS_E_CAPACITY, "state exceeds the maximum capacity");
  int r;
  if (!c->keys.p || c->st.cap != cap) {
    r = state_reserve(c, cap, 0);
    if (r) return r;
  } else {
    HIP_TRY(c, launch_hash_clear(c->st.hash, c->st.hmask + 1, c->stream), "hash clear");
  }
  if (n > 0) {
    HIP_TRY(c, hipMemcpyAsync(c->keys.p, keys, n * sizeof(u64), hipMemcpyHostToDevice, c->stream), "copy keys");
    HIP_TRY(c, hipMemcpyAsync(c->amps.p, amps, n * sizeof(double), hipMemcpyHostToDevice, c->stream), "copy amps");
  }
  Counters h;
  std::memset(&h, 0, sizeof(h));
  h.n = (u64)n;
  h.alive = (u64)n;
  HIP_TRY(c, launch_store_counters(c->st.ctr, h, c->stream), "counters");
  if (n > 0) HIP_TRY(c, launch_hash_build(c->st, (u64)n, c->stream), "hash build");
  r = build_filter(c, (u64)n, (u64)n);
  if (r) return r;
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  c->hc = h;
  c->hc_valid = true;
  c->peak_n = std::max<u64>(c->peak_n, (u64)n);
  c->have_state = true;
  c->ansatz_valid = false;
  return SWCS_OK;
}

// Export (key, vals[i]) of the alive entries sorted by key; vals = amps if NULL.
static int export_sorted(swcs_ctx* c, u64 n, u64 alive, const double* vals, uint64_t* keys,
                         double* out) {
  HIP_TRY(c, c->exp_keys.ensure(n * 8), "alloc");
  HIP_TRY(c, c->exp_amps.ensure(n * 8), "alloc");
  if (n <= export_small_max()) {
    HIP_TRY(c, launch_export_small(c->st, n, alive, vals, c->exp_keys.as<u64>(), c->exp_amps.as<double>(), c->stream),
            "sorted export");
  } else {
    HIP_TRY(c, c->exp_tmp_k.ensure(n * 8), "alloc");
    HIP_TRY(c, c->exp_tmp_v.ensure(n * 8), "alloc");
    const u64 scr = std::max(radix_sort_scratch_elems(n), compact_scratch_elems(n));
    HIP_TRY(c, c->sort_scratch.ensure(scr * 8), "alloc");
    HIP_TRY(c, launch_compact_alive(c->st, n, vals, c->exp_keys.as<u64>(), c->exp_amps.as<double>(),
                                    c->scalars.as<u64>() + 8, c->sort_scratch.as<u64>(), scr, c->stream), "compact");
    HIP_TRY(c, radix_sort_pairs(c->exp_keys.as<u64>(), c->exp_amps.as<u64>(), c->exp_tmp_k.as<u64>(),
                                c->exp_tmp_v.as<u64>(), alive, c->nso, c->sort_scratch.as<u64>(), scr,
                                c->stream), "sort");
  }
  HIP_TRY(c, hipMemcpyAsync(keys, c->exp_keys.p, alive * 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipMemcpyAsync(out, c->exp_amps.p, alive * 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  return SWCS_OK;
}

int swcs_get_state(swcs_ctx* c, uint64_t* keys, double* amps, int64_t cap, int64_t* n_out) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (n_out) *n_out = (int64_t)h.alive;
  if ((int64_t)h.alive > cap) return fail(c, SWCS_E_INVALID, "output capacity too small");
  if (h.alive == 0) return SWCS_OK;
  if (!keys || !amps) return fail(c, SWCS_E_INVALID, "null output arrays");
  return export_sorted(c, h.n, h.alive, nullptr, keys, amps);
}

// Enumeration probes every connection of every alive entry (alive * C
// probes); hole-pair grouping sorts n * C(N_e, 2) records instead.  The
// automatic choice takes grouping once the probe count passes this bound.
constexpr double kHolePairProbes = 3.0e7;
// Pair tests of the spin-string pass per hole-pair record up to which AUTO takes
// it.  A test costs about a tenth of a picosecond to a picosecond over the
// device, a record's share of emit, sort and group scan 60 to 100.  Strings
// against hole pairs, tests per record: 2e6 determinants of (26 orbitals, 8 + 8
// electrons) 4.8 to 9.5 ms at 3; 1e6 of (18, 6 + 6) 3.1 to 5.3 at 62; 3e5 of
// (14, 5 + 5) 1.9 to 3.0 at 158; 2e5 clustered of (26, 8 + 8) 2.6 to 6.1 at 411;
// 1e6 of (14, 5 + 5) 16.9 to 20.1 at 523.
constexpr double kStringTests = 500.0;

static bool use_holepair(swcs_ctx* c, u64 alive) {
  const int ne = c->na + c->nb;
  if (ne < 2 || c->sigma_method == SWCS_SIGMA_ENUMERATE) return false;
  if (c->sigma_method == SWCS_SIGMA_HOLE_PAIRS) return true;
  return (double)alive * (double)c->exc.total > kHolePairProbes;
}

// Small states: every pair of stored determinants is tested in LDS.  The
// automatic choice takes it when the pair count is at most 8 probes' worth
// of enumeration per determinant.
static bool use_sigma_pairs(swcs_ctx* c, u64 n) {
  if (n == 0 || n > (u64)pairwise_capacity()) return false;
  if (c->sigma_method == SWCS_SIGMA_PAIRS) return true;
  if (c->sigma_method != SWCS_SIGMA_AUTO) return false;
  return (double)n <= 8.0 * (double)c->exc.total;
}

// Diagonal elements of the n stored entries into c->diag (stream-ordered),
// unless already computed for the current state.
static int diag_enqueue(swcs_ctx* c, u64 n) {
  if (c->diag_version == c->state_version && c->diag.bytes >= n * 8 && c->st.diag == c->diag.p)
    return SWCS_OK;
  HIP_TRY(c, c->diag.ensure(std::max<u64>(1, n) * 8), "alloc diagonal");
  c->st.diag = c->diag.as<double>();
  HIP_TRY(c, launch_diag(c->st, ints_view(c), n, grid_blocks(c, n * kDiagLanes, 256), c->stream), "diagonal");
  c->diag_version = c->state_version;
  return SWCS_OK;
}

// sigma_P by spin strings into c->sigma (k_strings.hip); returns 1 when
// hole-pair grouping is the better choice: the entries share so few strings that
// the groups' pair tests outweigh its sort.  Synchronizes for that decision,
// which rests on a sample (20 us; deciding after the sorts cost a state that is
// turned away 200).
static int string_sigma_enqueue(swcs_ctx* c, const Counters& h) {
  const u64 n = h.n, alive = h.alive;
  if (c->sigma_method != SWCS_SIGMA_AUTO || alive == 0 || n >= (1ULL << 31)) return 1;
  const int ne = c->na + c->nb;
  const int occ[2] = {c->na, c->nb};
  const int shift = (c->n + 1 + 7) / 8 * 8;  // whole digits: the sort never reads the index
  if (shift < 64 && ((n - 1) >> (64 - shift)) != 0) return 1;
  // Tests per determinant, from the sampled chance that two share a string.
  // The spin whose strings lead the (1, 1) pass is the one with fewer tests: a
  // string's neighbours are at most nocc nvir groups of about its own size.
  unsigned sample[kStrSampleBlocks][5];
  HIP_TRY(c, c->partial.ensure(sizeof(sample)), "alloc partial");
  HIP_TRY(c, launch_str_sample(c->st, n, c->partial.as<unsigned>(), c->stream), "sample strings");
  const unsigned blocks = str_sample_blocks(n);
  HIP_TRY(c, hipMemcpyAsync(sample, c->partial.p, blocks * sizeof(sample[0]), hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  double hits[2] = {0.0, 0.0}, cols = 0.0, self = 0.0;
  for (unsigned b = 0; b < blocks; ++b) {
    for (int s = 0; s < 2; ++s) hits[s] += sample[b][s];
    cols += sample[b][2];
    self += sample[b][4];
  }
  const double pairs = std::max(1.0, cols * sample[0][3] - self);
  double own[2], adj[2];
  for (int s = 0; s < 2; ++s) {
    own[s] = 1.0 + hits[s] / pairs * (double)(alive - 1);
    adj[s] = own[s] * (double)(occ[s] * (c->n - occ[s]));
  }
  const int lead = adj[0] <= adj[1] ? 0 : 1;
  if (adj[lead] + own[0] + own[1] > kStringTests * (double)(ne * (ne - 1) / 2)) return 1;
  const u64 scr = radix_sort_scratch_elems(n);
  u64 slots[2];  // strings that can occur, at load 1/2
  for (int s = 0; s < 2; ++s)
    slots[s] = next_pow2(2 * std::max<u64>(32, std::min<u64>(alive, binomial_u64(c->n, occ[s]))));
  const int grid = grid_blocks(c, alive, 256);
  // per spin: records and their sort buffer, then keys, amplitudes and strings
  // in sorted order
  HIP_TRY(c, c->str_rec.ensure(4 * n * 8), "alloc strings");
  HIP_TRY(c, c->str_key.ensure(2 * alive * 8), "alloc strings");
  HIP_TRY(c, c->str_val.ensure(2 * alive * 8), "alloc strings");
  HIP_TRY(c, c->str_oth.ensure(2 * alive * 4), "alloc strings");
  HIP_TRY(c, c->str_tab.ensure((slots[0] + slots[1]) * str_slot_bytes()), "alloc strings");
  HIP_TRY(c, c->sort_scratch.ensure(scr * 8), "alloc sort scratch");
  u64* rec[2] = {c->str_rec.as<u64>(), c->str_rec.as<u64>() + n};
  u64* tmp[2] = {c->str_rec.as<u64>() + 2 * n, c->str_rec.as<u64>() + 3 * n};
  void* tab[2] = {c->str_tab.p, (char*)c->str_tab.p + slots[0] * str_slot_bytes()};
  HIP_TRY(c, launch_str_emit(c->st, n, c->n, shift, rec[0], rec[1], grid_blocks(c, n, 256), c->stream), "strings");
  for (int s = 0; s < 2; ++s) {
    HIP_TRY(c, radix_sort_keys(rec[s], tmp[s], n, shift, c->sort_scratch.as<u64>(), scr, c->stream, &rec[s]), "sort");
    HIP_TRY(c, launch_str_groups(c->st, rec[s], alive, c->n, shift, s, c->str_key.as<u64>() + s * alive,
                                 c->str_val.as<double>() + s * alive, c->str_oth.as<unsigned>() + s * alive, tab[s],
                                 slots[s], grid, c->stream), "groups");
  }
  const Ints I = ints_view(c);
  HIP_TRY(c, launch_sigma_diag(c->st, I, n, c->sigma.as<double>(), grid_blocks(c, n, 256), c->stream), "diagonal sigma");
  for (int s = 0; s < 2; ++s)
    TIMED(c, SWCS_K_STRINGS,
          launch_str_sigma(I, rec[s], alive, shift, occ[s], c->str_key.as<u64>() + s * alive,
                           c->str_val.as<double>() + s * alive, c->str_oth.as<unsigned>() + s * alive, tab[s], slots[s],
                           s == lead, c->sigma.as<double>(), grid_blocks(c, alive, 32), c->stream), "string pairs");
  return SWCS_OK;
}

// Same; a state without room for the strings is left to hole pairs, which may
// find their records' buffers in place.
static int string_sigma(swcs_ctx* c, const Counters& h) {
  const Busy busy(c->strings_busy);
  const int r = string_sigma_enqueue(c, h);
  if (r != SWCS_E_OOM) return r;
  DevBuf* bufs[] = {&c->str_rec, &c->str_key, &c->str_val, &c->str_oth, &c->str_tab};
  for (DevBuf* b : bufs) b->release();
  return 1;
}

// sigma_P over the stored entries; (numer, norm2) land in scalars[0..1] on
// the device (synchronizing only where a pass has to size or choose itself).
static int energy_enqueue(swcs_ctx* c, u64 n) {
  const int grid = sigma_grid(c, n);
  int rd = diag_enqueue(c, n);
  if (rd) return rd;
  HIP_TRY(c, c->sigma.ensure(std::max<u64>(1, n) * 8), "alloc sigma");
  HIP_TRY(c, c->partial.ensure((size_t)2 * grid * 8), "alloc partial");
  hipError_t e;
  const Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (use_sigma_pairs(c, n)) {
    const int pgrid = (int)std::min<u64>((n + 3) / 4, (u64)c->num_cu * 8);
    HIP_TRY(c, c->partial.ensure((size_t)2 * pgrid * 8), "alloc partial");
    TIMED(c, SWCS_K_SIGMA_PROJ, launch_sigma_pairwise(c->st, ints_view(c), n, c->sigma.as<double>(),
                                 c->partial.as<double>(), pgrid, c->stream), "sigma pairs");
    HIP_TRY(c, launch_reduce_partials(c->partial.as<double>(), pgrid, pgrid, 2, c->scalars.as<double>(), c->stream), "reduce");
    return SWCS_OK;
  }
  int by_strings = 1;
  if (n > 0 && use_holepair(c, h.alive)) {
    by_strings = string_sigma(c, h);
    if (by_strings < 0) return by_strings;
  }
  if (by_strings == SWCS_OK) {
    HIP_TRY(c, c->partial.ensure((size_t)2 * grid * 8), "alloc partial");
    HIP_TRY(c, launch_sigma_dots(c->st, c->sigma.as<double>(), n, c->partial.as<double>(), grid, c->stream), "dots");
  } else if (n > 0 && n < (1ULL << 32) && use_holepair(c, h.alive)) {
    const int ne = c->na + c->nb;
    const u64 total = n * ((u64)ne * (u64)(ne - 1) / 2);
    // Segments of the three removal classes (alpha-alpha, alpha-beta,
    // beta-beta), each sorted on its own on the key bits of the largest
    // class; the dead marker's low bits are all ones, above every key.
    const u64 na = (u64)c->na, nb = (u64)c->nb;
    const u64 seg_len[3] = {n * (na * (na - 1) / 2), n * na * nb, n * (nb * (nb - 1) / 2)};
    u64 cmax = 1;
    if (na >= 2) cmax = std::max(cmax, binomial_u64(c->n, c->na - 2) * binomial_u64(c->n, c->nb));
    if (na >= 1 && nb >= 1) cmax = std::max(cmax, binomial_u64(c->n, c->na - 1) * binomial_u64(c->n, c->nb - 1));
    if (nb >= 2) cmax = std::max(cmax, binomial_u64(c->n, c->na) * binomial_u64(c->n, c->nb - 2));
    int rank_bits = 1;
    while (rank_bits < 60 && (cmax >> rank_bits) != 0) ++rank_bits;
    // Records are single words when key and entry index fit: the key in the
    // low bytes that the radix passes read (rank_bits rounded up to whole
    // digits, so no pass sees index bits), the index above.  Otherwise a
    // 64-bit key plus a 32-bit index.
    int idx_bits = 1;
    while (idx_bits < 63 && ((n - 1) >> idx_bits) != 0) ++idx_bits;
    const int digit_bits = (rank_bits + 7) / 8 * 8;
    const int shift = (digit_bits + idx_bits <= 64) ? digit_bits : 0;
    HIP_TRY(c, c->hp_key.ensure(total * 8), "alloc hole-pair keys");
    HIP_TRY(c, c->hp_tk.ensure(total * 8), "alloc hole-pair keys");
    if (!shift) {
      HIP_TRY(c, c->hp_val.ensure(total * 4), "alloc hole-pair values");
      HIP_TRY(c, c->hp_tv.ensure(total * 4), "alloc hole-pair values");
    }
    // the segments are sorted one by one; a short segment uses small tiles
    // and can need more scratch than a longer one
    u64 scr = 0;
    for (u64 len : seg_len) scr = std::max(scr, radix_sort_scratch_elems(len));
    HIP_TRY(c, c->sort_scratch.ensure(scr * 8), "alloc sort scratch");
    u64* key = c->hp_key.as<u64>();
    u64* tkey = c->hp_tk.as<u64>();
    unsigned* val = shift ? nullptr : c->hp_val.as<unsigned>();
    unsigned* tval = shift ? nullptr : c->hp_tv.as<unsigned>();
    HIP_TRY(c, launch_holepair_emit(c->st, n, c->n, c->na, c->nb, shift, key, val, grid_blocks(c, n * 64, 256),
                                    c->stream), "emit");
    // every segment of two or more records ends in the same buffers (same
    // pass count); a single record stays put and is copied if needed
    const bool in_tmp = ((rank_bits + 7) / 8) % 2 == 1;
    u64 off = 0;
    for (int sgm = 0; sgm < 3; ++sgm) {
      const u64 len = seg_len[sgm];
      if (len >= 2) {
        u64* ok = nullptr;  // where the last pass left the segment (not copied back)
        if (shift) {
          HIP_TRY(c, radix_sort_keys(key + off, tkey + off, len, shift, c->sort_scratch.as<u64>(), scr,
                                     c->stream, &ok), "sort");
        } else {
          unsigned* ov = nullptr;
          HIP_TRY(c, radix_sort_pairs32(key + off, val + off, tkey + off, tval + off, len, rank_bits,
                                        c->sort_scratch.as<u64>(), scr, c->stream, &ok, &ov), "sort");
        }
        if (ok != (in_tmp ? tkey + off : key + off)) return fail(c, SWCS_E_DEVICE, "sort parity");
      } else if (len == 1 && in_tmp) {
        HIP_TRY(c, hipMemcpyAsync(tkey + off, key + off, 8, hipMemcpyDeviceToDevice, c->stream), "copy");
        if (!shift) HIP_TRY(c, hipMemcpyAsync(tval + off, val + off, 4, hipMemcpyDeviceToDevice, c->stream), "copy");
      }
      off += len;
    }
    u64* sk = in_tmp ? tkey : key;
    unsigned* sv = shift ? nullptr : (in_tmp ? tval : val);
    HIP_TRY(c, launch_sigma_diag(c->st, ints_view(c), n, c->sigma.as<double>(), grid_blocks(c, n, 256),
                                 c->stream), "diagonal sigma");
    off = 0;
    for (int sgm = 0; sgm < 3; ++sgm) {
      const u64 len = seg_len[sgm];
      TIMED(c, SWCS_K_HOLEPAIR, launch_holepair_sigma(c->st, ints_view(c), c->na, n, sk + off, sv ? sv + off : nullptr,
                                                      shift, len, sgm, c->sigma.as<double>(),
                                                      grid_blocks(c, len, 256), c->stream), "hole pairs");
      off += len;
    }
    HIP_TRY(c, launch_sigma_dots(c->st, c->sigma.as<double>(), n, c->partial.as<double>(), grid, c->stream), "dots");
  } else {
    TIMED(c, SWCS_K_SIGMA_PROJ, launch_sigma_proj(c->st, ints_view(c), c->exc, n, c->sigma.as<double>(),
                                 c->partial.as<double>(), nullptr, grid, c->stream), "sigma");
  }
  HIP_TRY(c, launch_reduce_partials(c->partial.as<double>(), grid, grid, 2, c->scalars.as<double>(), c->stream), "reduce");
  return SWCS_OK;
}

// Same, returning numer and norm2 on the host.
static int energy_internal(swcs_ctx* c, u64 n, double* numer, double* norm2) {
  int r = energy_enqueue(c, n);
  if (r) return r;
  double out[2];
  HIP_TRY(c, hipMemcpyAsync(out, c->scalars.p, 16, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  *numer = out[0];
  *norm2 = out[1];
  return SWCS_OK;
}

int swcs_energy(swcs_ctx* c, double* E, double* numer, double* norm2) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_ints) return fail(c, SWCS_E_STATE, "integrals not set");
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  double nu = 0.0, no = 0.0;
  int r = energy_internal(c, h.n, &nu, &no);
  if (r) return r;
  if (numer) *numer = nu;
  if (norm2) *norm2 = no;
  if (E) *E = nu / no;
  return SWCS_OK;
}

int swcs_energy_noalloc(swcs_ctx* c, double* E, double* numer, double* norm2) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_ints) return fail(c, SWCS_E_STATE, "integrals not set");
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  const Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  const u64 n = h.n;
  if (n > kNoAllocMaxEntries)
    return fail(c, SWCS_E_CAPACITY, "state has " + std::to_string(n) + " stored entries; the allocation-free "
                                     "energy takes at most " + std::to_string(kNoAllocMaxEntries));
  double* base = nullptr;
  HIP_TRY(c, noalloc_scratch(c->device, &base), "scratch address");
  double* partial = base;
  double* res = base + kNoAllocPartials;
  DeviceState st = c->st;
  st.diag = base + kNoAllocHead;
  double* sig = st.diag + n;
  const Ints I = ints_view(c);
  if (n > 0) {
    HIP_TRY(c, launch_diag(st, I, n, grid_blocks(c, n * kDiagLanes, 256), c->stream), "diagonal");
    if (n <= (u64)pairwise_capacity()) {
      const int pgrid = (int)std::min<u64>((n + 3) / 4, kNoAllocPartials / 2);
      HIP_TRY(c, launch_sigma_pairwise(st, I, n, sig, partial, pgrid, c->stream), "sigma pairs");
      HIP_TRY(c, launch_reduce_partials(partial, pgrid, pgrid, 2, res, c->stream), "reduce");
    } else {
      const int grid = std::min<int>(sigma_grid(c, n), (int)(kNoAllocPartials / 2));
      HIP_TRY(c, launch_sigma_proj(st, I, c->exc, n, sig, partial, nullptr, grid, c->stream), "sigma");
      HIP_TRY(c, launch_reduce_partials(partial, grid, grid, 2, res, c->stream), "reduce");
    }
  } else {
    HIP_TRY(c, launch_fill_u32(res, 0u, 4, c->stream), "zero");
  }
  double out[2];
  HIP_TRY(c, hipMemcpyAsync(out, res, 16, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  if (numer) *numer = out[0];
  if (norm2) *norm2 = out[1];
  if (E) *E = out[0] / out[1];
  return SWCS_OK;
}

int swcs_sigma_projected(swcs_ctx* c, uint64_t* keys, double* sigma, int64_t cap, int64_t* n_out) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_ints) return fail(c, SWCS_E_STATE, "integrals not set");
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (n_out) *n_out = (int64_t)h.alive;
  if ((int64_t)h.alive > cap) return fail(c, SWCS_E_INVALID, "output capacity too small");
  if (h.alive == 0) return SWCS_OK;
  if (!keys || !sigma) return fail(c, SWCS_E_INVALID, "null output arrays");
  double nu, no;
  int r = energy_internal(c, h.n, &nu, &no);
  if (r) return r;
  return export_sorted(c, h.n, h.alive, c->sigma.as<double>(), keys, sigma);
}

// <psi|psi> into scalars[2] on the device, without synchronizing (kept while
// the state is unchanged).
static int norm2_enqueue(swcs_ctx* c, u64 n) {
  if (c->norm_version == c->state_version) return SWCS_OK;
  const int grid = grid_blocks(c, n, 256);
  HIP_TRY(c, c->partial.ensure((size_t)grid * 8 * 2), "alloc partial");
  HIP_TRY(c, launch_occupations(c->st, n, 0, c->partial.as<double>(), grid, c->stream), "norm");
  HIP_TRY(c, launch_reduce_partials(c->partial.as<double>(), grid, grid, 1, c->scalars.as<double>() + 2, c->stream), "reduce");
  c->norm_version = c->state_version;
  return SWCS_OK;
}

// Records per sort of the density-matrix pass (2 GB and as much again for the
// sort); a state with more is taken in hash classes of its subsets.
constexpr u64 kRdmMaxRecords = 1ULL << 28;
// About this many determinants are looked at before the pass is taken.
constexpr u64 kRdmSample = 1024;
// Largest number of pairs (determinants within a triple excitation, counted
// once per subset they share) per record of the join, where every pair is added
// in memory: one device-scope add, 18 G/s measured, against 14-22 G/s for a join
// record.
constexpr double kRdmPairLimit = 1.0;
// Pairs per subset record from which the rows of the density matrix are summed
// in LDS: listing and sorting the records by row costs as much as one add in
// memory each (50 ps), and a pair then 5 ps instead of 55.  224,982 determinants
// of 30 spin-orbitals (7 pairs a record): 14.4 to 3.0 ms for this part;
// 137,595 of 52 (0.3 a record) would go from 2.0 to 4.
constexpr double kRdmRowPairs = 1.0;

// Whether that form is taken where the pairs outnumber the join's records: its
// measured share per subset record and per pair (both on the safe side), 0.85 ms
// for what does not depend on the state, and 65 ps per join record.  Measured
// against the join: 100,000 of (12 orbitals, 5 + 6 electrons) 2.6 to 13.6 ms at
// 1.3 pairs per join record; the full (12, 6 + 6) sector 69 to 118 at 10.6; the
// full (10, 5 + 5) sector, 63,504 determinants, is even (4.5).
static bool rdm_rows_pay(double records, double pairs, double join_records) {
  return 0.85e-3 + 8e-11 * records + 5.1e-12 * pairs < 6.5e-11 * join_records;
}

// Seconds of the density-matrix pass at n orbitals and `records` subset records,
// `each` seconds a record: fifteen small launches and the sample, the
// contraction's n^7, and emit, sort and pairs.
static double rdm_seconds(int n, double records, double each) {
  return 0.6e-3 + 4e-13 * std::pow((double)n, 7.0) + each * records;
}
// Whether AUTO takes it for a whole pool: 55 ps a subset record (the pairs of a
// crowded state are judged by the sample) against 65 ps a join record.  Matrix
// against join: 14 orbitals, 4 + 4 electrons 0.5 to 0.9 ms at 1.3e7 join records;
// 18 orbitals, 5 + 4 electrons 0.6 to 0.8 against 1.3 to 1.4 at 1.8e7; 22
// orbitals, 6 + 5 electrons 1.6 to 1.9 against 2.0 to 2.2 at 3.2e7; 26 orbitals,
// 8 + 8 electrons 4.0 against 5.5 at 8.9e7, 3.7 against 2.8 at 4.6e7.
static bool rdm_pays(int n, double records, double join_records) {
  return join_records >= 9.0e6 && rdm_seconds(n, records, 5.5e-11) < 6.5e-11 * join_records;
}
// Whether it is taken for a share of the pool.  The screened pass takes 15 to 25
// ps a join record and 350 to 550 more times the share of the operators (1 to
// 10 % of 15 to 26 orbitals, 3e7 to 5e8 records); a subset record here 150 with
// the pairs of a clustered state.  26 orbitals, 8 + 8 electrons, 4,392
// determinants: 4.9 against 8.6 ms at 10 %, 4.8 against 3.2 at 3 %.
static bool rdm_pays_screened(int n, double records, double join_records, double share) {
  return rdm_seconds(n, records, 1.5e-10) + 0.3e-3 < (1.5e-11 + 3.5e-10 * share) * join_records;
}

// A density-matrix pass: record format, sort, hash classes, and what the sample
// found.
struct RdmPlan {
  RdmFmt fm;
  int nbatch, sort_bits;
  u64 ntri, total, cap;  // triples of a determinant; records in all and a class's room
  double join_records, need, have;
  bool rows, crowded;
};

// Whether the pass can be taken at all; fills everything of the plan but the
// sample's findings.
static bool rdm_plan(swcs_ctx* c, const Counters& h, RdmPlan* p) {
  if (c->pool_method != SWCS_POOL_AUTO || c->table_budget > 0) return false;
  const int ne = c->na + c->nb;
  if (ne < 3 || ne > kRdmMaxElectrons) return false;
  p->join_records = (double)h.alive * (double)(c->exc.total + 1);
  p->ntri = (u64)ne * (u64)(ne - 1) * (u64)(ne - 2) / 6;
  p->total = h.alive * p->ntri;
  if (!rdm_pays(c->n, (double)p->total, p->join_records)) return false;
  // pairs of a state that is spread evenly over its sector: a state is at least
  // this crowded, so a full sector needs no sample
  {
    const double a = c->na, b = c->nb, va = c->n - c->na, vb = c->n - c->nb;
    auto c2 = [](double m) { return 0.5 * m * (m - 1.0); };
    auto c3 = [](double m) { return m * (m - 1.0) * (m - 2.0) / 6.0; };
    const double t1 = a * va + b * vb, t2 = c2(a) * c2(va) + c2(b) * c2(vb) + a * b * va * vb;
    const double t3 = c3(a) * c3(va) + c3(b) * c3(vb) + c2(a) * c2(va) * b * vb + c2(b) * c2(vb) * a * va;
    const double share = (double)h.alive / (double)c->sector;
    const double pairs = 0.5 * (double)h.alive * share * (t3 + (ne - 2.0) * t2 + c2(ne - 1.0) * t1);
    if (pairs > kRdmPairLimit * p->join_records && !rdm_rows_pay((double)p->total, pairs, p->join_records)) return false;
  }
  auto bits_for = [](u64 v) {
    int b = 1;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
  };
  p->fm.bt = bits_for(p->ntri - 1);
  p->fm.hb = std::min(48, 64 - p->fm.bt - bits_for(h.n - 1));
  p->nbatch = 1;
  while (p->nbatch < 256 && p->total / (u64)p->nbatch > kRdmMaxRecords) p->nbatch *= 2;
  // room for an uneven split of the subsets over the hash classes
  const u64 even = p->total / (u64)p->nbatch;
  p->cap = p->nbatch == 1 ? p->total : even + even / 8 + 65536;
  p->sort_bits = p->cap < (1ULL << 19) ? 16 : 24;
  if (p->fm.hb < p->sort_bits + 8 || even > kRdmMaxRecords) return false;
  p->need = 8.0 * ((double)rdm_gamma_elems(c->n) + (double)rdm_part_elems(c->n) + (double)rdm_two_elems(c->n) +
                   (double)rdm_vtab_elems(c->n) + 2.0 * (double)p->cap + (double)radix_sort_scratch_elems(p->cap));
  p->have = (double)(avail_bytes(c) + c->hp_key.bytes + c->hp_tk.bytes + c->sort_scratch.bytes + c->rdm_g3.bytes +
                     c->rdm_part.bytes + c->rdm_g2.bytes + c->rdm_vtab.bytes + c->rdm_mem.bytes);
  return p->need <= 0.5 * p->have;
}

// Record buffers of r records.
static int rdm_records(swcs_ctx* c, u64 r) {
  HIP_TRY(c, c->hp_key.ensure(r * 8), "alloc subset records");
  HIP_TRY(c, c->hp_tk.ensure(r * 8), "alloc subset records");
  HIP_TRY(c, c->sort_scratch.ensure(radix_sort_scratch_elems(r) * 8), "alloc sort scratch");
  return SWCS_OK;
}

// Decides by the pairs among a sample of the determinants, one in `share`: sets
// rows and crowded, and returns 1 for a state that is left to the join or the
// table.  Nothing but the record buffers, which the join uses as well, is allocated
// before.
static int rdm_sample(swcs_ctx* c, const Counters& h, RdmPlan* p) {
  u64* cursor = c->scalars.as<u64>() + 32;
  double share = 8.0;
  while (share < 1024.0 && ((double)h.alive / share > 2.0 * (double)kRdmSample ||
                            (double)p->total / share > 0.5 * (double)p->cap)) share *= 2.0;
  int r = rdm_records(c, p->cap);
  if (r) return r;
  HIP_TRY(c, launch_fill_u32(cursor, 0u, 2, c->stream), "zero cursor");
  HIP_TRY(c, launch_rdm_emit(c->st, h.n, c->na + c->nb, p->fm, 1, 0, (u64)share - 1, c->hp_key.as<u64>(), p->cap, cursor,
                             grid_blocks(c, h.n, 32), c->stream), "subset records");
  u64 R = 0;
  HIP_TRY(c, hipMemcpyAsync(&R, cursor, 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  if (R > p->cap) {
    HIP_TRY(c, launch_clear_flag(c->st.ctr, kFlagOverflow, c->stream), "clear flag");
    return 1;
  }
  double pairs = 0.0;
  if (R > 0) {
    // records that share a bucket's sort bits by chance are no pairs; their
    // expected number is taken off (16 bits keep it known to a percent of
    // the limit for up to 2^22 records)
    const int bits = R < (1ULL << 22) ? 16 : 24;
    u64* sorted = c->hp_key.as<u64>();
    HIP_TRY(c, radix_sort_keys(sorted, c->hp_tk.as<u64>(), R, bits, c->sort_scratch.as<u64>(),
                               radix_sort_scratch_elems(p->cap), c->stream, &sorted), "subset sort");
    const int cgrid = grid_blocks(c, R, 256);
    HIP_TRY(c, c->partial2.ensure((size_t)cgrid * 8), "alloc partials");
    HIP_TRY(c, launch_rdm_count(sorted, R, bits, c->partial2.as<double>(), cgrid, c->stream), "pair count");
    HIP_TRY(c, launch_reduce_partials(c->partial2.as<double>(), cgrid, cgrid, 1, c->scalars.as<double>() + 26,
                                      c->stream), "pair count");
    HIP_TRY(c, hipMemcpyAsync(&pairs, c->scalars.as<double>() + 26, 8, hipMemcpyDeviceToHost, c->stream), "copy");
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    pairs = std::max(0.0, pairs - 0.5 * (double)R * (double)R / (double)(1ULL << bits));
  }
  pairs *= share * share;
  const double mem = (double)p->cap * (double)rdm_member_bytes() + (double)((size_t)4 << rdm_row_bits());
  const bool many = pairs > kRdmRowPairs * (double)p->total;
  p->rows = many && p->need + mem <= 0.5 * p->have;
  p->crowded = pairs > kRdmPairLimit * p->join_records;
  if (p->crowded && !(many && rdm_rows_pay((double)p->total, pairs, p->join_records))) {
    c->rdm_declined = c->state_version;
    return 1;
  }
  return p->crowded && !p->rows ? 1 : SWCS_OK;
}

// The pass itself; returns 1 where a class of a crowded state or the records of a
// class turn out to be more than it takes.
static int rdm_pass(swcs_ctx* c, const Counters& h, const RdmPlan& p, const int* d_subset, int64_t count,
                    const double* norm2, double* d_out) {
  const int ne = c->na + c->nb;
  const u64 n = h.n, cap = p.cap;
  const u64 scr = radix_sort_scratch_elems(cap);
  u64* cursor = c->scalars.as<u64>() + 32;
  // In a new context the matrix is allocated while the first records are written and
  // sorted (0.2 ms); one in place is cleared before them, so that the sorted records
  // are still in the caches when the pairs read them (0.05 ms at 26 orbitals).
  double* gam = nullptr;
  auto matrix = [&]() -> int {
    HIP_TRY(c, c->rdm_g3.ensure(rdm_gamma_elems(c->n) * 8), "alloc density matrix");
    HIP_TRY(c, c->rdm_part.ensure(rdm_part_elems(c->n) * 8), "alloc density matrix");
    HIP_TRY(c, c->rdm_g2.ensure(rdm_two_elems(c->n) * 8), "alloc density matrix");
    HIP_TRY(c, c->rdm_vtab.ensure(rdm_vtab_elems(c->n) * 8), "alloc density matrix");
    HIP_TRY(c, c->rdm_bs.ensure((size_t)2 * c->n * c->n * 8), "alloc density matrix");
    if (p.rows)
      HIP_TRY(c, c->rdm_mem.ensure(cap * rdm_member_bytes() + ((size_t)4 << rdm_row_bits())), "alloc subset members");
    gam = c->rdm_g3.as<double>();
    HIP_TRY(c, launch_rdm_clear(c->n, gam, c->stream), "zero density matrix");
    return SWCS_OK;
  };
  if (c->rdm_g3.bytes >= rdm_gamma_elems(c->n) * 8) {
    int r = matrix();
    if (r) return r;
  }
  for (int b = 0; b < p.nbatch; ++b) {
    HIP_TRY(c, launch_fill_u32(cursor, 0u, 2, c->stream), "zero cursor");
    HIP_TRY(c, launch_rdm_emit(c->st, n, ne, p.fm, p.nbatch, b, 0, c->hp_key.as<u64>(), cap, cursor,
                               grid_blocks(c, n, p.nbatch > 1 ? 4 : 32), c->stream), "subset records");
    u64 R = p.total;
    if (p.nbatch > 1) {
      HIP_TRY(c, hipMemcpyAsync(&R, cursor, 8, hipMemcpyDeviceToHost, c->stream), "copy");
      HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
      if (R > cap) {  // a class far above its share (many entries on few subsets)
        HIP_TRY(c, launch_clear_flag(c->st.ctr, kFlagOverflow, c->stream), "clear flag");
        return 1;
      }
    }
    u64* sorted = c->hp_key.as<u64>();
    HIP_TRY(c, radix_sort_keys(sorted, c->hp_tk.as<u64>(), R, p.sort_bits, c->sort_scratch.as<u64>(), scr, c->stream,
                               &sorted), "subset sort");
    if (!gam) {
      int r = matrix();
      if (r) return r;
    }
    const int tiles = (int)std::min<u64>(std::max<u64>((R + 1023) / 1024, 1), (u64)c->num_cu * 16);
    if (p.rows && R > 0) {
      u64* list = sorted == c->hp_key.as<u64>() ? c->hp_tk.as<u64>() : c->hp_key.as<u64>();
      HIP_TRY(c, launch_rdm_members(c->st, n, c->n, ne, p.fm, p.sort_bits, sorted, R, c->rdm_mem.p, list, cursor, tiles,
                                    c->stream), "subset members");
      u64 got[2] = {0, 0};  // records of the list; a bucket longer than the pass takes
      HIP_TRY(c, hipMemcpyAsync(got, cursor, sizeof(got), hipMemcpyDeviceToHost, c->stream), "copy");
      HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
      if (!got[1]) {
        HIP_TRY(c, radix_sort_keys(list, sorted, got[0], rdm_row_bits(), c->sort_scratch.as<u64>(), scr, c->stream,
                                   &list), "row sort");
        HIP_TRY(c, launch_rdm_rows(c->n, list, got[0], (unsigned*)((char*)c->rdm_mem.p + cap * rdm_member_bytes()),
                                   c->rdm_mem.p, R, gam, c->stream), "rows");
        continue;
      }
      if (p.crowded) return 1;
    }
    HIP_TRY(c, launch_rdm_pairs(c->st, n, c->n, ne, p.fm, p.sort_bits, sorted, R, gam, tiles, c->stream), "pairs");
  }
  HIP_TRY(c, launch_rdm_diag(c->st, n, c->n, gam, (int)std::min<u64>((n + 7) / 8, (u64)c->num_cu), c->stream),
          "diagonal");
  HIP_TRY(c, launch_rdm_gradients(ints_view(c), c->eri.as<double>(), c->na, c->nb, gam, c->rdm_g2.as<double>(), c->rdm_vtab.as<double>(),
                                  c->rdm_part.as<double>(), c->rdm_bs.as<double>(), c->ops.as<OpDesc>(), d_subset,
                                  count, norm2, d_out, c->stream), "contraction");
  c->ps_keys = (double)p.total;
  c->ps_slots = 0;
  c->ps_batches = p.nbatch;
  c->ps_passes = 1;
  return SWCS_OK;
}

// Pool gradients of the `count` operators d_subset (NULL: the whole pool) into
// d_out from the three-body density matrix (k_rdm.hip).  Returns 1 when the
// pass does not apply: another method or a table budget is set, fewer than
// three electrons, a small state, too little memory, or so many pairs of
// determinants within a triple excitation that the join or the table does
// less work.  Synchronizes (the pair count decides), but a state that was found
// too crowded is not looked at again: 0.13 of 1.08 ms a call by the sample (4,600
// determinants of 14 orbitals), 0.9 of 35.4 where the pass itself finds it (100,000
// of 32).
static int rdm_gradients(swcs_ctx* c, const Counters& h, const int* d_subset, int64_t count, const double* norm2,
                         double* d_out) {
  RdmPlan p;
  if (c->rdm_declined == c->state_version || !rdm_plan(c, h, &p)) return 1;
  const Busy busy(c->matrix_busy);
  int r = rdm_sample(c, h, &p);
  if (r == SWCS_OK) {
    r = rdm_pass(c, h, p, d_subset, count, norm2, d_out);
    if (r == 1) c->rdm_declined = c->state_version;
    if (r == 1 || r == SWCS_E_OOM) (void)matrix_scratch(c, true);  // the join or the table may need the room
  }
  return r == SWCS_E_OOM ? 1 : r;
}

// The screened query table is sized from a bound on its key count (no host
// round trip) when that table stays below this size and no table budget is
// set, otherwise from an exact count.
constexpr double kQueryBoundBytes = 512.0 * 1024 * 1024;

// Screened pool gradients of the n_subset operators d_subset (valid device
// indices) into d_out (device, n_subset doubles): sigma only on the
// determinants the selected operators reach.  Small subsets are walked
// operator-major (|psi| x n_subset activity tests), larger ones
// determinant-major through the generator table.  Synchronizes only when the
// query table has to be sized by an exact count.
static int mark_subset(swcs_ctx* c, const int* d_subset, int64_t n_subset);

static int screened_gradients(swcs_ctx* c, const Counters& h, const int* d_subset, int64_t n_subset,
                              const double* norm2, double* d_out, bool may_sync) {
  const u64 n = h.n, alive = h.alive;
  const bool op_major = n_subset <= c->exc.total;
  const double bound = std::min<double>((double)c->sector,
                                        (double)alive * (double)(op_major ? n_subset : c->exc.total));
  // The density matrix of the state gives any subset at the price of the whole
  // pool.  It synchronizes: for calls that do so anyway, and those that would
  // count their query keys.
  const double ne = c->na + c->nb;
  if ((may_sync || 2.0 * bound * sizeof(AccSlot) > kQueryBoundBytes) &&
      rdm_pays_screened(c->n, (double)alive * ne * (ne - 1.0) * (ne - 2.0) / 6.0,
                        (double)alive * (double)(c->exc.total + 1), (double)n_subset / (double)c->K_pool)) {
    int r = rdm_gradients(c, h, d_subset, n_subset, norm2, d_out);
    if (r <= 0) {
      c->ps_screened = 1;
      return r;
    }
  }
  // a state too large for the join makes its scratch dead weight
  if (!join_fits_state(c, alive)) release_join_scratch(c);
  const unsigned char* d_sel = nullptr;
  if (!op_major) {
    // the determinant-major passes test the operator flags and accumulate
    // into the pool-wide g
    int r = mark_subset(c, d_subset, n_subset);
    if (r) return r;
    d_sel = c->selected.as<unsigned char>();
  }
  u64 nq;
  bool counted = false, sampled = false;
  if (c->table_budget == 0 && 2.0 * bound * sizeof(AccSlot) <= kQueryBoundBytes) {
    nq = (u64)bound;
  } else {
    // count the (determinant, operator) pairs, on every 16th determinant
    // (or tile) of a state of 16,384 stored entries or more: the scaled
    // sample sizes the table, and a pass whose table fills is repeated with
    // twice the estimate (a full count costs as much as the insert pass)
    counted = true;
    const int stride = n >= 16384 ? 16 : 1;
    sampled = stride > 1;
    u64* qcount = c->scalars.as<u64>() + 16;
    HIP_TRY(c, launch_fill_u32(qcount, 0u, 2, c->stream), "zero counter");
    if (op_major)
      HIP_TRY(c, launch_query_ops(c->st, n, c->ops.as<OpDesc>(), d_subset, n_subset, nullptr, 0, stride,
                                  qcount, c->stream), "count");
    else
      HIP_TRY(c, launch_query_set(c->st, c->exc, c->n, n, c->opmap.as<int>(), c->n, d_sel,
                                  nullptr, 0, stride, qcount, sigma_grid(c, n), c->stream), "count");
    HIP_TRY(c, hipMemcpyAsync(&nq, qcount, 8, hipMemcpyDeviceToHost, c->stream), "copy");
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    if (sampled) nq = (u64)(1.25 * (double)nq * stride) + 4096;
  }
  // The query keys number at most q; a table for all of them that would
  // not fit in 40% of the free device memory is split by key hash into
  // batches, each a full query / push / contract pass over its own keys.
  // Counted pairs repeat keys many times over: the query keys are external
  // determinants, so the distinct external count of the last full-pool call
  // (scaled by the alive count) caps the estimate, and a pass that
  // overflows is repeated with twice the estimate.
  double q = (double)std::min<u64>(nq, c->sector);
  bool estimated = sampled;
  if (counted && c->ext_count > 0.0 && c->ext_alive > 0.0) {
    const double est = 1.5 * c->ext_count * std::max(1.0, (double)alive / c->ext_alive);
    if (est < q) {
      q = est;
      estimated = true;
    }
  }
  double budget = (double)c->table_budget;
  auto slots_for = [&](int nb) { return next_pow2((u64)std::max(64.0, (nb > 1 ? 2.5 : 2.0) * q / nb)); };
  auto batches = [&]() {
    int nb = 1;
    if (budget <= 0.0 && (double)slots_for(1) * sizeof(AccSlot) <= kQueryBoundBytes) return nb;
    if (budget <= 0.0) budget = free_table_budget(c, (double)slots_for(1) * sizeof(AccSlot));
    while (nb < 4096 && (double)slots_for(nb) * sizeof(AccSlot) > budget) nb *= 2;
    return nb;
  };
  int nbatch = batches();
  bool checked = false, replanned = false;
  int passes = 0;
  for (int attempt = 0;;) {
    const u64 qslots = slots_for(nbatch);
    HIP_TRY(c, c->acc_tab.ensure(qslots * sizeof(AccSlot)), "alloc sigma table");
    // presence filter of the batch's query keys: 8 bits per table slot (1/16
    // of the table's bytes), at least 4,096 bits and at most 2^30 (128 MB,
    // so that it stays in the last-level cache)
    const u64 qbits = std::min<u64>((u64)1 << 30, next_pow2(std::max<u64>(4096, 8 * qslots)));
    HIP_TRY(c, c->qfilt.ensure(qbits / 8), "alloc query filter");
    unsigned* qf = c->qfilt.as<unsigned>();
    ++passes;
    if (op_major)
      HIP_TRY(c, launch_fill_u32(d_out, 0u, (u64)n_subset * 2, c->stream), "zero g");
    else
      HIP_TRY(c, launch_fill_u32(c->gacc.p, 0u, (u64)c->K_pool * 2, c->stream), "zero g");
    bool replan = false;
    for (int b = 0; b < nbatch; ++b) {
      HIP_TRY(c, launch_fill_u32(c->acc_tab.p, 0u, qslots * (sizeof(AccSlot) / 4), c->stream), "clear table");
      HIP_TRY(c, launch_fill_u32(qf, 0u, qbits / 32, c->stream), "clear filter");
      // The estimate that set the batch count is an upper bound (pairs, or
      // the distinct count of all external keys); the first batch of a
      // batched pass counts its new keys, and since key-hash batches split
      // the query set evenly, a set much smaller than planned restarts the
      // pass with fewer batches (only this batch's query pass is lost).
      u64* qnew = (b == 0 && nbatch > 1 && estimated && !replanned) ? c->scalars.as<u64>() + 40 : nullptr;
      if (qnew) HIP_TRY(c, launch_fill_u32(qnew, 0u, 2, c->stream), "zero counter");
      if (op_major)
        HIP_TRY(c, launch_query_ops(c->st, n, c->ops.as<OpDesc>(), d_subset, n_subset,
                                    c->acc_tab.as<AccSlot>(), qslots - 1, 0, qnew, c->stream, nbatch, b,
                                    qf, qbits - 1), "query set");
      else
        HIP_TRY(c, launch_query_set(c->st, c->exc, c->n, n, c->opmap.as<int>(), c->n, d_sel,
                                    c->acc_tab.as<AccSlot>(), qslots - 1, 0, qnew, sigma_grid(c, n),
                                    c->stream, nbatch, b, qf, qbits - 1), "query set");
      if (qnew) {
        replanned = true;
        u64 got = 0;
        HIP_TRY(c, hipMemcpyAsync(&got, qnew, 8, hipMemcpyDeviceToHost, c->stream), "copy");
        HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
        const double q_new = std::max(64.0, 1.25 * (double)got * nbatch);
        if (q_new < 0.5 * q) {
          const double q_old = q;
          q = q_new;
          const int nb_new = batches();
          if (nb_new < nbatch) {
            nbatch = nb_new;
            replan = true;
            break;
          }
          q = q_old;
        }
      }
      TIMED(c, SWCS_K_SIGMA_PUSH_INTO, launch_sigma_push_into(c->st, ints_view(c), c->exc, n, c->acc_tab.as<AccSlot>(),
                                                              qslots - 1, sigma_grid(c, n), c->stream, nbatch, b,
                                                              qf, qbits - 1),
            "sigma push");
      if (op_major)
        TIMED(c, SWCS_K_CONTRACT_OPS, launch_contract_ops(c->st, n, c->ops.as<OpDesc>(), d_subset, n_subset,
                                                          c->acc_tab.as<AccSlot>(), qslots - 1, d_out, c->stream,
                                                          nbatch, b), "contract");
      else
        TIMED(c, SWCS_K_POOL_CONTRACT, launch_pool_contract_det(c->st, c->exc, c->n, n, c->opmap.as<int>(), c->n,
                                                                d_sel, c->acc_tab.as<AccSlot>(), qslots - 1, nbatch, b,
                                                                c->gacc.as<double>(), sigma_grid(c, n), c->stream),
              "contract");
    }
    if (replan) continue;
    // A single bound-sized table (at most half full) is checked on the
    // device when the caller does not synchronize (below); otherwise a pass
    // in which a table filled is repeated with twice the estimate.
    if (!may_sync && nbatch == 1 && !estimated) break;
    checked = true;
    hipError_t e;
    Counters h2 = read_counters(c, &e);  // synchronizes
    if (e != hipSuccess) return hip_fail(c, e, "read counters");
    if (!(h2.flags & kFlagOverflow)) break;
    h2.flags &= ~kFlagOverflow;
    HIP_TRY(c, launch_store_counters(c->st.ctr, h2, c->stream), "counters");
    c->hc = h2;
    if (++attempt > 16) return fail(c, SWCS_E_DEVICE, "sigma table overflow");
    q *= 2.0;
    nbatch = batches();
  }
  c->ps_keys = q;
  c->ps_slots = slots_for(nbatch);
  c->ps_batches = nbatch;
  c->ps_passes = passes;
  c->ps_screened = 1;
  if (op_major)
    HIP_TRY(c, launch_gather_scaled(d_out, nullptr, n_subset, norm2, d_out, c->stream), "scale");
  else
    HIP_TRY(c, launch_gather_scaled(c->gacc.as<double>(), d_subset, n_subset, norm2, d_out, c->stream), "gather");
  if (!checked) {
    // unchecked pass: a table that filled turns every result into NaN, and
    // the flag is cleared for later calls
    HIP_TRY(c, launch_nan_if_flag(c->st.ctr, kFlagOverflow, d_out, n_subset, c->stream), "overflow check");
    HIP_TRY(c, launch_clear_flag(c->st.ctr, kFlagOverflow, c->stream), "overflow clear");
  }
  return SWCS_OK;
}

// Shared set-up of both pool-gradient entry points: counters, norm, diagonal
// elements and the pool-wide accumulator's allocation.
static int pool_setup(swcs_ctx* c, Counters* h) {
  int r = check_ready(c);
  if (r) return r;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  *h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (h->alive == 0) return fail(c, SWCS_E_STATE, "state is empty");
  r = norm2_enqueue(c, h->n);
  if (r) return r;
  r = diag_enqueue(c, h->n);
  if (r) return r;
  HIP_TRY(c, c->gacc.ensure((size_t)c->K_pool * 8), "alloc g accumulator");
  return SWCS_OK;
}

static int mark_subset(swcs_ctx* c, const int* d_subset, int64_t n_subset) {
  const u64 words = ((u64)c->K_pool + 3) / 4;
  HIP_TRY(c, c->selected.ensure(words * 4), "alloc selection");
  HIP_TRY(c, launch_fill_u32(c->selected.p, 0u, words, c->stream), "zero selection");
  HIP_TRY(c, launch_mark_selected(d_subset, n_subset, c->selected.as<unsigned char>(), c->stream), "mark");
  return SWCS_OK;
}

int swcs_pool_gradients_device(swcs_ctx* c, const int32_t* d_subset, int64_t n_subset, double* d_g) {
  if (!c) return SWCS_E_INVALID;
  if (n_subset < 0) return fail(c, SWCS_E_INVALID, "n_subset < 0");
  if (n_subset > 0 && (!d_subset || !d_g)) return fail(c, SWCS_E_INVALID, "null device pointer");
  if (n_subset == 0) return SWCS_OK;
  Counters h;
  int r = pool_setup(c, &h);
  if (r) return r;
  HIP_TRY(c, c->subset_buf.ensure((size_t)n_subset * 4), "alloc subset");
  HIP_TRY(c, launch_sanitize_subset(d_subset, n_subset, c->K_pool, c->subset_buf.as<int>(), c->stream), "subset");
  const int* sub = c->subset_buf.as<int>();
  const double* norm2 = c->scalars.as<double>() + 2;
  r = screened_gradients(c, h, sub, n_subset, norm2, d_g, false);
  if (r) return r;
  HIP_TRY(c, launch_nan_invalid(d_subset, n_subset, c->K_pool, d_g, c->stream), "flag invalid");
  return SWCS_OK;
}

// Full-pool (or large-subset) gradients by sort and join (k_join.hip).
// Returns 1 when the join does not apply (method, memory, record word) or a
// join step overflowed its LDS table and AUTO may fall back to the table,
// else an SWCS status; on SWCS_OK the scaled gradients are in gbuf.
static int join_gradients(swcs_ctx* c, const Counters& h, const unsigned char* d_sel, const int* d_subset,
                          int64_t count, const double* norm2) {
  if (c->pool_method == SWCS_POOL_TABLE) return 1;
  if (c->pool_method == SWCS_POOL_AUTO && c->table_budget > 0) return 1;
  const bool forced = c->pool_method == SWCS_POOL_JOIN;
  const u64 n = h.n, C = (u64)c->exc.total;
  const u64 R = h.alive * (C + 1);
  // Measured at 52 spin-orbitals: 1.54e9 records take 120 ms by the join
  // against 187 ms by the table, but 7.9e9 records (266,101 determinants)
  // take 1.9 s, where the table needs about 1 s: beyond 2^31 records AUTO
  // takes the table (and gives back the join's scratch, which a state of
  // this size leaves unused).
  if (!join_fits_state(c, h.alive)) {
    release_join_scratch(c);
    return 1;
  }
  int kb, bh, bp, orb;
  if (!join_format(c->exc, n, R, &kb, &bh, &bp, &orb)) {
    if (forced) return fail(c, SWCS_E_CAPACITY, "join records do not fit 64 bits");
    return 1;
  }
  const u64 scr = radix_sort_scratch_elems(R);
  const u64 list_bytes = n * 16;  // (key, psi) of every stored entry
  const double need = 16.0 * (double)R + 8.0 * (double)scr + (double)list_bytes;
  // Gradient terms by operator bin (2^lb bins of at most kJoinTermSlots
  // operators, k mod 2^lb), each with room for 1.25 times an even share of
  // the records: the device-scope adds into g[K] then number about 8192 per
  // bin and chunk instead of one per record.  Terms past a full bin, and
  // every term when the bins do not fit, take the direct adds.
  int lb = 0;
  while (lb < kJoinBinsLog && (u64)c->K_pool > (256ULL << lb)) ++lb;
  while (lb <= kJoinMaxBinsLog && (u64)c->K_pool > ((u64)kJoinTermSlots << lb)) ++lb;
  const bool bins = lb <= kJoinMaxBinsLog;
  const u64 cap = ((u64)(1.25 * (double)R / (double)(1ULL << lb)) + 4096 + 7) & ~7ULL;
  const double bin_bytes = 10.0 * (double)cap * (double)(1ULL << lb);
  auto room = [&]() {
    return 0.5 * (double)(avail_bytes(c) + c->hp_key.bytes + c->hp_tk.bytes + c->sort_scratch.bytes +
                          c->join_src.bytes + c->join_w.bytes);
  };
  double half = room();
  const double gain = 0.5 * (double)matrix_scratch(c, false);
  if ((need > half && need <= half + gain) || (bins && need + bin_bytes > half && need + bin_bytes <= half + gain)) {
    (void)matrix_scratch(c, true);
    half = room();
  }
  if (need > half) {
    if (forced) return fail(c, SWCS_E_CAPACITY, "join records exceed half of the free device memory");
    return 1;
  }
  JoinTerms terms{-1, 0, nullptr, nullptr, nullptr};
  if (bins && need + bin_bytes <= half) {
    // one buffer: the bins' cursors (2 KB kept for them), values, operators
    const size_t head = (size_t)8 << kJoinMaxBinsLog;
    HIP_TRY(c, c->join_w.ensure(head + (size_t)(cap << lb) * 10), "alloc join terms");
    HIP_TRY(c, launch_fill_u32(c->join_w.p, 0u, (u64)2 << lb, c->stream), "zero bins");
    double* w = (double*)((char*)c->join_w.p + head);
    terms = JoinTerms{lb, cap, c->join_w.as<u64>(), w, (unsigned short*)(w + (cap << lb))};
  }
  HIP_TRY(c, c->hp_key.ensure(R * 8), "alloc join records");
  HIP_TRY(c, c->hp_tk.ensure(R * 8), "alloc join records");
  HIP_TRY(c, c->sort_scratch.ensure(scr * 8), "alloc sort scratch");
  HIP_TRY(c, c->join_src.ensure(std::max<u64>(16, list_bytes)), "alloc join sources");
  const int rgrid = (int)std::min<u64>((R + kJoinRunHost - 1) / kJoinRunHost, (u64)c->num_cu * 8);
  HIP_TRY(c, c->partial2.ensure((size_t)std::max(rgrid, 1) * 8), "alloc partials");
  u64* cursor = c->scalars.as<u64>() + 32;
  HIP_TRY(c, launch_fill_u32(cursor, 0u, 2, c->stream), "zero cursor");
  u64* recs = c->hp_key.as<u64>();
  TIMED(c, SWCS_K_JOIN_EMIT, launch_join_emit(c->st, c->exc, n, recs, R, cursor, kb, bh, bp, orb,
                                                c->join_src.p, sigma_grid(c, n), c->stream),
        "join emit");
  u64* sorted = recs;
  TIMED(c, SWCS_K_JOIN_SORT, radix_sort_keys(recs, c->hp_tk.as<u64>(), R, kb, c->sort_scratch.as<u64>(), scr,
                                             c->stream, &sorted), "join sort");
  HIP_TRY(c, launch_fill_u32(c->gacc.p, 0u, (u64)c->K_pool * 2, c->stream), "zero g");
  double* ins = c->partial2.as<double>();
  TIMED(c, SWCS_K_JOIN_REDUCE, launch_join_reduce(c->st, sorted, R, cursor, kb, bh, bp, orb, c->join_src.p, n,
                                                  ints_view(c), c->exc, c->opmap.as<int>(),
                                                  c->n, d_sel, c->gacc.as<double>(), terms, ins, rgrid,
                                                  c->stream),
        "join reduce");
  TIMED(c, SWCS_K_JOIN_TERMS, launch_join_terms(terms, c->gacc.as<double>(), c->K_pool, c->stream), "join terms");
  HIP_TRY(c, launch_reduce_partials(ins, rgrid, rgrid, 1, c->scalars.as<double>() + 24, c->stream), "count");
  double distinct = 0.0;
  HIP_TRY(c, hipMemcpyAsync(&distinct, c->scalars.as<double>() + 24, 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, launch_gather_scaled(c->gacc.as<double>(), d_subset, count, norm2, c->gbuf.as<double>(), c->stream),
          "gather");
  hipError_t e;
  Counters h2 = read_counters(c, &e);  // synchronizes
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (h2.flags & kFlagOverflow) {
    h2.flags &= ~kFlagOverflow;
    HIP_TRY(c, launch_store_counters(c->st.ctr, h2, c->stream), "counters");
    c->hc = h2;
    if (forced) return fail(c, SWCS_E_DEVICE, "join group overflowed its LDS table");
    return 1;
  }
  c->ext_count = distinct;
  c->ext_alive = (double)h.alive;
  c->ps_keys = distinct;
  c->ps_slots = 0;
  c->ps_batches = 1;
  c->ps_passes = 1;
  c->ps_screened = 0;
  return SWCS_OK;
}

int swcs_pool_gradients(swcs_ctx* c, const int32_t* subset, int64_t n_subset, double* g_out) {
  if (!c) return SWCS_E_INVALID;
  if (!g_out) return fail(c, SWCS_E_INVALID, "null g_out");
  const int64_t count = subset ? n_subset : c->K_pool;
  if (subset) {
    if (n_subset < 0) return fail(c, SWCS_E_INVALID, "n_subset < 0");
    for (int64_t t = 0; t < n_subset; ++t)
      if (subset[t] < 0 || subset[t] >= c->K_pool) return fail(c, SWCS_E_INVALID, "subset index out of range");
  }
  int r = check_ready(c);
  if (r) return r;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  if (count == 0) return SWCS_OK;
  Counters h;
  r = pool_setup(c, &h);
  if (r) return r;
  hipError_t e;
  const u64 n = h.n;
  const double* norm2 = c->scalars.as<double>() + 2;
  HIP_TRY(c, c->gbuf.ensure((size_t)count * 8), "alloc g");
  const int* d_subset = nullptr;
  const unsigned char* d_sel = nullptr;
  if (subset) {
    HIP_TRY(c, c->subset_buf.ensure((size_t)n_subset * 4), "alloc subset");
    HIP_TRY(c, hipMemcpyAsync(c->subset_buf.p, subset, (size_t)n_subset * 4, hipMemcpyHostToDevice, c->stream), "copy subset");
    // the host array is pageable: wait for the copy before the kernels that
    // read it are enqueued
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    d_subset = c->subset_buf.as<int>();
  }
  if (subset && 2 * n_subset < c->K_pool) {
    r = screened_gradients(c, h, d_subset, n_subset, norm2, c->gbuf.as<double>(), true);
    if (r) return r;
    HIP_TRY(c, hipMemcpyAsync(g_out, c->gbuf.p, (size_t)count * 8, hipMemcpyDeviceToHost, c->stream), "copy g");
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    return SWCS_OK;
  }
  r = rdm_gradients(c, h, d_subset, count, norm2, c->gbuf.as<double>());
  if (r <= 0) {
    if (r) return r;
    c->ps_screened = 0;
    HIP_TRY(c, hipMemcpyAsync(g_out, c->gbuf.p, (size_t)count * 8, hipMemcpyDeviceToHost, c->stream), "copy g");
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    return SWCS_OK;
  }
  if (subset) {
    r = mark_subset(c, d_subset, n_subset);
    if (r) return r;
    d_sel = c->selected.as<unsigned char>();
  }
  r = join_gradients(c, h, d_sel, d_subset, count, norm2);
  if (r <= 0) {
    if (r) return r;
    HIP_TRY(c, hipMemcpyAsync(g_out, c->gbuf.p, (size_t)count * 8, hipMemcpyDeviceToHost, c->stream), "copy g");
    HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
    return SWCS_OK;
  }
  // External-space table.  At most alive * (C + 1) distinct keys (and never
  // more than the sector) can occur, but states built by gate chains overlap
  // heavily, so the table is sized from the distinct-key count of the
  // previous call scaled by the alive count; load factor <= 1/2; split by key
  // hash only when the table would exceed the memory budget.  A table that
  // fills up raises kFlagOverflow and the pass is repeated with twice the
  // estimate.
  const double bound_d = std::min<double>((double)c->sector, (double)h.alive * (double)(c->exc.total + 1));
  double guess = bound_d;
  if (c->ext_count > 0.0 && c->ext_alive > 0.0)
    guess = std::min(bound_d, 1.5 * c->ext_count * std::max(1.0, (double)h.alive / c->ext_alive));
  // Tables up to 256 MB need no free-memory query.
  double budget = 256.0 * 1024 * 1024;
  if (c->table_budget > 0) {
    budget = (double)c->table_budget;
  } else if (4.0 * guess * sizeof(AccSlot) > budget) {
    budget = free_table_budget(c, 4.0 * guess * sizeof(AccSlot));
  }
  const int sgrid = sigma_grid(c, n);
  for (int attempt = 0;; ++attempt) {
    int nbatch = 1;
    while ((2.0 * guess / nbatch) * sizeof(AccSlot) > budget && nbatch < 4096) nbatch *= 2;
    u64 slots = next_pow2((u64)std::max<double>(64.0, 2.0 * guess / nbatch * (nbatch > 1 ? 1.25 : 1.0)));
    // a single table that fits twice over runs at load <= 1/4 (shorter probes)
    if (nbatch == 1 && 2.0 * (double)slots * sizeof(AccSlot) <= budget) slots *= 2;
    HIP_TRY(c, c->acc_tab.ensure(slots * sizeof(AccSlot)), "alloc sigma table");
    HIP_TRY(c, c->partial2.ensure((size_t)sgrid * nbatch * 8), "alloc partials");
    HIP_TRY(c, launch_fill_u32(c->gacc.p, 0u, (u64)c->K_pool * 2, c->stream), "zero g");
    double* ins = c->partial2.as<double>();
    for (int b = 0; b < nbatch; ++b) {
      HIP_TRY(c, launch_fill_u32(c->acc_tab.p, 0u, slots * (sizeof(AccSlot) / 4), c->stream), "clear table");
      TIMED(c, SWCS_K_SIGMA_PUSH, launch_sigma_push(c->st, ints_view(c), c->exc, n, c->acc_tab.as<AccSlot>(), slots - 1,
                                   nbatch, b, ins + (size_t)b * sgrid, sgrid, c->stream), "sigma push");
      TIMED(c, SWCS_K_POOL_CONTRACT, launch_pool_contract_det(c->st, c->exc, c->n, n, c->opmap.as<int>(), c->n,
                                          d_sel, c->acc_tab.as<AccSlot>(), slots - 1, nbatch, b,
                                          c->gacc.as<double>(), sgrid, c->stream), "contract");
    }
    // distinct keys over all batches (the batches partition the keys)
    HIP_TRY(c, launch_reduce_partials(ins, sgrid * nbatch, sgrid * nbatch, 1, c->scalars.as<double>() + 24,
                                      c->stream), "count");
    double distinct = 0.0;
    HIP_TRY(c, hipMemcpyAsync(&distinct, c->scalars.as<double>() + 24, 8, hipMemcpyDeviceToHost, c->stream), "copy");
    HIP_TRY(c, launch_gather_scaled(c->gacc.as<double>(), d_subset, count, norm2, c->gbuf.as<double>(),
                                    c->stream), "gather");
    HIP_TRY(c, hipMemcpyAsync(g_out, c->gbuf.p, (size_t)count * 8, hipMemcpyDeviceToHost, c->stream), "copy g");
    Counters h2 = read_counters(c, &e);  // synchronizes
    if (e != hipSuccess) return hip_fail(c, e, "read counters");
    if (!(h2.flags & kFlagOverflow)) {
      c->ext_count = distinct;
      c->ext_alive = (double)h.alive;
      c->ps_keys = distinct;
      c->ps_slots = slots;
      c->ps_batches = nbatch;
      c->ps_passes = attempt + 1;
      c->ps_screened = 0;
      return SWCS_OK;
    }
    h2.flags &= ~kFlagOverflow;
    HIP_TRY(c, launch_store_counters(c->st.ctr, h2, c->stream), "counters");
    c->hc = h2;
    if (guess >= bound_d || attempt >= 16) return fail(c, SWCS_E_DEVICE, "sigma table overflow");
    guess = std::min(bound_d, 2.0 * guess);
  }
}

// Segments replayed side by side: as many as fit these bytes of logs and
// working copies and half of the memory there is, at least one (a large state's
// gate fills the device by itself, so there is nothing to gain from holding more).
constexpr size_t kReplayGroupBytes = (size_t)4 << 30;
// Records of a gate that one workgroup walks back (eight per thread); from
// there a launch of many blocks is faster.
constexpr u64 kWalkMaxRecords = 8192;

// Buffers for replaying *segs segments of n entries side by side.  Groups of up to
// 512 MB need no look at free memory (0.1 ms).  Where a block is refused it is tried
// with half as many segments, and one segment once more after everything that
// holds nothing has been given back.
static int replay_reserve(swcs_ctx* c, u64 n, int nseg, size_t gate_log_bytes, int* segs) {
  DevBuf* bufs[] = {&c->seg_states, &c->work, &c->ncut_cand, &c->ncut_state};
  const size_t seg_bytes = (size_t)c->seg * gate_log_bytes + n * 8 + (c->a_ncut ? n * 4 + ncut_select_bytes() : 0);
  size_t s = std::min<size_t>((size_t)nseg, std::max<size_t>(1, kReplayGroupBytes / seg_bytes));
  size_t held = 0;
  for (DevBuf* b : bufs) held += b->bytes;
  if (s * seg_bytes > std::max<size_t>(held, (size_t)512 << 20)) s = std::min(s, std::max<size_t>(1, (held + avail_bytes(c)) / 2 / seg_bytes));
  auto take = [&]() -> int {
    HIP_TRY(c, c->seg_states.ensure(s * c->seg * gate_log_bytes), "alloc pair logs");
    HIP_TRY(c, c->work.ensure(s * n * 8), "alloc working amplitudes");
    HIP_TRY(c, c->ctr_r.ensure(2 * s * c->seg * sizeof(u64)), "alloc log counters");
    return c->a_ncut ? ncut_reserve(c, (int)s, n) : SWCS_OK;
  };
  int r = take();
  for (bool all_given = false; r == SWCS_E_OOM && !all_given; r = take()) {
    for (DevBuf* b : bufs) b->release();
    if (s == 1) {
      release_scratch(c);
      all_given = true;
    }
    s = (s + 1) / 2;
  }
  *segs = (int)s;
  return r;
}

int swcs_param_gradients(swcs_ctx* c, double* dE, double* E_out) {
  if (!c) return SWCS_E_INVALID;
  if (!c->ansatz_valid) return fail(c, SWCS_E_STATE, "no ansatz applied from the reference");
  if (!dE && c->a_theta.size() > 0) return fail(c, SWCS_E_INVALID, "null dE_dtheta");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  const int64_t M = (int64_t)c->a_ops.size();  // unitaries (a parameter may drive two)
  const int64_t M_par = (int64_t)c->a_theta.size();
  hipError_t e;
  Counters hfin = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  const u64 n = hfin.n;
  int r;
  if (M == 0) {
    double numer = 0.0, norm2 = 0.0;
    r = energy_internal(c, n, &numer, &norm2);
    if (r) return r;
    if (E_out) *E_out = numer / norm2;
    return SWCS_OK;
  }
  r = energy_enqueue(c, n);
  if (r) return r;
  const double* nn = c->scalars.as<double>();
  const int seg = c->seg;
  const int nseg = (int)((M + seg - 1) / seg);
  const int grid = grid_blocks(c, n, 256);
  HIP_TRY(c, c->mu.ensure(n * 8), "alloc mu");
  HIP_TRY(c, c->gbuf.ensure((size_t)(M + 3) * 8), "alloc dE");  // and the energy's sums and the flags
  bool lds = n <= (u64)lds_chain_capacity();
  const GenGate* gens = nullptr;
  const int* kinds = nullptr;
  if (c->a_has_star) {
    r = upload_generators(c, c->a_gen.data(), c->a_kind.data(), M, &gens, &kinds);
    if (r) return r;
  }
  // Pair logs: at most one record per stored entry per gate, for every gate
  // (single-workgroup path, all segments replayed at once) or for a group of
  // segments at a time (HBM path); with overlapping generators each gate's
  // slot also holds up to one star record per stored entry.
  const size_t gate_log_bytes = n * (sizeof(PairRec) + (c->a_has_star ? sizeof(StarRec) : 0));
  HIP_TRY(c, launch_mu_init(c->st, c->sigma.as<double>(), n, nn, c->mu.as<double>(), c->stream), "mu init");
  const Busy busy(c->adjoint_busy);
  if (lds) {
    const hipError_t el = c->seg_states.ensure((size_t)M * gate_log_bytes);
    if (el != hipSuccess && el != hipErrorOutOfMemory) return hip_fail(c, el, "alloc pair logs");
    lds = el == hipSuccess;  // without room for every gate's log: in groups of segments
  }
  if (lds) {
    // Segments replayed side by side (one workgroup each), then one
    // workgroup walks every gate back with mu in LDS; the gate table of the
    // last apply call is reused.
    int r2 = upload_ckpt_table(c, nseg);
    if (r2) return r2;
    char* logs = (char*)c->seg_states.p;
    HIP_TRY(c, c->ctr_r.ensure((size_t)2 * M * sizeof(unsigned)), "alloc log counters");
    HIP_TRY(c, c->partial2.ensure(adjoint_lds_part_elems((int)M) * sizeof(double)), "alloc partials");
    TIMED(c, SWCS_K_ADJOINT_REPLAY_LDS, launch_adjoint_replay_lds(c->st.keys, (unsigned)n, c->gate_tab.as<GateDesc>(), kinds, gens, (int)M, seg,
                                          c->a_ncut ? 0.0 : c->a_eps, c->ckpt_ptrs.as<double*>(), c->ckpt_n.as<u64>(),
                                          logs, gate_log_bytes, c->ctr_r.as<unsigned>(), &c->st.ctr->flags, (unsigned)c->a_ncut,
                                          c->stream), "adjoint replay");
    TIMED(c, SWCS_K_ADJOINT_LDS, launch_adjoint_reverse_lds((unsigned)n, c->gate_tab.as<GateDesc>(), kinds, gens, (int)M, c->mu.as<double>(),
                                  logs, gate_log_bytes, c->ctr_r.as<unsigned>(), c->partial2.as<double>(), c->gbuf.as<double>(),
                                  c->stream), "adjoint");
  } else {
    // Per group of segments, the last first: restore the checkpoints into
    // working copies, replay the segments side by side (one launch per step
    // of a segment) logging the active pairs of every gate, then walk the
    // logs back.
    int gsegs = 1;
    r = replay_reserve(c, n, nseg, gate_log_bytes, &gsegs);
    if (r) return r;
    const u64 pstride = (u64)std::max(grid, 16);  // the walk's sixteen wavefronts
    HIP_TRY(c, c->partial2.ensure((size_t)M * pstride * 8), "alloc partials");
    HIP_TRY(c, launch_fill_u32(c->partial2.p, 0u, (u64)M * pstride * 2, c->stream), "zero partials");
    r = upload_ckpt_table(c, nseg);
    if (r) return r;
    double* W = c->work.as<double>();
    const double eps_r = c->a_ncut ? 0.0 : c->a_eps;
    const GateDesc* gates = c->gate_tab.as<GateDesc>();
    std::vector<u64> counts((size_t)2 * gsegs * seg);
    for (int hi = nseg; hi > 0; hi -= gsegs) {
      const int lo = std::max(0, hi - gsegs), segs = hi - lo;
      const int g_lo = lo * seg, g_hi = (int)std::min<int64_t>(M, (int64_t)hi * seg), ng = g_hi - g_lo;
      u64* lc = c->ctr_r.as<u64>();
      const ReplayGroup G{(char*)c->seg_states.p, gate_log_bytes, lc, lc + (size_t)gsegs * seg, kinds, n,
                          seg, lo, g_lo, (int)M};
      HIP_TRY(c, launch_restore(W, c->ckpt_ptrs.as<double*>(), c->ckpt_n.as<u64>(), lo, segs, n, c->stream), "restore");
      HIP_TRY(c, launch_fill_u32(lc, 0u, (u64)gsegs * seg * 4, c->stream), "zero log counters");
      for (int t = 0; t < std::min(seg, ng); ++t) {
        bool plain = false, star = false;
        for (int j = 0; j < segs; ++j) {
          const int g = (lo + j) * seg + t;
          if (g < g_hi) (c->a_kind[(size_t)g] ? star : plain) = true;
        }
        if (star)
          HIP_TRY(c, launch_gen_replay(c->st, W, n, gens, eps_r, G, t, segs, grid, c->stream), "generator replay");
        if (plain)
          TIMED(c, SWCS_K_GATE_REPLAY, launch_gate_replay(c->st, W, n, gates, eps_r, G, t, segs,
                                                          gate_grid(c, n, kReplayTile), c->stream), "replay");
        if (c->a_ncut)
          HIP_TRY(c, launch_ncut(W, n, c->st.keys, n, nullptr, 0, n, c->ncut_state.p, c->ncut_cand.as<unsigned>(), n,
                                 (unsigned)c->a_ncut, n, segs, c->stream), "ncut");
      }
      // Gates of few records are walked back by one workgroup, the others by a
      // launch each: the counts decide.
      HIP_TRY(c, hipMemcpyAsync(counts.data(), lc, (size_t)2 * gsegs * seg * 8, hipMemcpyDeviceToHost, c->stream), "copy");
      HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
      auto records = [&](int g) { return counts[(size_t)(g - g_lo)] + counts[(size_t)gsegs * seg + (size_t)(g - g_lo)]; };
      for (int g = g_hi; g > g_lo;) {
        int first = g;
        while (first > g_lo && records(first - 1) <= kWalkMaxRecords) --first;
        if (first < g) {
          TIMED(c, SWCS_K_ADJOINT_REC, launch_adjoint_walk(G, gates, gens, first, g, c->mu.as<double>(),
                                                           c->partial2.as<double>(), pstride, c->ckpt_n.as<u64>(), nseg,
                                                           c->stream), "reverse");
          g = first;
          continue;
        }
        --g;
        double* part = c->partial2.as<double>() + (size_t)g * pstride;
        TIMED(c, SWCS_K_ADJOINT_REC, launch_adjoint_rec(G.pairs(g), lc + (g - g_lo), c->mu.as<double>(), c->a_c[(size_t)g],
                                                        c->a_s[(size_t)g], part, grid, c->stream), "reverse");
        if (c->a_kind[(size_t)g])
          HIP_TRY(c, launch_adjoint_star(G.stars(g), G.star_counts + (g - g_lo), c->mu.as<double>(), c->a_gen[(size_t)g],
                                         part, grid, c->stream), "reverse stars");
      }
    }
    HIP_TRY(c, launch_reduce_partials(c->partial2.as<double>(), (int)pstride, (int)pstride, (int)M, c->gbuf.as<double>(),
                                      c->stream), "reduce");
  }
  // one copy brings derivatives, energy and flags
  std::vector<double> d_unit((size_t)M + 3);
  HIP_TRY(c, launch_pack_result(c->gbuf.as<double>() + M, nn, c->st.ctr, c->stream), "pack results");
  HIP_TRY(c, hipMemcpyAsync(d_unit.data(), c->gbuf.p, (size_t)(M + 3) * 8, hipMemcpyDeviceToHost, c->stream), "copy dE");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  const double nn_host[2] = {d_unit[(size_t)M], d_unit[(size_t)M + 1]};
  if ((unsigned)d_unit[(size_t)M + 2] & kFlagOverflow) {
    Counters hchk = read_counters(c, &e);
    if (e != hipSuccess) return hip_fail(c, e, "sync");
    hchk.flags &= ~kFlagOverflow;
    HIP_TRY(c, launch_store_counters(c->st.ctr, hchk, c->stream), "counters");
    c->hc = hchk;
    return fail(c, SWCS_E_DEVICE, "recomputation diverged from the forward run");
  }
  // per parameter: the unitaries it drives, each scaled by d(angle)/d(parameter)
  for (int64_t i = 0; i < M_par; ++i) dE[i] = 0.0;
  for (int64_t g = 0; g < M; ++g) dE[c->a_owner[(size_t)g]] += c->a_factor[(size_t)g] * d_unit[(size_t)g];
  if (E_out) *E_out = nn_host[0] / nn_host[1];
  return SWCS_OK;
}

int swcs_gate_active(swcs_ctx* c, int64_t* n_act, int64_t M) {
  if (!c) return SWCS_E_INVALID;
  if (M != c->last_M) return fail(c, SWCS_E_INVALID, "M differs from the last apply call");
  if (M == 0) return SWCS_OK;
  if (!n_act) return fail(c, SWCS_E_INVALID, "null n_act");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, hipMemcpyAsync(n_act, c->gate_n_act.p, (size_t)M * 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  return SWCS_OK;
}

int swcs_compact(swcs_ctx* c, int64_t* stored) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (h.alive < h.n) {
    int r = state_compact(c, &h);
    if (r) return r;
    r = build_filter(c, h.n, h.alive);
    if (r) return r;
    c->ansatz_valid = false;  // the checkpoints refer to the old positions
  }
  if (stored) *stored = (int64_t)h.n;
  return SWCS_OK;
}

int swcs_state_counts(swcs_ctx* c, int64_t* stored, int64_t* alive) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  const Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  if (stored) *stored = (int64_t)h.n;
  if (alive) *alive = (int64_t)h.alive;
  return SWCS_OK;
}

int swcs_pool_stats(swcs_ctx* c, double* keys, int64_t* table_slots, int32_t* batches, int32_t* passes,
                    int32_t* screened) {
  if (!c) return SWCS_E_INVALID;
  if (!c->ps_passes) return fail(c, SWCS_E_STATE, "no pool-gradient pass yet");
  if (keys) *keys = c->ps_keys;
  if (table_slots) *table_slots = (int64_t)c->ps_slots;
  if (batches) *batches = c->ps_batches;
  if (passes) *passes = c->ps_passes;
  if (screened) *screened = c->ps_screened;
  return SWCS_OK;
}

int swcs_gate_sizes(swcs_ctx* c, int64_t* n_in, int64_t M) {
  if (!c) return SWCS_E_INVALID;
  if (M != c->last_M) return fail(c, SWCS_E_INVALID, "M differs from the last apply call");
  if (M == 0) return SWCS_OK;
  if (!n_in) return fail(c, SWCS_E_INVALID, "null n_in");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, hipMemcpyAsync(n_in, c->gate_n_in.p, (size_t)M * 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  return SWCS_OK;
}

static int occupations_device(swcs_ctx* c, u64 n) {
  const int grid = grid_blocks(c, n, 256);
  HIP_TRY(c, c->partial.ensure((size_t)grid * (c->nso + 1) * 8), "alloc partial");
  HIP_TRY(c, c->occ.ensure((size_t)(c->nso + 1) * 8), "alloc occ");
  HIP_TRY(c, launch_occupations(c->st, n, c->nso, c->partial.as<double>(), grid, c->stream), "occupations");
  HIP_TRY(c, launch_reduce_partials(c->partial.as<double>(), grid, grid, c->nso + 1, c->occ.as<double>(), c->stream), "reduce");
  return SWCS_OK;
}

int swcs_occupations(swcs_ctx* c, double* n_out) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  if (!n_out) return fail(c, SWCS_E_INVALID, "null n_out");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  int r = occupations_device(c, h.n);
  if (r) return r;
  std::vector<double> tmp((size_t)c->nso + 1);
  HIP_TRY(c, hipMemcpyAsync(tmp.data(), c->occ.p, tmp.size() * 8, hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  for (int P = 0; P < c->nso; ++P) n_out[P] = tmp[(size_t)P] / tmp[(size_t)c->nso];
  return SWCS_OK;
}

int swcs_timer_start(swcs_ctx* c, int kernel_id) {
  if (!c) return SWCS_E_INVALID;
  if (kernel_id < SWCS_K_CHAIN_LDS || kernel_id > SWCS_K_STRINGS)
    return fail(c, SWCS_E_INVALID, "unknown kernel id");
  c->timer_kernel = kernel_id;
  c->ev_used = 0;
  return SWCS_OK;
}

int swcs_timer_stop(swcs_ctx* c, int64_t* launches, double* total_ms) {
  if (!c) return SWCS_E_INVALID;
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  double tot = 0.0;
  for (size_t i = 0; i < c->ev_used; ++i) {
    float ms = 0.0f;
    HIP_TRY(c, hipEventElapsedTime(&ms, c->ev_start[i], c->ev_stop[i]), "elapsed");
    tot += ms;
  }
  if (launches) *launches = (int64_t)c->ev_used;
  if (total_ms) *total_ms = tot;
  c->timer_kernel = 0;
  c->ev_used = 0;
  return SWCS_OK;
}

int64_t swcs_mlp_param_count(void) { return kMlpParams; }

int swcs_fock_diagonal(swcs_ctx* c, double* f_out) {
  if (!c) return SWCS_E_INVALID;
  if (!c->have_ints) return fail(c, SWCS_E_STATE, "integrals not set");
  if (!f_out) return fail(c, SWCS_E_INVALID, "null f_out");
  if (c->na != c->nb) return fail(c, SWCS_E_UNSUPPORTED, "closed-shell Fock needs n_alpha == n_beta");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  const int n = c->n;
  std::vector<double> f((size_t)n * n);
  HIP_TRY(c, hipMemcpyAsync(f.data(), c->fock.p, f.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream),
          "copy");
  HIP_TRY(c, hipStreamSynchronize(c->stream), "sync");
  for (int p = 0; p < n; ++p) f_out[p] = f[(size_t)p * n + p];
  return SWCS_OK;
}

int swcs_features(swcs_ctx* c, const float* d_prev_absg, const float* d_age, const float* d_count,
                  float* d_feat) {
  if (!c) return SWCS_E_INVALID;
  int r = check_ready(c);
  if (r) return r;
  if (!c->have_state) return fail(c, SWCS_E_STATE, "no current state");
  if (!d_prev_absg || !d_age || !d_count || !d_feat) return fail(c, SWCS_E_INVALID, "null device pointer");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  hipError_t e;
  Counters h = get_counters(c, &e);
  if (e != hipSuccess) return hip_fail(c, e, "read counters");
  r = occupations_device(c, h.n);
  if (r) return r;
  HIP_TRY(c, launch_features(c->ops.as<OpDesc>(), c->K_pool, c->fock.as<double>(), c->eri.as<double>(),
                             c->n, c->occ.as<double>(), d_prev_absg, d_age, d_count, d_feat, c->stream), "features");
  return SWCS_OK;
}

int swcs_mlp_forward(swcs_ctx* c, const float* d_W, const float* d_x, int64_t B, float* d_y,
                     float* d_act) {
  if (!c) return SWCS_E_INVALID;
  if (B < 0 || (B > 0 && (!d_W || !d_x || !d_y))) return fail(c, SWCS_E_INVALID, "bad mlp arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, launch_mlp_forward(d_W, d_x, B, d_y, d_act, c->stream), "mlp forward");
  return SWCS_OK;
}

int swcs_mlp_backward(swcs_ctx* c, const float* d_W, const float* d_x, const float* d_act,
                      const float* d_dy, int64_t B, float* d_dW) {
  if (!c) return SWCS_E_INVALID;
  if (B < 0 || !d_W || !d_dW || (B > 0 && (!d_x || !d_act || !d_dy)))
    return fail(c, SWCS_E_INVALID, "bad mlp arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  const long long rows = std::max<long long>(1, mlp_backward_partial_rows(B));
  HIP_TRY(c, c->mlp_partial.ensure((size_t)rows * kMlpParams * 4), "alloc partial");
  HIP_TRY(c, launch_mlp_backward(d_W, d_x, d_act, d_dy, B, d_dW, c->mlp_partial.as<float>(), rows,
                                 c->stream), "mlp backward");
  return SWCS_OK;
}

int swcs_mse(swcs_ctx* c, const float* d_y, const float* d_t, int64_t B, float* d_dy, float* d_loss) {
  if (!c) return SWCS_E_INVALID;
  if (B <= 0 || !d_y || !d_t || !d_dy || !d_loss) return fail(c, SWCS_E_INVALID, "bad mse arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, c->mse_partial.ensure((size_t)mse_partial_count(B) * 4), "alloc partial");
  HIP_TRY(c, launch_mse(d_y, d_t, B, d_dy, d_loss, c->mse_partial.as<float>(), c->stream), "mse");
  return SWCS_OK;
}

int swcs_log_abs(swcs_ctx* c, const double* d_g, int64_t n, float* d_t) {
  if (!c) return SWCS_E_INVALID;
  if (n < 0 || (n > 0 && (!d_g || !d_t))) return fail(c, SWCS_E_INVALID, "bad log_abs arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, launch_log_abs(d_g, n, d_t, c->stream), "log_abs");
  return SWCS_OK;
}

int swcs_add_feature(swcs_ctx* c, float* d_v, const float* d_feat, int64_t n, int col, int sign, float scale) {
  if (!c) return SWCS_E_INVALID;
  if (n < 0 || (n > 0 && (!d_v || !d_feat)) || col < 0 || col >= 16 || (sign != 1 && sign != -1) ||
      !(scale >= 0.0f && scale <= 1.0f))
    return fail(c, SWCS_E_INVALID, "bad add_feature arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, launch_add_feature(d_v, d_feat, n, col, (float)sign, scale, c->stream), "add_feature");
  return SWCS_OK;
}

int swcs_adam_step(swcs_ctx* c, float* d_W, float* d_m, float* d_v, const float* d_dW, int64_t P,
                   float lr, float b1, float b2, float eps, int step) {
  if (!c) return SWCS_E_INVALID;
  if (P <= 0 || !d_W || !d_m || !d_v || !d_dW || step < 1 || !(b1 >= 0 && b1 < 1) || !(b2 >= 0 && b2 < 1))
    return fail(c, SWCS_E_INVALID, "bad adam arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  HIP_TRY(c, launch_adam(d_W, d_m, d_v, d_dW, P, lr, b1, b2, eps, step, c->stream), "adam");
  return SWCS_OK;
}

int swcs_select(swcs_ctx* c, const float* d_score, const uint32_t* d_rand, int64_t K, int64_t n_top,
                int64_t n_rand, int32_t* d_idx) {
  if (!c) return SWCS_E_INVALID;
  if (K <= 0 || K > ((int64_t)1 << 31) - 1 || n_top < 0 || n_rand < 0 || n_top + n_rand > K ||
      !d_score || !d_idx || (n_rand > 0 && !d_rand))
    return fail(c, SWCS_E_INVALID, "bad select arguments");
  HIP_TRY(c, hipSetDevice(c->device), "hipSetDevice");
  const u64 need = select_scratch_elems(K);
  HIP_TRY(c, c->sel_scratch.ensure(need * 8), "alloc select scratch");
  TIMED(c, SWCS_K_SELECT, launch_select(d_score, d_rand, K, n_top, n_rand, d_idx, c->sel_scratch.as<u64>(), need,
                                        c->stream), "select");
  return SWCS_OK;
}

}  // extern "C"
