// Internal definitions shared by the HIP translation units of libswcs.
// Device data layout, hash tables, phase rules and host launch wrappers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

namespace swcs {

typedef unsigned long long u64;

// Amplitude bit pattern that marks a stored determinant as not part of the
// state (pruned, or never reached).  A quiet NaN no arithmetic produces.
constexpr u64 kDeadBits = 0x7ff8dead0000deadULL;
constexpr u64 kEmptyKey = 0ULL;  // no determinant of >= 1 electron has key 0

__host__ __device__ inline u64 mix64(u64 x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ULL;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebULL;
  x ^= x >> 31;
  return x;
}

__device__ inline bool is_dead(double a) { return (u64)__double_as_longlong(a) == kDeadBits; }
__device__ inline double dead_value() { return __longlong_as_double((long long)kDeadBits); }

// One operator of the pool, preprocessed on the host.
//   T = a+_P a+_Q a_S a_R (double) or a+_P a_Q (single, R = S = -1)
//   ann = bits annihilated by T, cre = bits created by T.
struct OpDesc {
  u64 ann;
  u64 cre;
  int P, Q, R, S;
};

// Sign of T acting on D (T must act: ann subset of D, cre disjoint from D).
// The rightmost ladder operator acts first; each contributes
// (-1)^(occupied spin-orbitals below its index) in the current determinant.
__device__ inline int phase_of_T(const OpDesc& op, u64 D) {
  int s;
  if (op.R < 0) {
    s = __popcll(D & ((1ULL << op.Q) - 1ULL));
    D ^= 1ULL << op.Q;
    s += __popcll(D & ((1ULL << op.P) - 1ULL));
  } else {
    s = __popcll(D & ((1ULL << op.R) - 1ULL));
    D ^= 1ULL << op.R;
    s += __popcll(D & ((1ULL << op.S) - 1ULL));
    D ^= 1ULL << op.S;
    s += __popcll(D & ((1ULL << op.Q) - 1ULL));
    D ^= 1ULL << op.Q;
    s += __popcll(D & ((1ULL << op.P) - 1ULL));
  }
  return (s & 1) ? -1 : 1;
}

// Open-addressing (linear probing) index from determinant key to position in
// the structure-of-arrays state.  Slots are 16 bytes so a probe touches one
// line for both key and index.  Capacity is a power of two.
struct HashSlot {
  u64 key;
  u64 idx;
};

__device__ inline long long hash_find(const HashSlot* __restrict__ tab, u64 mask, u64 key) {
  u64 h = mix64(key) & mask;
  while (true) {
    u64 k = tab[h].key;
    if (k == key) return (long long)tab[h].idx;
    if (k == kEmptyKey) return -1;
    h = (h + 1) & mask;
  }
}

// Insert a key known to be absent; concurrent inserts of other keys allowed.
__device__ inline void hash_insert_new(HashSlot* tab, u64 mask, u64 key, u64 idx) {
  u64 h = mix64(key) & mask;
  while (true) {
    u64 prev = atomicCAS(&tab[h].key, kEmptyKey, key);
    if (prev == kEmptyKey || prev == key) {
      tab[h].idx = idx;
      return;
    }
    h = (h + 1) & mask;
  }
}

// Accumulation table for the external sigma vector: key -> double.
struct AccSlot {
  u64 key;
  double val;
};

// Probe limit of the accumulation table: an insert that finds no free slot
// within this many probes fails (the caller raises kFlagOverflow and the host
// retries with a larger table), so a lookup that has not met its key within
// the same distance can stop.
constexpr u64 kAccMaxProbes = 4096;

// Adds v to the entry of key, inserting the key if needed.  Returns 2 if
// the key was inserted, 1 if it was present, 0 (adding nothing) if no slot
// within kAccMaxProbes is free.
__device__ inline int acc_add(AccSlot* tab, u64 mask, u64 key, double v) {
  u64 h = mix64(key) & mask;
  const u64 lim = mask < kAccMaxProbes ? mask : kAccMaxProbes;
  for (u64 probes = 0; probes <= lim; ++probes) {
    u64 k = tab[h].key;
    if (k == key) {
      unsafeAtomicAdd(&tab[h].val, v);
      return 1;
    }
    if (k == kEmptyKey) {
      u64 prev = atomicCAS(&tab[h].key, kEmptyKey, key);
      if (prev == kEmptyKey || prev == key) {
        unsafeAtomicAdd(&tab[h].val, v);
        return prev == kEmptyKey ? 2 : 1;
      }
    }
    h = (h + 1) & mask;
  }
  return 0;
}

__device__ inline bool acc_find(const AccSlot* __restrict__ tab, u64 mask, u64 key, double* v) {
  u64 h = mix64(key) & mask;
  const u64 lim = mask < kAccMaxProbes ? mask : kAccMaxProbes;
  for (u64 probes = 0; probes <= lim; ++probes) {
    u64 k = tab[h].key;
    if (k == key) {
      *v = tab[h].val;
      return true;
    }
    if (k == kEmptyKey) return false;
    h = (h + 1) & mask;
  }
  return false;
}

// kFlagOverflow: an append or table insert found no room (a bug guard: the
// host sizes buffers so it cannot happen).  kFlagStopped: a gate found too
// little capacity and did nothing; later gates of the chain skip too.
enum : unsigned int { kFlagOverflow = 1u, kFlagStopped = 2u };

// Entry counts of a chain that runs one launch per gate: n stored and alive ones
// of them before the gate, and what the gate adds, by atomics.
struct LiveCounts {
  u64 n;
  u64 alive;
  u64 app;
  long long dalive;
};

// Device counters of the state.  n: stored entries (alive or dead);
// alive: entries that are part of the state; flags: error bits.
// live: within a chain, three counts in rotation: gate g reads slot g - 1, adds
// to slot g and clears slot g + 1, so that no block has to be the last one and
// fold the sums in (gate launch at 40,000 entries 7.4 -> 7.0 us; what is left is
// the chain from counts and keys over index probe and partner to the append).
// k_live_begin fills the slot before the first gate, k_live_end leaves n and alive.
struct Counters {
  u64 n;
  u64 alive;
  unsigned int flags;
  unsigned int pad;
  u64 stop_gate;
  LiveCounts live[3];
};

__host__ __device__ inline unsigned live_slot(unsigned gate) { return gate % 3u; }
__host__ __device__ inline unsigned live_before(unsigned gate) { return (gate + 2u) % 3u; }
__host__ __device__ inline unsigned live_after(unsigned gate) { return (gate + 1u) % 3u; }

// Stored and alive entries by a slot that no block of the launch changes: plain
// loads, which a whole launch serves from its caches (loads that bypass them,
// by every wavefront of some hundred blocks, queued up at one memory channel).
__device__ inline void live_load(const LiveCounts* L, u64 cap, u64* n, u64* alive) {
  const u64 n0 = L->n, app = L->app;
  *n = n0 + (app < cap - n0 ? app : cap - n0);
  *alive = (u64)((long long)L->alive + L->dalive);
}

// Start of a gate, the same in every thread of the launch: whether it runs, and
// the entry counts.  A stopped chain skips every later gate; the host resumes it
// after growing.  Appends are bounded by `grow` times the alive sources and by
// the number of keys not yet stored (max_keys = size of the electron-number
// sector), so n_in + min(grow alive_in, max_keys - n_in) <= cap guarantees the
// gate fits.  Nothing has been modified when it stops.
__device__ inline bool gate_begin(Counters* ctr, unsigned gate, u64 cap, u64 max_keys, unsigned grow, u64* n_in,
                                  u64* gate_n_in) {
  const unsigned fl = ctr->flags;
  u64 n, alive;
  live_load(&ctr->live[live_before(gate)], cap, &n, &alive);
  *n_in = n;
  if (fl & kFlagStopped) return false;
  const u64 room = max_keys > n ? max_keys - n : 0, most = grow * alive;
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (n + (most < room ? most : room) > cap) {
    if (first) {
      ctr->stop_gate = gate;
      atomicOr(&ctr->flags, kFlagStopped);
    }
    return false;
  }
  if (first) {
    LiveCounts& own = ctr->live[live_slot(gate)];
    __hip_atomic_store(&own.n, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&own.alive, alive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    LiveCounts& next = ctr->live[live_after(gate)];
    __hip_atomic_store(&next.app, (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&next.dalive, 0LL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (gate_n_in) *gate_n_in = alive;
  }
  return true;
}

// Waits until this wavefront's device-scope atomics (and its other memory
// operations) are done.  Before a ticket that announces only such atomics this
// is all the order the last block needs; a device-scope fence would also write
// the L2 back, which cost each gate launch several microseconds and a launch of
// many blocks tens.
__device__ inline void device_atomics_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sum over the wavefront, in lane 63: row steps and row broadcasts in the vector
// units (six shuffles through LDS take some 700 cycles, and are most of a step
// where one workgroup walks a chain back).  Every lane of the wavefront calls it.
template <int CTRL, int ROWS>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ inline double wave_sum63(double v) {
  v = dpp_add<0xb1, 0xf>(v);   // quad_perm 1, 0, 3, 2
  v = dpp_add<0x4e, 0xf>(v);   // quad_perm 2, 3, 0, 1
  v = dpp_add<0x141, 0xf>(v);  // row_half_mirror
  v = dpp_add<0x140, 0xf>(v);  // row_mirror: every lane of a row of 16 has its sum
  v = dpp_add<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
  return v;
}

// Barrier of a block that shares nothing but LDS between its threads: waits for
// LDS operations only, so loads made ahead and stores that no thread of the block
// reads stay in flight across it (__syncthreads waits for them: a microsecond
// where they go to memory).
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders a wavefront's own LDS accesses (its LDS operations execute in order;
// this keeps the compiler from moving or reusing them across the point).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Integrals on the device, spin-free spatial arrays.
struct Ints {
  const double* h;    // n*n
  const double* eri;  // (pq|rs) packed by its 8-fold symmetry: eri_packed_index
  const double* J;    // n*n, J[p*n+q] = (pp|qq)
  const double* K;    // n*n, K[p*n+q] = (pq|qp)
  double ecore;
  int n;
};

// Position of (pq|rs) in the packed array: pair indices pq = p (p + 1) / 2 +
// q (p >= q), rs likewise, then pq (pq + 1) / 2 + rs (pq >= rs).  The array
// has m (m + 1) / 2 entries, m = n (n + 1) / 2 (61,776 doubles, 494 KB, at
// n = 26 against 3.7 MB for n^4), so the lookups of the sigma and gradient
// kernels stay in L2.
// Orbital indices are below 64, so every product fits 24 bits; the masks let
// the compiler use full-rate 24-bit multiplies instead of 32-bit ones.
__host__ __device__ inline unsigned eri_packed_index(unsigned p, unsigned q, unsigned r, unsigned s) {
  p &= 63u;
  q &= 63u;
  r &= 63u;
  s &= 63u;
  const unsigned hi1 = p >= q ? p : q, lo1 = p >= q ? q : p;
  const unsigned hi2 = r >= s ? r : s, lo2 = r >= s ? s : r;
  const unsigned pq = ((hi1 * hi1 + hi1) >> 1) + lo1, rs = ((hi2 * hi2 + hi2) >> 1) + lo2;
  const unsigned a = (pq >= rs ? pq : rs) & 0xFFFu, b = pq >= rs ? rs : pq;
  return ((a * a + a) >> 1) + b;
}

__device__ inline double eri_sp(const Ints& I, int p, int q, int r, int s) {
  return I.eri[eri_packed_index((unsigned)p, (unsigned)q, (unsigned)r, (unsigned)s)];
}

// Spin-orbital (PQ|RS) with the spin deltas.
__device__ inline double eri_so(const Ints& I, int P, int Q, int R, int S) {
  if (((P ^ Q) & 1) || ((R ^ S) & 1)) return 0.0;
  return eri_sp(I, P >> 1, Q >> 1, R >> 1, S >> 1);
}

// <D'|H|D> for D' = a+_A a_I D (same spin, I in D, A not in D).
__device__ inline double single_element(const Ints& I, u64 D, int Ih, int A) {
  int s = __popcll(D & ((1ULL << Ih) - 1ULL));
  u64 x = D ^ (1ULL << Ih);
  s += __popcll(x & ((1ULL << A) - 1ULL));
  int a = A >> 1, i = Ih >> 1, n = I.n;
  double v = I.h[a * n + i];
  u64 y = D;
  while (y) {
    int Q = __ffsll((long long)y) - 1;
    y &= y - 1;
    int q = Q >> 1;
    v += eri_sp(I, a, i, q, q);
    if (((Q ^ A) & 1) == 0) v -= eri_sp(I, a, q, q, i);
  }
  return (s & 1) ? -v : v;
}

// <D'|H|D> for D' = a+_A a+_B a_J a_I D with I < J in D and A < B not in D.
__device__ inline double double_element(const Ints& I, u64 D, int Ih, int Jh, int A, int B) {
  int s = __popcll(D & ((1ULL << Ih) - 1ULL));
  u64 x = D ^ (1ULL << Ih);
  s += __popcll(x & ((1ULL << Jh) - 1ULL));
  x ^= 1ULL << Jh;
  s += __popcll(x & ((1ULL << B) - 1ULL));
  x ^= 1ULL << B;
  s += __popcll(x & ((1ULL << A) - 1ULL));
  double v = eri_so(I, A, Ih, B, Jh) - eri_so(I, A, Jh, B, Ih);
  return (s & 1) ? -v : v;
}

// Enumeration of the spin-conserving single and double excitations of a
// determinant with na alpha and nb beta electrons in n spatial orbitals.
// Connection c in [0, C) decodes to (holes, particles) in spin-orbitals.
struct ExcSpace {
  int n, na, nb;
  int va, vb;        // virtual counts
  long long s_a, s_b, d_aa, d_bb, d_ab;  // counts per class
  long long total;
};

inline ExcSpace make_exc_space(int n, int na, int nb) {
  ExcSpace e;
  e.n = n; e.na = na; e.nb = nb;
  e.va = n - na; e.vb = n - nb;
  e.s_a = (long long)na * e.va;
  e.s_b = (long long)nb * e.vb;
  e.d_aa = (long long)na * (na - 1) / 2 * ((long long)e.va * (e.va - 1) / 2);
  e.d_bb = (long long)nb * (nb - 1) / 2 * ((long long)e.vb * (e.vb - 1) / 2);
  e.d_ab = (long long)na * nb * e.va * e.vb;
  e.total = e.s_a + e.s_b + e.d_aa + e.d_bb + e.d_ab;
  return e;
}

// <D'|H|D> for the connection decoded above.
__device__ inline double connection_element(const Ints& I, u64 D, int nh, int h0, int h1, int p0,
                                            int p1) {
  if (nh == 1) return single_element(I, D, h0, p0);
  return double_element(I, D, h0, h1, p0, p1);
}

// One gate of an ansatz as the device sees it.
struct GateDesc {
  OpDesc op;
  double c;  // cos(theta)
  double s;  // sin(theta)
};

// A spin-complemented generator G = A1 + s A2 whose rows share spin-orbitals,
// applied as one gate exp(theta G) (k_generator.hip).
struct GenGate {
  OpDesc op1, op2;
  double c, sn;   // cos theta, sin theta: pairs of row 1
  double sn2;     // s sin theta: pairs of row 2
  double c2, s2;  // cos(sqrt(2) theta), sin(sqrt(2) theta): stars
  double rt;      // 1 / sqrt(2)
  double sg;      // s = +-1
};

// Largest state the single-workgroup LDS kernels hold (24 B per entry for
// the forward chain, 32 B for the adjoint sweep: 128 KB of LDS).
constexpr int kLdsCap = 4096;

// Multi-block gate kernels in HBM: threads per block, entries per thread and
// tile sizes (a tile's appended keys / logged pairs are staged in LDS).
constexpr int kDiagLanes = 8;  // lanes per determinant in k_diag
constexpr int kGateThreads = 1024;
constexpr int kGateItems = 2;                              // listed entries per thread and round
constexpr int kGateTile = kGateThreads * kGateItems;       // listed entries per round
// Keys per thread in the gate's scan: wide tiles for state arrays of at least
// kGateWideCap entries, narrow ones below (more blocks for small states).
constexpr int kGateScanWide = 16;
constexpr int kGateScanNarrow = 2;
constexpr u64 kGateWideCap = 1ULL << 21;
// entries per tile of the gate kernel for a state array of capacity cap
__host__ __device__ inline int gate_scan_tile(u64 cap) {
  return kGateThreads * (cap >= kGateWideCap ? kGateScanWide : kGateScanNarrow);
}
constexpr int kReplayTile = 2048;

// ---------------------------------------------------------------- host side
struct DeviceState {
  u64* keys = nullptr;
  double* amps = nullptr;
  HashSlot* hash = nullptr;
  Counters* ctr = nullptr;
  u64 cap = 0;        // SoA capacity
  u64 hmask = 0;      // hash capacity - 1
  unsigned* filt = nullptr;  // presence filter of the alive keys (1 bit per hash)
  u64 fmask = 0;             // filter bits - 1
  double* diag = nullptr;    // diagonal elements H_DD of the stored entries (launch_diag)
};

// Presence filter: one bit per (independent) hash of an alive key, about 16
// bits per key so that it stays in L2; a clear bit proves absence, so most
// probes for determinants that are not in the state never reach the table.
__device__ inline u64 filter_bit(u64 key, u64 fmask) {
  return mix64(key ^ 0xd6e8feb86659fd93ULL) & fmask;
}

__device__ inline bool filter_maybe(const unsigned* __restrict__ filt, u64 fmask, u64 key) {
  const u64 b = filter_bit(key, fmask);
  return (filt[b >> 5] >> (b & 31)) & 1u;
}

// Launch wrappers (defined in the .hip files).  All enqueue on `stream`.
struct PairRec;
struct StarRec;
hipError_t launch_gen_gate(const DeviceState& st, const GenGate& g, double eps, u64* gate_n_in,
                           unsigned gate_index, u64 max_keys, int grid, hipStream_t stream,
                           u64* gate_n_act = nullptr);
// to[0..2] = the energy's two sums and the error flags.
hipError_t launch_pack_result(double* to, const double* sums, const Counters* ctr, hipStream_t stream);
// The counts before gate g of a chain, from the state's; the state's counts after
// the chain's gates up to M, or up to the one that stopped it.
hipError_t launch_live_begin(const DeviceState& st, unsigned g, hipStream_t stream);
hipError_t launch_live_end(const DeviceState& st, unsigned M, hipStream_t stream);
struct ReplayGroup;
hipError_t launch_gen_replay(const DeviceState& st, double* work, u64 n, const GenGate* gens, double eps,
                             const ReplayGroup& G, int step, int segs, int grid, hipStream_t stream);
hipError_t launch_adjoint_star(const StarRec* slog, const u64* scount, double* mu, const GenGate& g,
                               double* partial, int grid, hipStream_t stream);
hipError_t launch_fill_u32(void* p, unsigned v, u64 words, hipStream_t stream);
hipError_t launch_store_counters(Counters* ctr, const Counters& v, hipStream_t stream);
hipError_t launch_clear_flag(Counters* ctr, unsigned bit, hipStream_t stream);
hipError_t launch_nan_if_flag(const Counters* ctr, unsigned bit, double* out, long long count,
                              hipStream_t stream);
hipError_t launch_hash_clear(HashSlot* tab, u64 slots, hipStream_t stream);
hipError_t launch_hash_build(const DeviceState& st, u64 n, hipStream_t stream);
hipError_t launch_gate(const DeviceState& st, const OpDesc& op, double c, double sn, double eps,
                       u64* gate_n_in, unsigned gate_index, u64 max_keys, int grid,
                       hipStream_t stream, u64* gate_n_act = nullptr);
hipError_t launch_prune_all(const DeviceState& st, double eps, unsigned gate, int grid, hipStream_t stream);
hipError_t launch_hash_build_dev(const DeviceState& st, int grid, hipStream_t stream);
hipError_t launch_filter_build(const DeviceState& st, u64 n, int grid, hipStream_t stream);
hipError_t launch_reset_reference(const DeviceState& st, u64 ref, hipStream_t stream);
// N_CUT selection on `states` amplitude arrays amps + y * stride of the same
// keys: select holds ncut_select_bytes() per state, zeroed before the first
// use; cand room for one index per entry (cand_stride apart).  n_most bounds
// the stored entries for the launch grid.
size_t ncut_select_bytes();
hipError_t launch_ncut(double* amps, u64 stride, const u64* keys, u64 n_host, Counters* ctr, unsigned gate, u64 cap, void* select,
                       unsigned* cand, u64 cand_stride, unsigned ncut, u64 n_most, int states, hipStream_t stream);
int lds_chain_capacity();
hipError_t launch_chain_lds(const DeviceState& st, const GateDesc* gates, const int* kinds, const GenGate* gens,
                            int g0, int M, double eps, int prune_first, double* const* ckpt, u64* ckpt_n, int seg,
                            u64* gate_n_in, u64* gate_n_act, u64 max_keys, unsigned ncut, hipStream_t stream);
hipError_t launch_adjoint_replay_lds(const u64* keys, unsigned n, const GateDesc* gates, const int* kinds,
                                     const GenGate* gens, int M, int seg, double eps, const double* const* ckpt,
                                     const u64* ckpt_n, char* logbuf, size_t log_bytes, unsigned* logcnt,
                                     unsigned* flags, unsigned ncut, hipStream_t stream);
hipError_t launch_adjoint_reverse_lds(unsigned n, const GateDesc* gates, const int* kinds, const GenGate* gens, int M,
                                      const double* mu_init, const char* logbuf, size_t log_bytes,
                                      const unsigned* logcnt, double* dE_part, double* dE, hipStream_t stream);
size_t adjoint_lds_part_elems(int M);
hipError_t launch_gate_replay(const DeviceState& st, double* work, u64 n, const GateDesc* gates, double eps,
                             const ReplayGroup& G, int step, int segs, int grid, hipStream_t stream);
hipError_t launch_adjoint_walk(const ReplayGroup& G, const GateDesc* gates, const GenGate* gens, int g_lo, int g_hi,
                               double* mu, double* partial, u64 pstride, const u64* ckpt_n, int nseg,
                               hipStream_t stream);
hipError_t launch_adjoint_rec(const PairRec* log, const u64* log_count, double* mu, double c,
                              double sn, double* partial, int grid, hipStream_t stream);
hipError_t launch_ckpt_save(const DeviceState& st, unsigned gate, double* dst, u64* dst_n, int grid,
                            hipStream_t stream);
hipError_t launch_restore(double* work, const double* const* ckpt, const u64* ckpt_n, int seg0, int segs, u64 n,
                          hipStream_t stream);
hipError_t launch_mark_dead_range(double* amps, u64 lo, u64 hi, hipStream_t stream);
hipError_t launch_sigma_proj(const DeviceState& st, const Ints& I, const ExcSpace& E, u64 n,
                             double* sigma, double* partial_num, double* partial_norm, int grid,
                             hipStream_t stream);
int pairwise_capacity();
hipError_t launch_sigma_pairwise(const DeviceState& st, const Ints& I, u64 n, double* sigma,
                                 double* partial, int grid, hipStream_t stream);
hipError_t launch_diag(const DeviceState& st, const Ints& I, u64 n, int grid, hipStream_t stream);
hipError_t launch_holepair_emit(const DeviceState& st, u64 n, int n_spatial, int na, int nb, int shift,
                                u64* out_key, unsigned* out_val, int grid, hipStream_t stream);
hipError_t launch_sigma_diag(const DeviceState& st, const Ints& I, u64 n, double* sigma, int grid,
                             hipStream_t stream);
hipError_t launch_holepair_sigma(const DeviceState& st, const Ints& I, int na, u64 n, const u64* skey,
                                 const unsigned* sidx, int shift, u64 total, int cls, double* sigma, int grid,
                                 hipStream_t stream);
// sigma_P by spin strings (k_strings.hip).
size_t str_slot_bytes();
constexpr unsigned kStrSampleBlocks = 64;  // lines of five counts
unsigned str_sample_blocks(u64 cnt);
hipError_t launch_str_sample(const DeviceState& st, u64 cnt, unsigned* out, hipStream_t stream);
hipError_t launch_str_emit(const DeviceState& st, u64 cnt, int n, int shift, u64* ra, u64* rb, int grid, hipStream_t stream);
hipError_t launch_str_groups(const DeviceState& st, const u64* rec, u64 alive, int n, int shift, int spin, u64* skey,
                             double* sval, unsigned* oth, void* tab, u64 slots, int grid, hipStream_t stream);
hipError_t launch_str_sigma(const Ints& I, const u64* rec, u64 alive, int shift, int nocc, const u64* skey,
                            const double* sval, const unsigned* oth, const void* tab, u64 slots, bool adj,
                            double* sigma, int grid, hipStream_t stream);
hipError_t launch_sigma_dots(const DeviceState& st, const double* sigma, u64 n, double* partial,
                             int grid, hipStream_t stream);
hipError_t launch_mu_init(const DeviceState& st, const double* sigma, u64 n, const double* nn,
                          double* mu, hipStream_t stream);
hipError_t launch_reduce_partials(const double* partial, int count, int stride, int nvec,
                                  double* out, hipStream_t stream);
// Full-pool gradients by sort and join (k_join.hip); kJoinRunHost records
// per step of the join kernel.
constexpr u64 kJoinRunHost = 2048;
// Largest record count for which SWCS_POOL_AUTO takes the join.
constexpr u64 kJoinAutoMaxRecords = 1ULL << 31;
bool join_format(const ExcSpace& E, u64 n, u64 R, int* kb, int* bh, int* bp, int* orb);
hipError_t launch_join_emit(const DeviceState& st, const ExcSpace& E, u64 n, u64* recs, u64 cap_recs,
                            u64* cursor, int kb, int bh, int bp, int orb, void* src, int grid, hipStream_t stream);
// Gradient terms of the join partitioned by operator: bin b = k mod 2^lb
// holds the terms of operators k = j 2^lb + b (j < kJoinTermSlots) as
// (j, value) at w / j arrays [b cap, b cap + cap), filled up to cursor[b];
// lb < 0 sends every term straight to g[k] with a device-scope add.
constexpr int kJoinTermSlots = 8192;  // operators per bin (one FP64 LDS table of 64 KB)
constexpr int kJoinMaxBinsLog = 8;
// Small pools take up to 2^6 bins of some 256 operators: a block of the term sums
// then adds few sums to memory (22,750 operators, 1.8e6 terms: 33 us with four bins
// of up to 8,192, 8 with 64).
constexpr int kJoinBinsLog = 6;
struct JoinTerms {
  int lb;
  u64 cap;
  u64* cursor;
  double* w;
  unsigned short* j;
};
hipError_t launch_join_reduce(const DeviceState& st, const u64* recs, u64 R, const u64* cursor, int kb, int bh,
                              int bp, int orb, const void* src, u64 n, const Ints& I, const ExcSpace& E,
                              const int* optab, int nsp, const unsigned char* selected, double* gacc,
                              JoinTerms terms, double* inserted, int grid, hipStream_t stream);
// Sums the binned terms into g[K] (nothing when terms.lb < 0).
hipError_t launch_join_terms(JoinTerms terms, double* gacc, long long K, hipStream_t stream);
// Pool gradients from the three-body density matrix (k_rdm.hip; sizes in
// doubles).
struct RdmFmt;
size_t rdm_gamma_elems(int n);
size_t rdm_two_elems(int n);
size_t rdm_vtab_elems(int n);
size_t rdm_part_elems(int n);
hipError_t launch_rdm_emit(const DeviceState& st, u64 n, int ne, RdmFmt fm, int nbatch, int batch, u64 smask,
                           u64* recs, u64 cap, u64* cursor, int grid, hipStream_t stream);
hipError_t launch_rdm_clear(int n_spatial, double* g3, hipStream_t stream);
hipError_t launch_rdm_count(const u64* recs, u64 R, int sort_bits, double* partial, int grid, hipStream_t stream);
hipError_t launch_rdm_pairs(const DeviceState& st, u64 n, int n_spatial, int ne, RdmFmt fm, int sort_bits,
                            const u64* recs, u64 R, double* g3, int grid, hipStream_t stream);
size_t rdm_member_bytes();
int rdm_row_bits();
hipError_t launch_rdm_members(const DeviceState& st, u64 n, int n_spatial, int ne, RdmFmt fm, int sort_bits,
                              const u64* recs, u64 R, void* mem, u64* list, u64* cursor, int grid,
                              hipStream_t stream);
hipError_t launch_rdm_rows(int n_spatial, const u64* list, u64 Q, unsigned* row_end, const void* mem, u64 R, double* g3,
                           hipStream_t stream);
hipError_t launch_rdm_diag(const DeviceState& st, u64 n, int n_spatial, double* g3, int grid, hipStream_t stream);
hipError_t launch_rdm_gradients(const Ints& I, const double* eri, int na, int nb, double* g3, double* g2, double* vtab, double* part, double* bs,
                                const OpDesc* ops, const int* subset, long long count, const double* norm2,
                                double* out, hipStream_t stream);
hipError_t launch_sigma_push(const DeviceState& st, const Ints& I, const ExcSpace& E, u64 n,
                             AccSlot* tab, u64 tmask, int nbatch, int batch, double* inserted,
                             int grid, hipStream_t stream);
hipError_t launch_pool_contract_det(const DeviceState& st, const ExcSpace& E, int n_spatial, u64 n,
                                   const int* optab, int nsp, const unsigned char* selected,
                                   const AccSlot* tab, u64 tmask, int nbatch, int batch,
                                   double* gacc, int grid, hipStream_t stream);
hipError_t launch_query_set(const DeviceState& st, const ExcSpace& E, int n_spatial, u64 n,
                            const int* optab, int nsp, const unsigned char* selected,
                            AccSlot* tab, u64 tmask, int count_only, u64* counter, int grid,
                            hipStream_t stream, int nbatch = 1, int batch = 0, unsigned* qf = nullptr,
                            u64 qfmask = 0);
hipError_t launch_query_ops(const DeviceState& st, u64 n, const OpDesc* ops, const int* subset,
                            long long n_sub, AccSlot* tab, u64 tmask, int count_only, u64* counter,
                            hipStream_t stream, int nbatch = 1, int batch = 0, unsigned* qf = nullptr,
                            u64 qfmask = 0);
hipError_t launch_contract_ops(const DeviceState& st, u64 n, const OpDesc* ops, const int* subset,
                               long long n_sub, const AccSlot* tab, u64 tmask, double* gslot,
                               hipStream_t stream, int nbatch = 1, int batch = 0);
hipError_t launch_sigma_push_into(const DeviceState& st, const Ints& I, const ExcSpace& E, u64 n,
                                  AccSlot* tab, u64 tmask, int grid, hipStream_t stream, int nbatch = 1, int batch = 0,
                                  const unsigned* qf = nullptr, u64 qfmask = 0);
hipError_t launch_gather_scaled(const double* gacc, const int* subset, long long count,
                                const double* norm2, double* out, hipStream_t stream);
hipError_t launch_mark_selected(const int* subset, long long count, unsigned char* selected,
                                hipStream_t stream);
hipError_t launch_occupations(const DeviceState& st, u64 n, int nso, double* partial, int grid,
                              hipStream_t stream);
hipError_t launch_compact_alive(const DeviceState& st, u64 n, const double* vals, u64* out_keys,
                                double* out_amps, u64* d_count, u64* scratch, u64 scratch_elems,
                                hipStream_t stream);
hipError_t radix_sort_pairs(u64* keys, u64* vals, u64* tmp_keys, u64* tmp_vals, u64 count,
                            int key_bits, u64* scratch, u64 scratch_elems, hipStream_t stream,
                            u64** out_keys = nullptr, u64** out_vals = nullptr);
// Same with 32-bit payloads.
hipError_t radix_sort_pairs32(u64* keys, unsigned* vals, u64* tmp_keys, unsigned* tmp_vals, u64 count,
                              int key_bits, u64* scratch, u64 scratch_elems, hipStream_t stream,
                              u64** out_keys, unsigned** out_vals);
// Keys only (no LDS or traffic for values); out_keys as above.
hipError_t radix_sort_keys(u64* keys, u64* tmp_keys, u64 count, int key_bits, u64* scratch,
                           u64 scratch_elems, hipStream_t stream, u64** out_keys);
u64 radix_sort_scratch_elems(u64 count);
u64 compact_scratch_elems(u64 n);
// Sorted export of a state of at most export_small_max() stored entries.
u64 export_small_max();
hipError_t launch_export_small(const DeviceState& st, u64 n, u64 alive, const double* vals, u64* out_keys,
                               double* out_vals, hipStream_t stream);

// Screener.
hipError_t launch_fock(const double* h, const double* eri, int n, int n_occ, double* fock,
                       hipStream_t stream);
hipError_t launch_features(const OpDesc* ops, long long K, const double* fock, const double* eri,
                           int n, const double* occ, const float* prev_absg, const float* age,
                           const float* count, float* feat, hipStream_t stream);
hipError_t launch_mlp_forward(const float* W, const float* x, long long B, float* y, float* act,
                              hipStream_t stream);
long long mlp_backward_partial_rows(long long B);
hipError_t launch_mlp_backward(const float* W, const float* x, const float* act, const float* dy,
                               long long B, float* dW, float* partial, long long partial_rows,
                               hipStream_t stream);
int mse_partial_count(long long B);
hipError_t launch_mse(const float* y, const float* t, long long B, float* dy, float* loss,
                      float* partial, hipStream_t stream);
hipError_t launch_add_feature(float* v, const float* feat, long long n, int col, float sign, float scale,
                              hipStream_t stream);
hipError_t launch_log_abs(const double* g, long long n, float* t, hipStream_t stream);
hipError_t launch_sanitize_subset(const int* in, long long count, long long K, int* out,
                                  hipStream_t stream);
hipError_t launch_nan_invalid(const int* in, long long count, long long K, double* g,
                              hipStream_t stream);
hipError_t launch_adam(float* W, float* m, float* v, const float* g, long long P, float lr,
                       float b1, float b2, float eps, int step, hipStream_t stream);
hipError_t launch_select(const float* score, const uint32_t* rnd, long long K, long long n_top,
                         long long n_rand, int* idx, u64* scratch, u64 scratch_elems,
                         hipStream_t stream);
u64 select_scratch_elems(long long K);

constexpr int kMlpIn = 16;
constexpr int kMlpHidden = 128;
constexpr long long kMlpParams = kMlpIn * kMlpHidden + kMlpHidden + kMlpHidden * kMlpHidden +
                                 kMlpHidden + kMlpHidden + 1;

}  // namespace swcs
