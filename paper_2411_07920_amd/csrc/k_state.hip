// State kernels in HBM: the multi-block gate with fused pruning and wave-
// aggregated appends, the reverse (adjoint) step, hash index maintenance,
// checkpoints and small utilities.  The per-entry arithmetic is in
// gate_ops.h, shared with the LDS-resident single-workgroup kernels.
//
// State layout in HBM (structure of arrays, one entry per stored determinant):
//   keys[cap]  uint64 determinant bit strings (never reordered within a run)
//   amps[cap]  float64 amplitudes, kDeadBits for entries not in the state
//   hash[2^k]  16-byte slots {key, index}, linear probing, load <= 1/2
#include <algorithm>

#include "gate_ops.h"
#include "select_ops.h"

namespace swcs {

// One gate over the stored entries, in three phases per tile of
// kGateThreads * SCAN entries:
//   scan   -- every thread loads SCAN keys (coalesced) and the
//             entries the operator or its adjoint acts on are listed in LDS
//             (16-bit tile offsets), so that the next phase runs on full
//             wavefronts whatever the active fraction;
//   update -- rounds of kGateTile listed entries, kGateItems per thread
//             staged together (gate_entries_list): index probe, amplitudes,
//             update with fused pruning; the new partner keys of a round are
//             staged in LDS;
//   append -- one atomic on the append counter per round, then coalesced
//             writes of the new keys and amplitudes and their index inserts
//             (the probe that found the key absent has just brought its
//             slot's line into L2, so the insert's CAS hits there; inserts
//             deferred to a separate pass cost more than they saved).
// SCAN = 16 for large states (more entries in flight per block), 2 for
// states of up to a few hundred thousand entries (more blocks).
template <int SCAN>
__global__ void __launch_bounds__(kGateThreads, 8)
k_gate(u64* __restrict__ keys, double* __restrict__ amps, HashSlot* __restrict__ hash, u64 hmask,
       u64 cap, Counters* __restrict__ ctr, OpDesc op, double c, double sn, double eps,
       u64* __restrict__ gate_n_in, unsigned gate_index, u64 max_keys, u64* __restrict__ gate_n_act) {
  constexpr int kScan = kGateThreads * SCAN;  // entries per tile (< 2^16)
  __shared__ unsigned short s_act[kScan];
  __shared__ u64 s_key[kGateTile];
  __shared__ double s_val[kGateTile];
  __shared__ unsigned s_nact, s_cnt;
  __shared__ u64 s_base;
  __shared__ long long s_wsum[kGateThreads / 64];
  // In a launch that is mostly latency, the first tile's keys are on their way
  // before the entry count is known; wide tiles of blocks beyond it would be
  // read for nothing.
  constexpr bool kAhead = SCAN <= 2;
  u64 D[SCAN];
  if (kAhead) {
#pragma unroll
    for (int j = 0; j < SCAN; ++j) {
      const u64 i = (u64)blockIdx.x * kScan + (u64)j * kGateThreads + threadIdx.x;
      D[j] = keys[i < cap ? i : 0];
    }
  }
  u64 n_in;
  const bool run = gate_begin(ctr, gate_index, cap, max_keys, 1, &n_in, gate_n_in);
  if (!run) return;  // the same in every thread
  if (threadIdx.x == 0) {
    s_nact = 0;
    s_cnt = 0;
  }
  __syncthreads();
  LiveCounts* __restrict__ own = &ctr->live[live_slot(gate_index)];
  long long dalive = 0;
  u64 nact = 0;
  const int lane = __lane_id();
  const u64 below = (1ULL << lane) - 1ULL;
  const u64 ntiles = (n_in + kScan - 1) / kScan;
  const GlobalStore S{keys, amps, hash, hmask};
  for (u64 t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const u64 base = t * (u64)kScan;
    // scan: keys of the tile, active entries listed in LDS
    {
      if (!kAhead || t != blockIdx.x) {
#pragma unroll
        for (int j = 0; j < SCAN; ++j) {
          const u64 i = base + (u64)j * kGateThreads + threadIdx.x;
          D[j] = (i < n_in) ? keys[i] : 0ULL;
        }
      }
#pragma unroll
      for (int j = 0; j < SCAN; ++j) {
        const unsigned off = (unsigned)j * kGateThreads + threadIdx.x;
        const bool in = base + off < n_in;
        const bool isT = ((D[j] & op.ann) == op.ann) && ((D[j] & op.cre) == 0);
        const bool isTd = ((D[j] & op.cre) == op.cre) && ((D[j] & op.ann) == 0);
        const bool act = in && (isT || isTd);
        const u64 m = __ballot(act);
        if (m) {
          const int leader = __ffsll((long long)m) - 1;
          unsigned b = 0;
          if (lane == leader) b = atomicAdd(&s_nact, (unsigned)__popcll(m));
          b = __shfl(b, leader);
          if (act) s_act[b + (unsigned)__popcll(m & below)] = (unsigned short)off;
        }
      }
    }
    __syncthreads();
    const unsigned na = s_nact;
    nact += na;
    for (unsigned r0 = 0; r0 < na; r0 += kGateTile) {
      // update: kGateItems listed entries per thread
      u64 idx[kGateItems];
      bool use[kGateItems];
#pragma unroll
      for (int j = 0; j < kGateItems; ++j) {
        const unsigned q = r0 + (unsigned)j * kGateThreads + threadIdx.x;
        use[j] = q < na;
        idx[j] = base + (use[j] ? (u64)s_act[q] : 0ULL);
      }
      GateOut o[kGateItems];
      gate_entries_list<kGateItems>(S, idx, use, op, c, sn, eps, o);
#pragma unroll
      for (int j = 0; j < kGateItems; ++j) {
        dalive += o[j].dalive;
        const u64 m = __ballot(o[j].append);
        if (m) {
          const int leader = __ffsll((long long)m) - 1;
          unsigned b = 0;
          if (lane == leader) b = atomicAdd(&s_cnt, (unsigned)__popcll(m));
          b = __shfl(b, leader);
          if (o[j].append) {
            const unsigned slot = b + (unsigned)__popcll(m & below);
            s_key[slot] = o[j].key;
            s_val[slot] = o[j].val;
          }
        }
      }
      __syncthreads();
      // append: one counter atomic, coalesced writes
      const unsigned cnt = s_cnt;
      if (cnt) {
        if (threadIdx.x == 0) s_base = atomicAdd(&own->app, (u64)cnt);
        __syncthreads();
        const u64 gb = n_in + s_base;
        for (unsigned j = threadIdx.x; j < cnt; j += kGateThreads) {
          const u64 i = gb + j;
          if (i < cap) {
            keys[i] = s_key[j];
            amps[i] = s_val[j];
            hash_insert_new(hash, hmask, s_key[j], i);
          } else {
            atomicOr(&ctr->flags, kFlagOverflow);
          }
        }
        __syncthreads();
        if (threadIdx.x == 0) s_cnt = 0;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) s_nact = 0;
    __syncthreads();
  }
  // the block's change of the alive count
  for (int off = 32; off > 0; off >>= 1) dalive += __shfl_xor(dalive, off);
  if (lane == 0) s_wsum[threadIdx.x / 64] = dalive;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long d = 0;
    for (int w = 0; w < kGateThreads / 64; ++w) d += s_wsum[w];
    if (gate_n_act && nact) atomicAdd((unsigned long long*)gate_n_act, (unsigned long long)nact);
    if (d != 0) atomicAdd((unsigned long long*)&own->dalive, (unsigned long long)d);
  }
}

// Replay of one gate of every segment of a group (blockIdx.y) inside the
// adjoint's recomputation: the same update as k_gate on the segment's working
// copy of the amplitudes, plus one PairRec per active pair, staged per tile in
// LDS and appended to the gate's log behind one atomic per tile.  Every key the
// replay can reach is already stored, so nothing is appended to the state.
// Segments start from their own checkpoints and are independent: one launch per
// step of a segment instead of one per gate (at 40,000 entries a launch of one
// gate is 20 blocks and 5.5 us, nearly all of it latency; 300 of them took
// 1.6 ms, 18 launches over 17 segments 0.2 ms).
__global__ void __launch_bounds__(kGateThreads)
k_gate_replay(const u64* __restrict__ keys, double* __restrict__ work, const HashSlot* __restrict__ hash, u64 hmask,
              u64 n, const GateDesc* __restrict__ gates, double eps, ReplayGroup G, int step,
              unsigned* __restrict__ flags) {
  __shared__ PairRec s_rec[kReplayTile];
  __shared__ unsigned s_cnt;
  __shared__ u64 s_base;
  const int g = G.gate(step, (int)blockIdx.y);
  if (g < 0 || G.star(g)) return;  // uniform: past the end of the segment, or another kernel's
  if (threadIdx.x == 0) s_cnt = 0;
  __syncthreads();
  const GateDesc gd = gates[g];
  PairRec* __restrict__ log = G.pairs(g);
  u64* __restrict__ log_count = G.counts + (g - G.g0);
  const GlobalStore S{(u64*)keys, work + (u64)blockIdx.y * n, (HashSlot*)hash, hmask};
  const int lane = __lane_id();
  const u64 below = (1ULL << lane) - 1ULL;
  const u64 ntiles = (n + kReplayTile - 1) / kReplayTile;
  constexpr int kItems = kReplayTile / kGateThreads;
  for (u64 t = blockIdx.x; t < ntiles; t += gridDim.x) {
    GateOut o[kItems];
    gate_entries_staged<kItems>(S, n, t * (u64)kReplayTile + threadIdx.x, kGateThreads, gd.op, gd.c, gd.s,
                                eps, o);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (o[j].append) atomicOr(flags, kFlagOverflow);
      const u64 m = __ballot(o[j].active);
      if (m) {
        const int leader = __ffsll((long long)m) - 1;
        unsigned b = 0;
        if (lane == leader) b = atomicAdd(&s_cnt, (unsigned)__popcll(m));
        b = __shfl(b, leader);
        if (o[j].active) s_rec[b + (unsigned)__popcll(m & below)] = make_rec(o[j]);
      }
    }
    __syncthreads();
    const unsigned cnt = s_cnt;
    if (cnt) {
      if (threadIdx.x == 0) s_base = atomicAdd(log_count, (u64)cnt);
      __syncthreads();
      const u64 gb = s_base;
      for (unsigned j = threadIdx.x; j < cnt; j += kGateThreads) log[gb + j] = s_rec[j];
      __syncthreads();
      if (threadIdx.x == 0) s_cnt = 0;
      __syncthreads();
    }
  }
}

// Reverse step of one gate over its logged pairs (see adjoint_pair);
// per-block partial sums of dE/dtheta go to partial[blockIdx.x].
__global__ void __launch_bounds__(256)
k_adjoint_rec(const PairRec* __restrict__ log, const u64* __restrict__ log_count,
              double* __restrict__ mu, double c, double sn, double* __restrict__ partial) {
  GlobalMu m{mu};
  const u64 cnt = *log_count;
  double acc = 0.0;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x; r < cnt; r += stride)
    acc += adjoint_pair(log[r], m, c, sn);
  __shared__ double sacc[256];
  sacc[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sacc[threadIdx.x] += sacc[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sacc[0];
}

// Reverse steps of the gates [g_lo, g_hi) of a group, last first, by one
// workgroup: for gates of a few thousand pairs a step is a handful of loads per
// thread, and a barrier orders it before the next one where a launch per gate
// takes 3.2 us (300 gates of 40,000 determinants: 0.95 -> 0.60 ms).  Storage
// positions only grow along a chain, so before a checkpoint of at most kWalkLds
// entries every other one is yet to come, and its mu is 0 (the step back over the
// gate that appended it left that): from there on mu lies in LDS, the barrier
// waits for LDS only, and the records loaded ahead stay in flight (these 300
// gates 600 -> 456 us).  The first record of each thread, the count and the angle
// of the next three gates are loaded ahead.  Each wavefront's share of dE/dtheta_g
// goes to partial[g pstride + wavefront].
constexpr int kWalkThreads = 1024;
constexpr unsigned kWalkLds = 16384;  // 128 KB

struct WalkMu {
  double* p;
  unsigned n;  // entries from here on have mu = 0 (pairs with an entry of a later gate)
  __device__ double get(u64 i) const { return i < n ? p[i] : 0.0; }
  __device__ void set(u64 i, double v) {
    if (i < n) p[i] = v;
  }
};

template <bool LDS, class Mu>
__device__ inline void walk_gates(const ReplayGroup& G, const GateDesc* __restrict__ gates,
                                  const GenGate* __restrict__ gens, int g_lo, int g_hi, Mu& m,
                                  double* __restrict__ partial, u64 pstride) {
  constexpr int kAhead = 3;
  const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
  PairRec rec[kAhead];
  unsigned cnt[kAhead];
  double cs[kAhead], sn[kAhead];
  auto load = [&](int j, int g) {
    cnt[j] = 0;
    if (g < g_lo) return;
    cnt[j] = (unsigned)G.counts[g - G.g0];
    cs[j] = gates[g].c;
    sn[j] = gates[g].s;
    if ((u64)threadIdx.x < G.n) rec[j] = G.pairs(g)[threadIdx.x];  // a log has room for n records
  };
#pragma unroll
  for (int j = 0; j < kAhead; ++j) load(j, g_hi - 1 - j);
  for (int g0 = g_hi - 1; g0 >= g_lo; g0 -= kAhead) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int g = g0 - j;
      if (g < g_lo) break;  // uniform
      double acc = 0.0;
      if (threadIdx.x < cnt[j]) acc += adjoint_pair(rec[j], m, cs[j], sn[j]);
      const PairRec* __restrict__ log = G.pairs(g);
      for (unsigned r = threadIdx.x + kWalkThreads; r < cnt[j]; r += kWalkThreads)
        acc += adjoint_pair(log[r], m, cs[j], sn[j]);
      if (G.star(g)) {  // uniform
        const GenGate gg = gens[g];
        const StarRec* __restrict__ sl = G.stars(g);
        const unsigned ns = (unsigned)G.star_counts[g - G.g0];
        for (unsigned r = threadIdx.x; r < ns; r += kWalkThreads) acc += adjoint_star(sl[r], m, gg);
      }
      load(j, g - kAhead);
      acc = wave_sum63(acc);
      if (lane == 63) partial[(u64)g * pstride + wave] = acc;
      // every mu update of gate g precedes gate g - 1
      if (LDS) lds_barrier();
      else __syncthreads();
    }
  }
}

__global__ void __launch_bounds__(kWalkThreads)
k_adjoint_walk(ReplayGroup G, const GateDesc* __restrict__ gates, const GenGate* __restrict__ gens, int g_lo, int g_hi,
               double* __restrict__ mu, double* __restrict__ partial, u64 pstride, const u64* __restrict__ ckpt_n,
               int nseg) {
  extern __shared__ double s_mu[];  // kWalkLds
  __shared__ int s_seg;
  // last checkpoint of at most kWalkLds entries (the first one has one)
  if (threadIdx.x == 0) s_seg = 0;
  __syncthreads();
  for (int j = threadIdx.x; j < nseg; j += kWalkThreads)
    if (ckpt_n[j] <= kWalkLds) atomicMax(&s_seg, j);
  __syncthreads();
  const bool all = G.n <= kWalkLds;
  const long long cut = all ? (long long)g_hi : (long long)s_seg * G.seg;
  const int g_cut = (int)(cut < g_lo ? g_lo : cut < g_hi ? cut : g_hi);
  GlobalMu gm{mu};
  walk_gates<false>(G, gates, gens, g_cut, g_hi, gm, partial, pstride);
  if (g_cut == g_lo) return;
  const unsigned n = (unsigned)(all ? G.n : ckpt_n[s_seg]);
  __syncthreads();
  for (unsigned i = threadIdx.x; i < n; i += kWalkThreads) s_mu[i] = mu[i];
  __syncthreads();
  WalkMu lm{s_mu, n};
  walk_gates<true>(G, gates, gens, g_lo, g_cut, lm, partial, pstride);
  __syncthreads();
  for (unsigned i = threadIdx.x; i < n; i += kWalkThreads) mu[i] = s_mu[i];
}

__global__ void k_hash_clear(HashSlot* tab, u64 slots) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < slots; i += stride) {
    tab[i].key = kEmptyKey;
    tab[i].idx = 0;
  }
}

__global__ void k_hash_build(const u64* __restrict__ keys, HashSlot* hash, u64 hmask, u64 n) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    hash_insert_new(hash, hmask, keys[i], i);
}

// Presence filter of the alive keys: clear, then set one bit per key.
__global__ void k_filter_clear(unsigned* __restrict__ filt, u64 words) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) filt[i] = 0u;
}

__global__ void k_filter_set(const u64* __restrict__ keys, const double* __restrict__ amps, u64 n,
                             unsigned* __restrict__ filt, u64 fmask) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    if (is_dead(amps[i])) continue;
    const u64 b = filter_bit(keys[i], fmask);
    atomicOr(&filt[b >> 5], 1u << (b & 31));
  }
}

// N_CUT pruning of a state in HBM: a radix select of the ncut-th largest value
// in the N_CUT order (gate_ops.h) in three launches -- two histograms of twelve
// bits of |c| each, in which the next launch finds its digit (select_ops.h), and
// a marking pass that drops everything below the digits found, collects the
// entries that have them, and leaves their order (all of |c|, then the key) to
// its last block.  Where the first digit leaves few entries these are listed
// instead of counted, and every block of the marking pass finds the last one that
// stays by ordering them.  With 8-bit digits, a launch per histogram and one per pick the
// selection was 34 launches a gate: 100 us at 10,000 to 40,000 entries; the three
// take 14 us (evaluation of 100 generators at N_CUT = 10,000: 50.1 -> 6.1 ms in
// all).  blockIdx.y is one of several states of the same keys.  With ctr the
// counts are those after gate `gate` of a chain; otherwise n_host entries are
// scanned.
constexpr int kNcutThreads = 1024;
constexpr int kNcutBits = 12;
constexpr int kNcutBins = 1 << kNcutBits;

__device__ inline u64 ncut_bits(double a) { return (u64)__double_as_longlong(fabs(a)); }
// First digit: six bits of the exponent (2^-63 to 2) and six of the mantissa, so
// that one bin of a spread state holds few entries; smaller and larger values
// share the end bins.  Second: the next twelve bits, or within an end bin the
// whole exponent and one bit of the mantissa.
__device__ inline unsigned ncut_first(u64 hi) {
  const unsigned b = (unsigned)(hi >> 46), lo = (1023u - 63u) << 6;
  if (b < lo) return 0u;
  return b - lo < kNcutBins - 1u ? b - lo : kNcutBins - 1u;
}
__device__ inline unsigned ncut_second(u64 hi, unsigned first) {
  return first == 0u || first == kNcutBins - 1u ? (unsigned)(hi >> 51) : (unsigned)(hi >> 34) & (kNcutBins - 1u);
}

// True in every thread of the block that finishes last of this blockIdx.y.  The
// other blocks' device-scope atomics are then done (each wavefront waits for
// its own before the ticket); nothing else of theirs is read, so no fence is
// needed: a device-scope fence writes the L2 back, and one in every wavefront
// made each of these launches 40 us.
__device__ inline bool ncut_last_block(unsigned* ticket, bool* s_last) {
  device_atomics_done();
  __syncthreads();
  if (threadIdx.x == 0)
    *s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  return *s_last;
}

// Stored and alive entries after gate `gate` of a chain (ctr set), or n_host.
__device__ inline u64 ncut_count(const Counters* ctr, unsigned gate, u64 cap, u64 n_host, u64* alive) {
  u64 n = n_host;
  *alive = n_host;
  if (ctr) live_load(&ctr->live[live_slot(gate)], cap, &n, alive);
  return n;
}

// First digit.  Also clears what the second launch adds to.
__global__ void __launch_bounds__(kNcutThreads)
k_ncut_first(const double* __restrict__ amps, u64 stride_y, u64 n_host, const Counters* __restrict__ ctr,
             unsigned gate, u64 cap, NcutSelect* __restrict__ sel_y, unsigned ncut) {
  __shared__ unsigned h[kNcutBins];
  NcutSelect* sel = sel_y + blockIdx.y;
  const double* __restrict__ a_y = amps + stride_y * blockIdx.y;
  u64 alive;
  const u64 n = ncut_count(ctr, gate, cap, n_host, &alive);
  // nothing to drop: the same in every block (no block changes the counters)
  const bool skip = ctr && ((ctr->flags & kFlagStopped) || alive <= ncut);
  if (blockIdx.x == 0 && threadIdx.x == 0) sel->skip = skip ? 1u : 0u;
  if (skip) return;
  for (int t = threadIdx.x; t < kNcutBins; t += kNcutThreads) h[t] = 0;
  for (int t = blockIdx.x * kNcutThreads + threadIdx.x; t < kNcutBins; t += gridDim.x * kNcutThreads)
    sel->hist[1][t] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) sel->ncand = 0;
  __syncthreads();
  for (u64 i = (u64)blockIdx.x * kNcutThreads + threadIdx.x; i < n; i += (u64)gridDim.x * kNcutThreads) {
    const double a = a_y[i];
    if (!is_dead(a)) atomicAdd(&h[ncut_first(ncut_bits(a))], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kNcutBins; t += kNcutThreads)
    if (h[t]) atomicAdd(&sel->hist[0][t], h[t]);
}

// Finds the first digit; lists its entries where they are few, else counts their
// second digit.
__global__ void __launch_bounds__(kNcutThreads)
k_ncut_second(const double* __restrict__ amps, u64 stride_y, const u64* __restrict__ keys, u64 n_host,
              const Counters* __restrict__ ctr, unsigned gate, u64 cap, NcutSelect* __restrict__ sel_y, unsigned ncut) {
  __shared__ unsigned h[kNcutBins];
  __shared__ unsigned s_wave[kNcutThreads / 64], s_pick[3];
  NcutSelect* sel = sel_y + blockIdx.y;
  if (sel->skip) return;
  unsigned first, rest, held;
  const bool found = hist_find<kNcutBins, kNcutThreads>(sel->hist[0], ncut, s_wave, s_pick, &first, &rest, &held);
  const bool narrow = found && held <= kNcutRank;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sel->none = found ? 0u : 1u;  // fewer than ncut alive: everything stays
    sel->first = first;
    sel->k = rest;
    sel->narrow = narrow ? 1u : 0u;
  }
  if (!found) return;
  u64 alive;
  const u64 n = ncut_count(ctr, gate, cap, n_host, &alive);
  const double* __restrict__ a_y = amps + stride_y * blockIdx.y;
  if (narrow) {
    for (u64 i = (u64)blockIdx.x * kNcutThreads + threadIdx.x; i < n; i += (u64)gridDim.x * kNcutThreads) {
      const double a = a_y[i];
      if (is_dead(a)) continue;
      const u64 hi = ncut_bits(a);
      if (ncut_first(hi) == first) sel->cand[atomicAdd(&sel->ncand, 1u)] = NcutValue{hi, ~keys[i]};
    }
    return;
  }
  for (int t = threadIdx.x; t < kNcutBins; t += kNcutThreads) h[t] = 0;
  __syncthreads();
  for (u64 i = (u64)blockIdx.x * kNcutThreads + threadIdx.x; i < n; i += (u64)gridDim.x * kNcutThreads) {
    const double a = a_y[i];
    if (is_dead(a)) continue;
    const u64 hi = ncut_bits(a);
    if (ncut_first(hi) == first) atomicAdd(&h[ncut_second(hi, first)], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kNcutBins; t += kNcutThreads)
    if (h[t]) atomicAdd(&sel->hist[1][t], h[t]);
}

__device__ inline bool ncut_less(const NcutValue& x, const NcutValue& y) {
  return x.hi < y.hi || (x.hi == y.hi && x.lo < y.lo);
}

__global__ void __launch_bounds__(kNcutThreads)
k_ncut_mark(double* __restrict__ amps, u64 stride_y, const u64* __restrict__ keys, u64 n_host,
            Counters* __restrict__ ctr, unsigned gate, u64 cap, NcutSelect* __restrict__ sel_y,
            unsigned* __restrict__ cand_y, u64 cand_stride) {
  __shared__ NcutValue s_val[kNcutRank];
  __shared__ unsigned s_hist[256], s_pick[3], s_wave[kNcutThreads / 64];
  __shared__ bool s_last;
  __shared__ unsigned s_drop;
  NcutSelect* sel = sel_y + blockIdx.y;
  if (sel->skip) return;
  // for the next selection
  for (int t = blockIdx.x * kNcutThreads + threadIdx.x; t < kNcutBins; t += gridDim.x * kNcutThreads)
    sel->hist[0][t] = 0;
  if (sel->none) return;
  if (threadIdx.x == 0) s_drop = 0;
  double* __restrict__ a_y = amps + stride_y * blockIdx.y;
  unsigned* __restrict__ cand = cand_y + cand_stride * blockIdx.y;
  u64 alive_in;
  const u64 n = ncut_count(ctr, gate, cap, n_host, &alive_in);
  const bool narrow = sel->narrow != 0;
  unsigned prefix = sel->first, k = sel->k;  // digits found; candidates that stay
  NcutValue cut{0, 0};  // few candidates: the k-th of them, found by every block
  if (narrow) {
    __shared__ NcutValue s_cut;
    const unsigned nc = sel->ncand;
    NcutValue v{0, 0};
    if (threadIdx.x < nc) s_val[threadIdx.x] = v = sel->cand[threadIdx.x];
    __syncthreads();
    if (threadIdx.x < nc) {
      unsigned rank = 0;
      for (unsigned j = 0; j < nc; ++j) rank += ncut_less(v, s_val[j]) ? 1u : 0u;
      if (rank == k - 1) s_cut = v;  // one thread: the values differ in their keys
    }
    __syncthreads();
    cut = s_cut;
  } else {
    unsigned second, rest, held;
    (void)hist_find<kNcutBins, kNcutThreads>(sel->hist[1], k, s_wave, s_pick, &second, &rest, &held);
    prefix = prefix << kNcutBits | second;
    k = rest;
    __syncthreads();
  }
  const int lane = (int)(threadIdx.x & 63u);
  unsigned dropped = 0;
  const u64 step = (u64)gridDim.x * kNcutThreads;
  for (u64 base = (u64)blockIdx.x * kNcutThreads; base < n; base += step) {  // same trips in the whole block
    const u64 i = base + threadIdx.x;
    const double a = i < n ? a_y[i] : dead_value();
    const bool alive = !is_dead(a);
    unsigned p = 0;
    bool below = false;
    if (alive) {
      const u64 hi = ncut_bits(a);
      p = ncut_first(hi);
      if (narrow) {
        below = p < prefix || (p == prefix && ncut_less(NcutValue{hi, ~keys[i]}, cut));
      } else {
        p = p << kNcutBits | ncut_second(hi, p);
        below = p < prefix;
      }
    }
    if (below) {
      a_y[i] = dead_value();
      ++dropped;
    }
    if (narrow) continue;  // uniform
    const bool tie = alive && p == prefix;
    const u64 m = __ballot(tie);
    if (m) {
      unsigned b = 0;
      if (lane == 0) b = atomicAdd(&sel->ncand, (unsigned)__popcll(m));
      b = (unsigned)__shfl((int)b, 0);
      if (tie)  // read by the last block
        __hip_atomic_store(&cand[b + (unsigned)__popcll(m & ((1ULL << lane) - 1ULL))], (unsigned)i, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  auto count_drops = [&]() {  // one add of the block
    if (!ctr) return;
    unsigned d = (unsigned)dropped;
    for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off);
    if (lane == 0 && d) atomicAdd(&s_drop, d);
    __syncthreads();
    if (threadIdx.x == 0 && s_drop) {
      atomicAdd((unsigned long long*)&ctr->live[live_slot(gate)].dalive, (unsigned long long)(0ULL - (u64)s_drop));
      s_drop = 0;
    }
    __syncthreads();
  };
  count_drops();
  if (narrow) return;
  if (!ncut_last_block(&sel->ticket, &s_last)) return;
  dropped = 0;
  const unsigned nc = __hip_atomic_load(&sel->ncand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  auto value = [&](unsigned c, u64* at) {
    const u64 i = __hip_atomic_load(&cand[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *at = i;
    return NcutValue{ncut_bits(a_y[i]), ~keys[i]};
  };
  if (k < nc && nc <= kNcutRank) {
    u64 at = 0;
    NcutValue v{0, 0};
    if (threadIdx.x < nc) {
      v = value(threadIdx.x, &at);
      s_val[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x < nc) {
      unsigned rank = 0;
      for (unsigned j = 0; j < nc; ++j) rank += ncut_less(v, s_val[j]) ? 1u : 0u;
      if (rank >= k) {
        a_y[at] = dead_value();
        ++dropped;
      }
    }
  } else if (k < nc) {
    // many entries share both digits (equal amplitudes): radix select over the
    // candidates, eight bits at a time from |c| to the key
    NcutValue want{0, 0}, mask{0, 0};
    for (int d = 0; d < 16; ++d) {
      const int sh = 56 - 8 * (d & 7);
      for (int t = threadIdx.x; t < 256; t += kNcutThreads) s_hist[t] = 0;
      __syncthreads();
      for (unsigned c = threadIdx.x; c < nc; c += kNcutThreads) {
        u64 at;
        const NcutValue v = value(c, &at);
        if ((v.hi & mask.hi) != want.hi || (v.lo & mask.lo) != want.lo) continue;
        atomicAdd(&s_hist[((d < 8 ? v.hi : v.lo) >> sh) & 255u], 1u);
      }
      __syncthreads();
      if (threadIdx.x < 64) {  // four bins a lane, from the largest
        unsigned h[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          h[j] = s_hist[255 - (4 * lane + j)];
          sum += h[j];
        }
        unsigned inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
          const unsigned v = __shfl_up(inc, off);
          if (lane >= off) inc += v;
        }
        unsigned before = inc - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (before < k && before + h[j] >= k) {
            s_pick[0] = (unsigned)(255 - (4 * lane + j));
            s_pick[1] = k - before;
          }
          before += h[j];
        }
      }
      __syncthreads();
      const u64 digit = s_pick[0];
      k = s_pick[1];
      if (d < 8) {
        want.hi |= digit << sh;
        mask.hi |= 255ULL << sh;
      } else {
        want.lo |= digit << sh;
        mask.lo |= 255ULL << sh;
      }
      __syncthreads();
    }
    // want is the last value that stays
    for (unsigned c = threadIdx.x; c < nc; c += kNcutThreads) {
      u64 at;
      const NcutValue v = value(c, &at);
      if (ncut_less(v, want)) {
        a_y[at] = dead_value();
        ++dropped;
      }
    }
  }
  count_drops();
  if (threadIdx.x == 0) {
    sel->ticket = 0;
  }
}

// State = the single reference determinant with amplitude 1.
__global__ void k_reset_reference(u64* __restrict__ keys, double* __restrict__ amps,
                                  Counters* __restrict__ ctr, u64 ref) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    keys[0] = ref;
    amps[0] = 1.0;
    ctr->n = 1;
    ctr->alive = 1;
    ctr->flags = 0;
    ctr->stop_gate = 0;
  }
}

__global__ void k_live_begin(Counters* __restrict__ ctr, unsigned g) {
  if (threadIdx.x != 0) return;
  for (int j = 0; j < 3; ++j) ctr->live[j] = LiveCounts{0, 0, 0, 0};
  ctr->live[live_before(g)].n = ctr->n;
  ctr->live[live_before(g)].alive = ctr->alive;
}

__global__ void k_live_end(Counters* __restrict__ ctr, u64 cap, unsigned M) {
  if (threadIdx.x != 0) return;
  const unsigned g = (ctr->flags & kFlagStopped) ? (unsigned)ctr->stop_gate : M;
  live_load(&ctr->live[live_before(g)], cap, &ctr->n, &ctr->alive);
}

// Same, with the entry count read from the device counters.
__global__ void k_hash_build_dev(const u64* __restrict__ keys, HashSlot* hash, u64 hmask,
                                 const Counters* __restrict__ ctr) {
  const u64 n = __hip_atomic_load(&ctr->n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    hash_insert_new(hash, hmask, keys[i], i);
}

__global__ void k_mark_dead_range(double* amps, u64 lo, u64 hi) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = lo + (u64)blockIdx.x * blockDim.x + threadIdx.x; i < hi; i += stride)
    amps[i] = dead_value();
}

// Drop every alive entry with |c| < eps (used once after the first gate of a
// chain that starts from a caller-supplied state, whose untouched entries
// have not been tested against eps yet).  Skipped if the chain has stopped.
__global__ void __launch_bounds__(256)
k_prune_all(double* __restrict__ amps, Counters* __restrict__ ctr, unsigned gate, u64 cap, double eps) {
  if (__hip_atomic_load(&ctr->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFlagStopped)
    return;
  u64 n, alive;
  live_load(&ctr->live[live_slot(gate)], cap, &n, &alive);
  unsigned long long dropped = 0;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double a = amps[i];
    if (!is_dead(a) && fabs(a) < eps) {
      amps[i] = dead_value();
      ++dropped;
    }
  }
  const u64 m = __ballot(dropped != 0);
  if (m) {
    // wave sum of dropped, then one atomic per wave
    unsigned long long s = dropped;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (__lane_id() == 0)
      atomicAdd((unsigned long long*)&ctr->live[live_slot(gate)].dalive, (unsigned long long)(0ULL - s));
  }
}

// Copy amps[0, n) of the state before a gate to dst and record n, unless the chain
// has stopped (the host re-enqueues the copy when it resumes).
__global__ void k_ckpt_save(const double* __restrict__ amps, const Counters* __restrict__ ctr, unsigned gate,
                            u64 cap, double* __restrict__ dst, u64* __restrict__ dst_n) {
  if (__hip_atomic_load(&ctr->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFlagStopped)
    return;
  u64 n, alive;
  live_load(&ctr->live[live_before(gate)], cap, &n, &alive);
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = amps[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) *dst_n = n;
}

// Working copies of a group of segments: work[y n, y n + n) = the checkpoint of
// segment seg0 + y, dead beyond its entries.
__global__ void k_restore(double* __restrict__ work, const double* const* __restrict__ ckpt,
                          const u64* __restrict__ ckpt_n, int seg0, u64 n) {
  const int j = seg0 + (int)blockIdx.y;
  const u64 n_src = ckpt_n[j];
  const double* __restrict__ src = ckpt[j];
  double* __restrict__ dst = work + (u64)blockIdx.y * n;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    dst[i] = (i < n_src) ? src[i] : dead_value();
}

static int grid_for(u64 n, int block, int max_grid) {
  u64 g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > (u64)max_grid) g = max_grid;
  return (int)g;
}

hipError_t launch_hash_clear(HashSlot* tab, u64 slots, hipStream_t stream) {
  hipLaunchKernelGGL(k_hash_clear, dim3(grid_for(slots, 256, 8192)), dim3(256), 0, stream, tab, slots);
  return hipGetLastError();
}

hipError_t launch_hash_build(const DeviceState& st, u64 n, hipStream_t stream) {
  hipLaunchKernelGGL(k_hash_build, dim3(grid_for(n, 256, 8192)), dim3(256), 0, stream, st.keys,
                     st.hash, st.hmask, n);
  return hipGetLastError();
}

hipError_t launch_filter_build(const DeviceState& st, u64 n, int grid, hipStream_t stream) {
  const u64 words = (st.fmask + 1) / 32;
  hipLaunchKernelGGL(k_filter_clear, dim3(grid_for(words, 256, 4096)), dim3(256), 0, stream, st.filt,
                     words);
  if (n > 0)
    hipLaunchKernelGGL(k_filter_set, dim3(grid), dim3(256), 0, stream, st.keys, st.amps, n, st.filt,
                       st.fmask);
  return hipGetLastError();
}

size_t ncut_select_bytes() { return sizeof(NcutSelect); }

hipError_t launch_ncut(double* amps, u64 stride, const u64* keys, u64 n_host, Counters* ctr, unsigned gate, u64 cap, void* select,
                       unsigned* cand, u64 cand_stride, unsigned ncut, u64 n_most, int states, hipStream_t stream) {
  // one block per compute unit at most: every block adds its nonzero bins to
  // the same few addresses
  const dim3 grid((unsigned)grid_for(n_most, kNcutThreads, 256), (unsigned)states);
  NcutSelect* sel = (NcutSelect*)select;
  hipLaunchKernelGGL(k_ncut_first, grid, dim3(kNcutThreads), 0, stream, amps, stride, n_host, ctr, gate, cap, sel, ncut);
  hipLaunchKernelGGL(k_ncut_second, grid, dim3(kNcutThreads), 0, stream, amps, stride, keys, n_host, ctr, gate, cap, sel, ncut);
  hipLaunchKernelGGL(k_ncut_mark, grid, dim3(kNcutThreads), 0, stream, amps, stride, keys, n_host, ctr, gate, cap, sel, cand,
                     cand_stride);
  return hipGetLastError();
}

hipError_t launch_reset_reference(const DeviceState& st, u64 ref, hipStream_t stream) {
  hipLaunchKernelGGL(k_reset_reference, dim3(1), dim3(64), 0, stream, st.keys, st.amps, st.ctr, ref);
  return hipGetLastError();
}

hipError_t launch_hash_build_dev(const DeviceState& st, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_hash_build_dev, dim3(grid), dim3(256), 0, stream, st.keys, st.hash, st.hmask,
                     st.ctr);
  return hipGetLastError();
}

hipError_t launch_gate(const DeviceState& st, const OpDesc& op, double c, double sn, double eps,
                       u64* gate_n_in, unsigned gate_index, u64 max_keys, int grid,
                       hipStream_t stream, u64* gate_n_act) {
  if (st.cap >= kGateWideCap)
    hipLaunchKernelGGL(k_gate<kGateScanWide>, dim3(grid), dim3(kGateThreads), 0, stream, st.keys, st.amps,
                       st.hash, st.hmask, st.cap, st.ctr, op, c, sn, eps, gate_n_in, gate_index,
                       max_keys, gate_n_act);
  else
    hipLaunchKernelGGL(k_gate<kGateScanNarrow>, dim3(grid), dim3(kGateThreads), 0, stream, st.keys, st.amps,
                       st.hash, st.hmask, st.cap, st.ctr, op, c, sn, eps, gate_n_in, gate_index,
                       max_keys, gate_n_act);
  return hipGetLastError();
}

hipError_t launch_prune_all(const DeviceState& st, double eps, unsigned gate, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_prune_all, dim3(grid), dim3(256), 0, stream, st.amps, st.ctr, gate, st.cap, eps);
  return hipGetLastError();
}

hipError_t launch_gate_replay(const DeviceState& st, double* work, u64 n, const GateDesc* gates, double eps,
                             const ReplayGroup& G, int step, int segs, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_gate_replay, dim3(grid, segs), dim3(kGateThreads), 0, stream, st.keys, work, st.hash,
                     st.hmask, n, gates, eps, G, step, &st.ctr->flags);
  return hipGetLastError();
}

hipError_t launch_adjoint_walk(const ReplayGroup& G, const GateDesc* gates, const GenGate* gens, int g_lo, int g_hi,
                               double* mu, double* partial, u64 pstride, const u64* ckpt_n, int nseg,
                               hipStream_t stream) {
  if (g_hi <= g_lo) return hipSuccess;
  if (pstride < (u64)kWalkThreads / 64) return hipErrorInvalidValue;
  const size_t bytes = kWalkLds * sizeof(double);
  hipError_t e = hipFuncSetAttribute((const void*)k_adjoint_walk, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_adjoint_walk, dim3(1), dim3(kWalkThreads), bytes, stream, G, gates, gens, g_lo, g_hi, mu, partial,
                     pstride, ckpt_n, nseg);
  return hipGetLastError();
}

hipError_t launch_adjoint_rec(const PairRec* log, const u64* log_count, double* mu, double c,
                              double sn, double* partial, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_adjoint_rec, dim3(grid), dim3(256), 0, stream, log, log_count, mu, c, sn,
                     partial);
  return hipGetLastError();
}

hipError_t launch_live_begin(const DeviceState& st, unsigned g, hipStream_t stream) {
  hipLaunchKernelGGL(k_live_begin, dim3(1), dim3(64), 0, stream, st.ctr, g);
  return hipGetLastError();
}

hipError_t launch_live_end(const DeviceState& st, unsigned M, hipStream_t stream) {
  hipLaunchKernelGGL(k_live_end, dim3(1), dim3(64), 0, stream, st.ctr, st.cap, M);
  return hipGetLastError();
}

hipError_t launch_ckpt_save(const DeviceState& st, unsigned gate, double* dst, u64* dst_n, int grid,
                            hipStream_t stream) {
  hipLaunchKernelGGL(k_ckpt_save, dim3(grid), dim3(256), 0, stream, st.amps, st.ctr, gate, st.cap, dst, dst_n);
  return hipGetLastError();
}

hipError_t launch_restore(double* work, const double* const* ckpt, const u64* ckpt_n, int seg0, int segs, u64 n,
                          hipStream_t stream) {
  hipLaunchKernelGGL(k_restore, dim3(grid_for(n, 256, 2048), segs), dim3(256), 0, stream, work, ckpt, ckpt_n, seg0, n);
  return hipGetLastError();
}

hipError_t launch_mark_dead_range(double* amps, u64 lo, u64 hi, hipStream_t stream) {
  if (hi <= lo) return hipSuccess;
  hipLaunchKernelGGL(k_mark_dead_range, dim3(grid_for(hi - lo, 256, 8192)), dim3(256), 0, stream,
                     amps, lo, hi);
  return hipGetLastError();
}

}  // namespace swcs

namespace swcs {

// Buffer clears and small host-to-device writes as kernels on the stream
// (fills instead of runtime memsets, counters passed as kernel arguments), so
// every step of a call is one of the library's own launches, in stream order,
// and a caller may capture it.
__global__ void k_fill_u32(unsigned* __restrict__ p, unsigned v, u64 words) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) p[i] = v;
}

__global__ void k_pack_result(double* __restrict__ to, const double* __restrict__ sums, const Counters* __restrict__ ctr) {
  if (threadIdx.x < 2) to[threadIdx.x] = sums[threadIdx.x];
  if (threadIdx.x == 2) to[2] = (double)ctr->flags;
}

__global__ void k_store_counters(Counters* __restrict__ ctr, Counters v) { *ctr = v; }

__global__ void k_clear_flag(Counters* __restrict__ ctr, unsigned bit) {
  atomicAnd(&ctr->flags, ~bit);
}

hipError_t launch_fill_u32(void* p, unsigned v, u64 words, hipStream_t stream) {
  if (words == 0) return hipSuccess;
  const u64 blocks = std::min<u64>((words + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, stream, (unsigned*)p, v, words);
  return hipGetLastError();
}

hipError_t launch_pack_result(double* to, const double* sums, const Counters* ctr, hipStream_t stream) {
  hipLaunchKernelGGL(k_pack_result, dim3(1), dim3(64), 0, stream, to, sums, ctr);
  return hipGetLastError();
}

hipError_t launch_store_counters(Counters* ctr, const Counters& v, hipStream_t stream) {
  hipLaunchKernelGGL(k_store_counters, dim3(1), dim3(1), 0, stream, ctr, v);
  return hipGetLastError();
}

hipError_t launch_clear_flag(Counters* ctr, unsigned bit, hipStream_t stream) {
  hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, stream, ctr, bit);
  return hipGetLastError();
}

}  // namespace swcs
