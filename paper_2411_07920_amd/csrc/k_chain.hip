// Single-workgroup kernels that keep a small state in LDS and run a whole
// gate chain (or the whole adjoint sweep) in one launch.  A state of up to
// kLdsCap determinants (16 B of keys and amplitudes plus 8 B of hash index
// each) fits the 160 KB LDS of one CU; the gates then cost LDS latency
// instead of one kernel launch each.  The per-entry arithmetic is shared
// with the HBM kernels (gate_ops.h, gen_ops.h), so results are identical bit for
// bit.  Chains with overlapping generators have instances of their own (their
// gate needs more registers): 21 generators of 8 orbitals, 750 determinants, with
// gradients 841 us gate by gate in HBM, 357 here.
#include "gen_ops.h"

namespace swcs {

constexpr int kChainThreads = 1024;
constexpr int kGateChunk = 256;  // gate descriptors staged in LDS at a time

constexpr int kLdsNcutBins = kChainThreads;  // one a thread
constexpr unsigned kLdsNcutRank = 256;       // candidates ordered by counting

struct NcutState {
  unsigned hist[kLdsNcutBins];
  unsigned wsum[kChainThreads / 64];
  u64 hi[kLdsNcutRank], lo[kLdsNcutRank];
  unsigned pick, rest, held;  // digit found, rank within it, its count
  unsigned ncand, drop, aux;
};

// Keep only the ncut alive entries of amps[0, n), n <= 4 kChainThreads, that
// come first in the N_CUT order (gate_ops.h); the rest are marked dead.  Called by
// all threads of the block; returns the number of entries dropped (valid in every
// thread).  One histogram of ten bits of |c| -- six of the exponent (2^-63 to 2),
// four of the mantissa, the end bins take the rest -- and the entries of the bin
// that holds the cut are ordered by counting: six barriers.  Only where more than
// 256 share the bin, a radix select over them, eight bits of |c| and then of the
// key at a time.  (Sixteen such digits over the state, each picked by one thread,
// took most of a gate's time: 20 generators of 9 orbitals at N_CUT = 408 with
// gradients 1,937 us, now 412.)
__device__ inline unsigned lds_ncut(double* amps, const u64* keys, unsigned n, unsigned ncut,
                                    NcutState& st) {
  constexpr int kPer = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  st.hist[tid] = 0;
  if (tid == 0) {
    st.pick = 0xffffffffu;
    st.ncand = st.drop = 0;
  }
  lds_barrier();
  u64 hi[kPer];
  unsigned dig[kPer];  // 1 + digit, 0: no alive entry
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const unsigned i = (unsigned)tid + (unsigned)j * kChainThreads;
    const double a = i < n ? amps[i] : dead_value();
    dig[j] = 0;
    if (is_dead(a)) continue;
    hi[j] = (u64)__double_as_longlong(fabs(a));
    const unsigned b = (unsigned)(hi[j] >> 48), low = (1023u - 63u) << 4;
    const unsigned d = b < low ? 0u : (b - low < kLdsNcutBins - 1u ? b - low : kLdsNcutBins - 1u);
    dig[j] = 1u + d;
    atomicAdd(&st.hist[d], 1u);
  }
  lds_barrier();
  {
    const unsigned bin = (unsigned)(kLdsNcutBins - 1 - tid), h = st.hist[bin];
    unsigned inc = h;
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned v = __shfl_up(inc, off);
      if (lane >= off) inc += v;
    }
    if (lane == 63) st.wsum[wave] = inc;
    lds_barrier();
    unsigned before = inc - h;
    for (int w = 0; w < wave; ++w) before += st.wsum[w];
    if (before < ncut && before + h >= ncut) {
      st.pick = bin;
      st.rest = ncut - before;
      st.held = h;
    }
  }
  lds_barrier();
  if (st.pick == 0xffffffffu) return 0;  // fewer alive
  const unsigned cut = 1u + st.pick, held = st.held;
  unsigned k = st.rest, dropped = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const unsigned i = (unsigned)tid + (unsigned)j * kChainThreads;
    if (dig[j] != 0 && dig[j] < cut) {
      amps[i] = dead_value();
      ++dropped;
    } else if (dig[j] == cut && held <= kLdsNcutRank) {
      const unsigned at = atomicAdd(&st.ncand, 1u);
      st.hi[at] = hi[j];
      st.lo[at] = ~keys[i];
    }
  }
  if (k < held && held <= kLdsNcutRank) {
    lds_barrier();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (dig[j] != cut) continue;
      const unsigned i = (unsigned)tid + (unsigned)j * kChainThreads;
      const u64 lo = ~keys[i];
      unsigned rank = 0;
      for (unsigned q = 0; q < held; ++q)
        rank += (hi[j] < st.hi[q] || (hi[j] == st.hi[q] && lo < st.lo[q])) ? 1u : 0u;
      if (rank >= k) {
        amps[i] = dead_value();
        ++dropped;
      }
    }
  } else if (k < held) {
    u64 phi = 0, plo = 0, mhi = 0, mlo = 0;  // prefix found and its mask, in every thread
    for (int d = 0; d < 16; ++d) {
      const int sh = 56 - 8 * (d & 7);
      lds_barrier();  // the digit before has been read
      if (tid < 256) st.hist[tid] = 0;
      lds_barrier();
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (dig[j] != cut) continue;
        const u64 lo = ~keys[(unsigned)tid + (unsigned)j * kChainThreads];
        if ((hi[j] & mhi) == phi && (lo & mlo) == plo) atomicAdd(&st.hist[((d < 8 ? hi[j] : lo) >> sh) & 255u], 1u);
      }
      lds_barrier();
      if (tid < 64) {  // four bins a lane, from the largest
        unsigned h[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          h[q] = st.hist[255 - (4 * lane + q)];
          sum += h[q];
        }
        unsigned inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
          const unsigned v = __shfl_up(inc, off);
          if (lane >= off) inc += v;
        }
        unsigned before = inc - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (before < k && before + h[q] >= k) {
            st.pick = (unsigned)(255 - (4 * lane + q));
            st.rest = k - before;
          }
          before += h[q];
        }
      }
      lds_barrier();
      const u64 v = (u64)st.pick << sh, m = 255ULL << sh;
      k = st.rest;
      if (d < 8) {
        phi |= v;
        mhi |= m;
      } else {
        plo |= v;
        mlo |= m;
      }
    }
    // (phi, plo) is the last value that stays
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (dig[j] != cut) continue;
      const unsigned i = (unsigned)tid + (unsigned)j * kChainThreads;
      if (hi[j] < phi || (hi[j] == phi && ~keys[i] < plo)) {
        amps[i] = dead_value();
        ++dropped;
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) dropped += __shfl_xor(dropped, off);
  if (lane == 0 && dropped) atomicAdd(&st.drop, dropped);
  lds_barrier();
  return st.drop;
}
static_assert(kLdsCap <= 4 * kChainThreads, "lds_ncut holds four entries a thread");

// Forward chain of gates [g0, M) on the state held in keys / amps (HBM),
// moved into LDS for the duration.  Checkpoints (amplitudes before gate g
// for g % seg == 0) and the per-gate input sizes are written to HBM.  If a
// gate might not fit, the kernel stops before it: the state is written back
// and ctr->stop_gate / kFlagStopped tell the host where to continue.  STAR:
// gates with kinds[g] set are overlapping generators gens[g].  gate_n_act (may
// be NULL) receives the entries that each gate's operator acts on, as the
// multi-block kernels count them.
template <int CAP, bool STAR>
__global__ void __launch_bounds__(kChainThreads)
k_chain_lds(u64* __restrict__ keys, double* __restrict__ amps, Counters* __restrict__ ctr,
            const GateDesc* __restrict__ gates, const int* __restrict__ kinds, const GenGate* __restrict__ gens,
            int g0, int M, double eps, int prune_first, double* const* __restrict__ ckpt, u64* __restrict__ ckpt_n, int seg,
            u64* __restrict__ gate_n_in, u64* __restrict__ gate_n_act, u64 max_keys, unsigned ncut) {
  __shared__ NcutState nst;
  __shared__ u64 skeys[CAP];
  __shared__ double samps[CAP];
  __shared__ int sslots[2 * CAP];
  // Per-gate append, activity and alive-change counters, three in rotation: gate
  // g uses slot g % 3; after the gate's barrier every thread reads it, and
  // thread 0 clears slot (g + 2) % 3, last read before the previous barrier
  // and next used after the following one.
  __shared__ unsigned s_app[3], s_act[3];
  __shared__ int s_dal[3];
  __shared__ unsigned s_n0, s_alive0;
  __shared__ GateDesc sg[kGateChunk];
  __shared__ int sk[STAR ? kGateChunk : 1];
  const int tid = threadIdx.x;
  if (tid == 0) {
    s_n0 = (unsigned)ctr->n;
    s_alive0 = (unsigned)ctr->alive;
  }
  if (tid < 3) {
    s_app[tid] = 0;
    s_act[tid] = 0;
    s_dal[tid] = 0;
  }
  for (int t = tid; t < 2 * CAP; t += kChainThreads) sslots[t] = 0;
  lds_barrier();
  unsigned n = s_n0, alive = s_alive0;  // block-uniform, kept in every thread
  if (n > (unsigned)CAP) {
    if (tid == 0) {
      ctr->stop_gate = (u64)g0;
      atomicOr(&ctr->flags, kFlagStopped);
    }
    return;
  }
  for (unsigned i = tid; i < n; i += kChainThreads) {
    skeys[i] = keys[i];
    samps[i] = amps[i];
  }
  lds_barrier();
  LdsStore S{skeys, samps, sslots, 2u * CAP - 1u};
  for (unsigned i = tid; i < n; i += kChainThreads) S.insert(skeys[i], (int)i);
  int stop = -1;
  for (int g = g0; g < M; ++g) {
    // Every earlier read of sg and every write of the previous gate happened
    // before the previous gate's barrier (or the index build's).
    if ((g - g0) % kGateChunk == 0) {
      for (int t = tid; t < kGateChunk && g + t < M; t += kChainThreads) {
        sg[t] = gates[g + t];
        if (STAR) sk[t] = kinds[g + t];
      }
      lds_barrier();
    }
    const bool star = STAR && sk[(g - g0) % kGateChunk] != 0;  // uniform
    if (ckpt && g % seg == 0) {
      double* dst = ckpt[g / seg];
      for (unsigned i = tid; i < n; i += kChainThreads) dst[i] = samps[i];
      if (tid == 0) ckpt_n[g / seg] = n;
      lds_barrier();  // the copy precedes the gate's updates
    }
    const u64 room = max_keys > n ? max_keys - n : 0;
    const u64 most = star ? 2 * (u64)alive : (u64)alive;
    if ((u64)n + (most < room ? most : room) > (u64)CAP) {
      stop = g;
      break;  // uniform: every thread holds the same n and alive
    }
    const int slot = g % 3;
    int dal = 0;
    unsigned act = 0;
    auto append = [&](u64 key, double val) {
      const unsigned idx = n + atomicAdd(&s_app[slot], 1u);
      skeys[idx] = key;
      samps[idx] = val;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");  // before the slot that shows it
      S.insert(key, (int)idx);
    };
    if (star) {
      const GenGate gg = gens[g];
      for (unsigned i = tid; i < n; i += kChainThreads) {
        const GenOut o = gen_entry(S, i, gg, eps);
        dal += (int)o.dalive;
        act += (op_acts(gg.op1, skeys[i]) || op_acts(gg.op2, skeys[i])) ? 1u : 0u;
        if (o.napp > 0) append(o.key[0], o.val[0]);
        if (o.napp > 1) append(o.key[1], o.val[1]);
      }
    } else {
      const GateDesc gd = sg[(g - g0) % kGateChunk];
      for (unsigned i = tid; i < n; i += kChainThreads) {
        const GateOut o = gate_entry(S, i, gd.op, gd.c, gd.s, eps);
        dal += (int)o.dalive;
        act += o.acts ? 1u : 0u;
        if (o.append) append(o.key, o.val);
      }
    }
    if (dal) atomicAdd(&s_dal[slot], dal);
    if (gate_n_act && act) atomicAdd(&s_act[slot], act);
    lds_barrier();
    if (tid == 0) {
      if (gate_n_in) gate_n_in[g] = alive;
      if (gate_n_act) gate_n_act[g] = s_act[slot];
      s_app[(g + 2) % 3] = 0;
      s_act[(g + 2) % 3] = 0;
      s_dal[(g + 2) % 3] = 0;
    }
    n += s_app[slot];
    alive = (unsigned)((int)alive + s_dal[slot]);
    if (ncut && alive > ncut) alive -= lds_ncut(samps, skeys, n, ncut, nst);
    if (g == 0 && prune_first) {
      // Entries of a caller-supplied starting state that the first gate did
      // not touch have not been tested against eps yet.
      if (tid == 0) nst.aux = 0;
      lds_barrier();
      unsigned dropped = 0;
      for (unsigned i = tid; i < n; i += kChainThreads) {
        const double a = samps[i];
        if (!is_dead(a) && fabs(a) < eps) {
          samps[i] = dead_value();
          ++dropped;
        }
      }
      if (dropped) atomicAdd(&nst.aux, dropped);
      lds_barrier();
      alive -= nst.aux;
    }
  }
  lds_barrier();
  for (unsigned i = tid; i < n; i += kChainThreads) {
    keys[i] = skeys[i];
    amps[i] = samps[i];
  }
  if (tid == 0) {
    ctr->n = n;
    ctr->alive = alive;
    if (stop >= 0) {
      ctr->stop_gate = (u64)stop;
      atomicOr(&ctr->flags, kFlagStopped);
    }
  }
}

// Frozen-support adjoint sweep for a final state of n <= CAP stored
// determinants, in two launches.  (1) One workgroup per checkpoint segment
// restores the segment's checkpoint into LDS and replays its gates, logging
// one PairRec per active pair of gate g in logbuf[g * n ...] and the count in
// logcnt[g]; segments are independent, so they run side by side.  (2) One
// workgroup walks all gates backwards with the adjoint vector mu in LDS:
// one barrier per gate orders the mu updates, each wavefront's share of
// dE/dtheta_g goes to dE_part[g * 16 + wave], and the 16 shares are added in
// wave order at the end.
constexpr int kMaxSeg = 256;  // gate descriptors a segment stages in LDS at a time
constexpr int kWaves = kChainThreads / 64;

template <int CAP, bool STAR>
__global__ void __launch_bounds__(kChainThreads)
k_adjoint_replay_lds(const u64* __restrict__ keys, unsigned n, const GateDesc* __restrict__ gates,
                     const int* __restrict__ kinds, const GenGate* __restrict__ gens,
                     int M, int seg, double eps, const double* const* __restrict__ ckpt,
                     const u64* __restrict__ ckpt_n, char* __restrict__ logbuf, size_t log_bytes,
                     unsigned* __restrict__ logcnt, unsigned* __restrict__ flags, unsigned ncut) {
  __shared__ NcutState nst;
  __shared__ u64 skeys[CAP];
  __shared__ double sW[CAP];
  __shared__ int sslots[2 * CAP];
  __shared__ GateDesc sg[kMaxSeg];
  __shared__ int sk[STAR ? kMaxSeg : 1];
  __shared__ unsigned s_cnt, s_star;
  const int tid = threadIdx.x;
  const int j = blockIdx.x;
  const int g_lo = j * seg;
  const int g_hi = (g_lo + seg < M) ? g_lo + seg : M;
  const unsigned nj = (unsigned)ckpt_n[j];
  const double* src = ckpt[j];
  for (int t = tid; t < 2 * CAP; t += kChainThreads) sslots[t] = 0;
  for (unsigned i = tid; i < n; i += kChainThreads) {
    skeys[i] = keys[i];
    sW[i] = (i < nj) ? src[i] : dead_value();
  }
  if (tid == 0) s_cnt = s_star = 0;
  lds_barrier();
  LdsStore L{skeys, sW, sslots, 2u * CAP - 1u};
  for (unsigned i = tid; i < n; i += kChainThreads) L.insert(skeys[i], (int)i);
  const int lane = tid & 63;
  const u64 below = (1ULL << lane) - 1ULL;
  for (int g = g_lo; g < g_hi; ++g) {
    if ((g - g_lo) % kMaxSeg == 0) {
      lds_barrier();
      for (int t = tid; t < kMaxSeg && g + t < g_hi; t += kChainThreads) {
        sg[t] = gates[g + t];
        if (STAR) sk[t] = kinds[g + t];
      }
    }
    lds_barrier();
    const GateDesc gd = sg[(g - g_lo) % kMaxSeg];
    PairRec* lg = (PairRec*)(logbuf + (size_t)g * log_bytes);
    if (STAR && sk[(g - g_lo) % kMaxSeg]) {  // uniform
      const GenGate gg = gens[g];
      StarRec* ls = (StarRec*)(lg + n);
      for (unsigned i0 = 0; i0 < n; i0 += kChainThreads) {
        const unsigned i = i0 + tid;
        GenOut o;
        o.napp = 0;
        o.kind = 0;
        if (i < n) o = gen_entry(L, i, gg, eps);
        if (o.napp) atomicOr(flags, kFlagOverflow);  // cannot happen: all keys are stored
        const u64 mp = __ballot(o.kind == 1), ms = __ballot(o.kind == 2);
        unsigned bp = 0, bs = 0;
        if (lane == 0 && mp) bp = atomicAdd(&s_cnt, (unsigned)__popcll(mp));
        if (lane == 0 && ms) bs = atomicAdd(&s_star, (unsigned)__popcll(ms));
        bp = __shfl(bp, 0);
        bs = __shfl(bs, 0);
        if (o.kind == 1) lg[bp + (unsigned)__popcll(mp & below)] = o.pr;
        if (o.kind == 2) ls[bs + (unsigned)__popcll(ms & below)] = o.sr;
      }
    } else
    for (unsigned i0 = 0; i0 < n; i0 += kChainThreads) {
      const unsigned i = i0 + tid;
      GateOut o{false, 0ULL, 0.0, 0, false, kNoEntry, kNoEntry, 0.0, 0.0, 0};
      if (i < n) o = gate_entry(L, i, gd.op, gd.c, gd.s, eps);
      if (o.append) atomicOr(flags, kFlagOverflow);  // cannot happen: all keys are stored
      const u64 m = __ballot(o.active);
      if (m) {
        const int leader = __ffsll((long long)m) - 1;
        unsigned b = 0;
        if (lane == leader) b = atomicAdd(&s_cnt, (unsigned)__popcll(m));
        b = __shfl(b, leader);
        if (o.active) lg[b + (unsigned)__popcll(m & below)] = make_rec(o);
      }
    }
    lds_barrier();
    if (tid == 0) {
      logcnt[g] = s_cnt;
      if (STAR) logcnt[M + g] = s_star;
      s_cnt = s_star = 0;
    }
    if (ncut) lds_ncut(sW, skeys, n, ncut, nst);
  }
}

template <int CAP, bool STAR>
__global__ void __launch_bounds__(kChainThreads)
k_adjoint_reverse_lds(unsigned n, const GateDesc* __restrict__ gates, const int* __restrict__ kinds,
                      const GenGate* __restrict__ gens, int M,
                      const double* __restrict__ mu_init, const char* __restrict__ logbuf, size_t log_bytes,
                      const unsigned* __restrict__ logcnt, double* __restrict__ dE_part,
                      double* __restrict__ dE) {
  __shared__ double smu[CAP];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  for (unsigned i = tid; i < n; i += kChainThreads) smu[i] = mu_init[i];
  LdsMu mu{smu};
  // The first record of this thread, the count and the angle of the next four
  // (earlier) gates are on their way while a gate is processed.
  constexpr int kAhead = 4;
  auto log_of = [&](int g) { return (const PairRec*)(logbuf + (size_t)g * log_bytes); };
  PairRec rec[kAhead];
  unsigned cnt[kAhead];
  double cs[kAhead], sn[kAhead];
  auto load = [&](int j, int g) {
    cnt[j] = 0;
    if (g < 0) return;
    cs[j] = gates[g].c;
    sn[j] = gates[g].s;
    cnt[j] = logcnt[g];
    if ((unsigned)tid < n) rec[j] = log_of(g)[tid];
  };
#pragma unroll
  for (int j = 0; j < kAhead; ++j) load(j, M - 1 - j);
  lds_barrier();
  for (int g0 = M - 1; g0 >= 0; g0 -= kAhead) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int g = g0 - j;
      if (g < 0) break;  // uniform
      double acc = 0.0;
      if ((unsigned)tid < cnt[j]) acc += adjoint_pair(rec[j], mu, cs[j], sn[j]);
      const PairRec* lg = log_of(g);
      for (unsigned r = tid + kChainThreads; r < cnt[j]; r += kChainThreads)
        acc += adjoint_pair(lg[r], mu, cs[j], sn[j]);
      bool any = (unsigned)(64 * wave) < cnt[j];
      if (STAR && kinds[g]) {  // uniform
        const GenGate gg = gens[g];
        const unsigned ns = logcnt[M + g];
        const StarRec* ls = (const StarRec*)(lg + n);
        for (unsigned r = tid; r < ns; r += kChainThreads) acc += adjoint_star(ls[r], mu, gg);
        any = true;
      }
      load(j, g - kAhead);
      if (any) acc = wave_sum63(acc);
      if (lane == 63) dE_part[(size_t)g * kWaves + wave] = acc;
      lds_barrier();  // every mu update of gate g precedes gate g - 1
    }
  }
  __syncthreads();  // dE_part is read by other threads
  for (int g = tid; g < M; g += kChainThreads) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += dE_part[(size_t)g * kWaves + w];
    dE[g] = t;
  }
}

int lds_chain_capacity() { return kLdsCap; }

hipError_t launch_chain_lds(const DeviceState& st, const GateDesc* gates, const int* kinds, const GenGate* gens,
                            int g0, int M, double eps, int prune_first, double* const* ckpt, u64* ckpt_n, int seg,
                            u64* gate_n_in, u64* gate_n_act, u64 max_keys, unsigned ncut, hipStream_t stream) {
  if (kinds)
    hipLaunchKernelGGL((k_chain_lds<kLdsCap, true>), dim3(1), dim3(kChainThreads), 0, stream, st.keys, st.amps, st.ctr,
                       gates, kinds, gens, g0, M, eps, prune_first, ckpt, ckpt_n, seg, gate_n_in, gate_n_act, max_keys, ncut);
  else
    hipLaunchKernelGGL((k_chain_lds<kLdsCap, false>), dim3(1), dim3(kChainThreads), 0, stream, st.keys, st.amps, st.ctr,
                       gates, kinds, gens, g0, M, eps, prune_first, ckpt, ckpt_n, seg, gate_n_in, gate_n_act, max_keys, ncut);
  return hipGetLastError();
}

hipError_t launch_adjoint_replay_lds(const u64* keys, unsigned n, const GateDesc* gates, const int* kinds,
                                     const GenGate* gens, int M, int seg, double eps, const double* const* ckpt,
                                     const u64* ckpt_n, char* logbuf, size_t log_bytes, unsigned* logcnt,
                                     unsigned* flags, unsigned ncut, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  const int nseg = (M + seg - 1) / seg;
  if (kinds)
    hipLaunchKernelGGL((k_adjoint_replay_lds<kLdsCap, true>), dim3(nseg), dim3(kChainThreads), 0, stream, keys, n, gates,
                       kinds, gens, M, seg, eps, ckpt, ckpt_n, logbuf, log_bytes, logcnt, flags, ncut);
  else
    hipLaunchKernelGGL((k_adjoint_replay_lds<kLdsCap, false>), dim3(nseg), dim3(kChainThreads), 0, stream, keys, n,
                       gates, kinds, gens, M, seg, eps, ckpt, ckpt_n, logbuf, log_bytes, logcnt, flags, ncut);
  return hipGetLastError();
}

hipError_t launch_adjoint_reverse_lds(unsigned n, const GateDesc* gates, const int* kinds, const GenGate* gens, int M,
                                      const double* mu_init, const char* logbuf, size_t log_bytes,
                                      const unsigned* logcnt, double* dE_part, double* dE, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  if (kinds)
    hipLaunchKernelGGL((k_adjoint_reverse_lds<kLdsCap, true>), dim3(1), dim3(kChainThreads), 0, stream, n, gates, kinds,
                       gens, M, mu_init, logbuf, log_bytes, logcnt, dE_part, dE);
  else
    hipLaunchKernelGGL((k_adjoint_reverse_lds<kLdsCap, false>), dim3(1), dim3(kChainThreads), 0, stream, n, gates, kinds,
                       gens, M, mu_init, logbuf, log_bytes, logcnt, dE_part, dE);
  return hipGetLastError();
}

size_t adjoint_lds_part_elems(int M) { return (size_t)M * kWaves; }

}  // namespace swcs
