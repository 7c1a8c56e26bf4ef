// Gates of spin-complemented generators whose two parts overlap (Sec. III), in HBM
// (per-entry logic: gen_ops.h; states that fit LDS: k_chain.hip):
// G = A1 + s A2 for pool rows 1 and 2 (A_i = T_i - T_i^dagger, s = +-1) that
// share spin-orbitals, e.g. an opposite-spin double with p = q and its spin
// complement.  exp(theta G) is applied exactly with one parameter.
//
// G links each determinant to at most two others, in two shapes:
//   pair {D, X}: one row (or its adjoint) acts on D and nothing else links X;
//     the usual rotation, at angle theta for row 1 and s theta for row 2;
//   star {C, L1, L2}: both rows act on C, G C = alpha L1 + beta L2 (alpha,
//     beta = +-1), G L1 = -alpha C, G L2 = -beta C.  G^2 C = -2 C, so on the
//     star exp(theta G) turns C and u = (alpha x1 + beta x2) / sqrt(2) at
//     frequency sqrt(2) theta and keeps the leaf combination orthogonal to u:
//       xc' = c2 xc - s2 u,  u' = s2 xc + c2 u,
//       x1' = x1 + alpha (u' - u) / sqrt(2),  x2' = x2 + beta (u' - u) / sqrt(2)
//     (c2 = cos(sqrt(2) theta), s2 = sin(sqrt(2) theta)).
// Every determinant finds its shape from its own key: a star centre is acted
// on by both rows; the partner of a determinant acted on by one row is a star
// centre exactly when the other row acts on the partner.
//
// Ownership (race-free in-place update, as for one-row gates): a pair is
// updated by the thread of its source (the member the row's T acts on) when
// that is stored, else by the other member's; a star by its centre's thread
// when the centre is stored, else by the thread of the stored leaf with the
// smaller key.  The owner writes every stored member and appends the absent
// members that survive pruning (at most two per component).
#include "gen_ops.h"

namespace swcs {

// Wave-aggregated slot reservation: every lane of the wave calls it; lanes
// with `want` get consecutive slots counted on *counter.
__device__ inline u64 wave_reserve(bool want, u64* counter) {
  const u64 m = __ballot(want);
  if (!m) return 0;
  const int lane = __lane_id();
  const int leader = __ffsll((long long)m) - 1;
  u64 b = 0;
  if (lane == leader) b = atomicAdd((unsigned long long*)counter, (unsigned long long)__popcll(m));
  b = __shfl(b, leader);
  return b + (u64)__popcll(m & ((1ULL << lane) - 1ULL));
}

constexpr int kGenThreads = 256;

// Forward gate: the same stop and count protocol as k_gate (appends of a star
// gate are bounded by twice the alive count).  A block's new keys take one add
// on the append counter per 256 entries; one per wavefront and member on the
// same address made the launch 34 us at 100,000 entries; it takes 10.
__global__ void __launch_bounds__(kGenThreads)
k_gen_gate(u64* __restrict__ keys, double* __restrict__ amps, HashSlot* __restrict__ hash, u64 hmask,
           u64 cap, Counters* __restrict__ ctr, GenGate g, double eps, u64* __restrict__ gate_n_in,
           unsigned gate_index, u64 max_keys, u64* __restrict__ gate_n_act) {
  __shared__ long long s_wsum[kGenThreads / 64];
  __shared__ unsigned s_nact[kGenThreads / 64];
  __shared__ unsigned s_wcnt[2][kGenThreads / 64];
  __shared__ u64 s_base[2];
  u64 n_in;
  const bool run = gate_begin(ctr, gate_index, cap, max_keys, 2, &n_in, gate_n_in);
  if (!run) return;  // the same in every thread
  LiveCounts* __restrict__ own = &ctr->live[live_slot(gate_index)];
  GlobalStore S{keys, amps, hash, hmask};
  const int lane = __lane_id(), wave = (int)(threadIdx.x >> 6);
  const u64 below = (1ULL << lane) - 1ULL;
  long long dalive = 0;
  unsigned nact = 0, par = 0;
  const u64 stride = (u64)gridDim.x * kGenThreads;
  for (u64 base = (u64)blockIdx.x * kGenThreads; base < n_in; base += stride, par ^= 1u) {
    const u64 i = base + threadIdx.x;
    GenOut o;
    o.napp = 0;
    o.dalive = 0;
    if (i < n_in) {
      const u64 D = keys[i];
      nact += (op_acts(g.op1, D) || op_acts(g.op2, D)) ? 1u : 0u;
      o = gen_entry(S, i, g, eps);
    }
    dalive += o.dalive;
    const u64 m0 = __ballot(o.napp > 0), m1 = __ballot(o.napp > 1);
    const unsigned mine = (unsigned)(__popcll(m0) + __popcll(m1));
    if (lane == 0) s_wcnt[par][wave] = mine;
    __syncthreads();
    unsigned before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kGenThreads / 64; ++w) {
      before += w < wave ? s_wcnt[par][w] : 0u;
      all += s_wcnt[par][w];
    }
    if (all) {  // the same in the whole block
      if (threadIdx.x == 0) s_base[par] = atomicAdd((unsigned long long*)&own->app, (unsigned long long)all);
      __syncthreads();
      const u64 at = n_in + s_base[par] + before;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (o.napp <= a) continue;
        const u64 idx = at + (a ? (u64)__popcll(m0) + (u64)__popcll(m1 & below) : (u64)__popcll(m0 & below));
        if (idx < cap) {
          keys[idx] = o.key[a];
          amps[idx] = o.val[a];
          hash_insert_new(hash, hmask, o.key[a], idx);
        } else {
          atomicOr(&ctr->flags, kFlagOverflow);
        }
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    dalive += __shfl_xor(dalive, off);
    nact += __shfl_xor(nact, off);
  }
  if (lane == 0) {
    s_wsum[wave] = dalive;
    s_nact[wave] = nact;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    long long d = 0;
    u64 na = 0;
    for (int w = 0; w < kGenThreads / 64; ++w) {
      d += s_wsum[w];
      na += s_nact[w];
    }
    if (gate_n_act && na) atomicAdd((unsigned long long*)gate_n_act, (unsigned long long)na);
    if (d != 0) atomicAdd((unsigned long long*)&own->dalive, (unsigned long long)d);
  }
}

// Replay inside the adjoint's recomputation, one gate of every segment of a
// group (blockIdx.y) as k_gate_replay: the forward update on the segment's
// working copy over the final keys (every reachable key is stored, so nothing
// is appended), logging one PairRec per updated pair and one StarRec per
// updated star.
__global__ void __launch_bounds__(kGenThreads)
k_gen_replay(const u64* __restrict__ keys, double* __restrict__ work, const HashSlot* __restrict__ hash, u64 hmask,
             u64 n, const GenGate* __restrict__ gens, double eps, ReplayGroup G, int step,
             unsigned* __restrict__ flags) {
  const int gi = G.gate(step, (int)blockIdx.y);
  if (gi < 0 || !G.star(gi)) return;  // uniform
  const GenGate g = gens[gi];
  PairRec* __restrict__ plog = G.pairs(gi);
  StarRec* __restrict__ slog = G.stars(gi);
  u64* pcount = G.counts + (gi - G.g0);
  u64* scount = G.star_counts + (gi - G.g0);
  GlobalStore S{(u64*)keys, work + (u64)blockIdx.y * n, (HashSlot*)hash, hmask};
  const u64 stride = (u64)gridDim.x * kGenThreads;
  for (u64 base = (u64)blockIdx.x * kGenThreads; base < n; base += stride) {
    const u64 i = base + threadIdx.x;
    GenOut o;
    o.napp = 0;
    o.kind = 0;
    if (i < n) o = gen_entry(S, i, g, eps);
    if (o.napp) atomicOr(flags, kFlagOverflow);
    const u64 ps = wave_reserve(o.kind == 1, pcount);
    if (o.kind == 1) plog[ps] = o.pr;
    const u64 ss = wave_reserve(o.kind == 2, scount);
    if (o.kind == 2) slog[ss] = o.sr;
  }
}

// Reverse step of the logged stars of one gate (see adjoint_star); block sums
// are added to partial[blockIdx.x] (written by the pairs' reverse step of the
// same gate).
__global__ void __launch_bounds__(256)
k_adjoint_star(const StarRec* __restrict__ slog, const u64* __restrict__ scount, double* __restrict__ mu,
               GenGate g, double* __restrict__ partial) {
  GlobalMu m{mu};
  const u64 cnt = *scount;
  double acc = 0.0;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x; r < cnt; r += stride) acc += adjoint_star(slog[r], m, g);
  __shared__ double sacc[256];
  sacc[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sacc[threadIdx.x] += sacc[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] += sacc[0];
}

hipError_t launch_gen_gate(const DeviceState& st, const GenGate& g, double eps, u64* gate_n_in,
                           unsigned gate_index, u64 max_keys, int grid, hipStream_t stream, u64* gate_n_act) {
  hipLaunchKernelGGL(k_gen_gate, dim3(grid), dim3(kGenThreads), 0, stream, st.keys, st.amps, st.hash,
                     st.hmask, st.cap, st.ctr, g, eps, gate_n_in, gate_index, max_keys, gate_n_act);
  return hipGetLastError();
}

hipError_t launch_gen_replay(const DeviceState& st, double* work, u64 n, const GenGate* gens, double eps,
                             const ReplayGroup& G, int step, int segs, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_gen_replay, dim3(grid, segs), dim3(kGenThreads), 0, stream, st.keys, work, st.hash,
                     st.hmask, n, gens, eps, G, step, &st.ctr->flags);
  return hipGetLastError();
}

hipError_t launch_adjoint_star(const StarRec* slog, const u64* scount, double* mu, const GenGate& g,
                               double* partial, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_adjoint_star, dim3(grid), dim3(256), 0, stream, slog, scount, mu, g, partial);
  return hipGetLastError();
}

}  // namespace swcs
