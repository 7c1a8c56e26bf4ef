// Pool gradients from the three-body reduced density matrix of the stored
// determinants, without forming sigma = H psi on the external space.
//
// ADAPT step 4 (Sec. II.C) asks for g_k = <psi|[H, A_k]|psi> / <psi|psi>,
// A_k = T - T+.  The commutator of a two-body H with a two-body T is at most a
// three-body operator, so g_k is a contraction of the integrals with
//   Gamma(A, B) = <C_A psi | C_B psi>,   C_A = three annihilators,
// which needs only pairs of stored determinants that share N_e - 3 electrons.
// At 52 spin-orbitals and 16 electrons a determinant has C(16, 3) = 560 such
// subsets against 29,593 records of the sort-and-join pass (k_join.hip), and
// Gamma is dense but small (1.25 GB for 26 spatial orbitals, 43 MB for 15).
// With h absorbed into V(pP|rs) = (pP|rs) + d_rs h_pP / (N_e - 3/2) and
//   G(P; Q; S, R) = sum_{p r s} V(pP|rs) [ d_sQ / 2 <p+ r+ a_S a_R>
//                                          - <p+ r+ Q+ a_s a_S a_R> ]
// a double T = P+ Q+ a_S a_R has
//   g = (2 / <psi|psi>) [G(P;Q;S,R) - G(Q;P;S,R) - G(R;S;Q,P) + G(S;R;Q,P)],
// and a single T = P+ a_Q, with B(P;Q) = sum_p h_pP <p+ a_Q> +
// sum_{p r s} (pP|rs) <p+ r+ a_s a_Q>, has g = (2 / <psi|psi>) [B(P;Q) - B(Q;P)].
// (From [H, P+] = sum_p h_pP p+ + sum (pP|rs) p+ r+ a_s, the normal ordering of
// its product with Q+, and the antisymmetry of the term that ordering leaves.)
//
// Passes: emit   -- every alive D writes one 64-bit record per subset of
//                   N_e - 3 electrons: entry index, removed triple, hash of
//                   the subset;
//         sort   -- radix sort on low hash bits (k_sort.hip);
//         pairs  -- records of one subset are the entries that share it:
//                   psi_D psi_D' into one triangle of Gamma for each pair; a
//                   state with more pairs than records sums the rows in LDS;
//         diag   -- Gamma(A, A), every subset's own square, summed in LDS;
//         mirror -- the other triangle;
//         two    -- the two-body matrix as the partial trace of Gamma;
//         contract -- G as a matrix product over (p, r, s) on the FP64 matrix
//                   cores: 1,001 x 26 x 26 by 26 per Q and column at 26
//                   orbitals, the only dense work;
//         finish -- g_k of the asked operators.
//
// Measured, whole pool, against the sort and join (to 2^31 records) or the
// accumulation table (beyond): 39,484 determinants of 52 spin-orbitals and 16
// electrons 69.6 -> 4.8 ms, 137,595 of them 480 -> 7.8 ms (813 where three
// contexts share the memory and the table is split), 224,982 of 30
// spin-orbitals and 11 electrons 67.7 -> 6.2 ms; 6 % of the pool on the first
// state 38.6 -> 4.6 ms.  Errors against 64-bit references are those of the
// other paths (2.6e-14, 1.5e-14 relative).
#include <algorithm>

#include "conn_ops.h"
#include "rdm_ops.h"

namespace swcs {

// Row strides and matrix offsets (in doubles) of Gamma's four spin blocks.
struct RdmView {
  RdmDims d;
  double* g3;
  const double* g2;
};

// ---------------------------------------------------------------- emit
constexpr int kRdmEmitBlock = 256;
constexpr int kRdmStage = 4096;  // records staged in LDS per flush (32 KB)

// The value v of lane l (uniform).
__device__ inline u64 rdm_lane(u64 v, int l) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), l);
  return ((u64)hi << 32) | lo;
}

// Position of the r-th (from 0) set bit of m.
__device__ inline int rdm_select(u64 m, unsigned r) {
  int pos = 0;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) {
    const u64 low = m & ((1ULL << w) - 1ULL);
    const unsigned c = (unsigned)__popcll(low);
    if (r >= c) {
      r -= c;
      m >>= w;
      pos += w;
    } else {
      m = low;
    }
  }
  return pos;
}

// Electron ranks i < j < k of triple code t = C(k, 3) + C(j, 2) + i.
__device__ inline void rdm_triple(unsigned t, int ne, unsigned* i, unsigned* j, unsigned* k) {
  unsigned c = 2;
  while ((int)c + 1 < ne && (c + 1) * c * (c - 1) / 6 <= t) ++c;
  t -= c * (c - 1) * (c - 2) / 6;
  unsigned b = 1;
  while (b + 1 < c && (b + 1) * b / 2 <= t) ++b;
  *k = c;
  *j = b;
  *i = t - b * (b - 1) / 2;
}

// Triple table of a block: i | j << 8 | k << 16 per code.
__device__ inline void rdm_triple_table(unsigned* tri, int ne, unsigned ntri) {
  for (unsigned t = threadIdx.x; t < ntri; t += blockDim.x) {
    unsigned i, j, k;
    rdm_triple(t, ne, &i, &j, &k);
    tri[t] = i | (j << 8) | (k << 16);
  }
}

// Record of triple t of determinant D (entry d), bits = the one-bit masks of
// D's electrons; *cls the hash class of the subset.
__device__ inline u64 rdm_emit_record(const RdmFmt& fm, u64 d, u64 D, const u64* bits, const unsigned* tri, unsigned t,
                                      unsigned* cls) {
  const unsigned c = tri[t];
  const u64 x = mix64(D ^ bits[c & 255u] ^ bits[(c >> 8) & 255u] ^ bits[c >> 16]);
  *cls = (unsigned)(x >> 56);
  return rdm_record(fm, d, t, x & ((1ULL << fm.hb) - 1ULL));
}

// All subsets of every determinant: a wavefront takes eight entries, reserves
// room for the live ones with one cursor add and writes each one's records as
// one run, lanes over its triples.  With smask only determinants whose hash is
// 0 under it (an unbiased sample: a pair is kept with the square of a
// determinant's share).  Bound by the hashes and the record write, 8 B each.
constexpr int kRdmEmitChunk = 8;
__global__ void __launch_bounds__(kRdmEmitBlock)
k_rdm_emit(const u64* __restrict__ keys, const double* __restrict__ amps, u64 n, int ne, unsigned ntri, RdmFmt fm,
           u64 smask, u64* __restrict__ recs, u64 cap, u64* __restrict__ cursor, unsigned* __restrict__ flags) {
  extern __shared__ unsigned s_tri[];  // ntri
  __shared__ u64 s_bit[kRdmEmitBlock / 64][32];
  rdm_triple_table(s_tri, ne, ntri);
  __syncthreads();
  const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
  constexpr int kW = kRdmEmitBlock / 64;
  const u64 nch = (n + kRdmEmitChunk - 1) / kRdmEmitChunk;
  for (u64 ch = (u64)blockIdx.x * kW + (u64)wave; ch < nch; ch += (u64)gridDim.x * kW) {
    const u64 e = ch * kRdmEmitChunk + (u64)lane;
    bool live = lane < kRdmEmitChunk && e < n;
    live = live && !is_dead(amps[live ? e : 0]);
    const u64 key = live ? keys[e] : 0ULL;
    if (smask) live = live && (mix64(key ^ 0x9e3779b97f4a7c15ULL) & smask) == 0;
    u64 m = __ballot(live);
    if (m == 0) continue;  // uniform over the wavefront
    const u64 cnt = (u64)__popcll(m) * ntri;
    u64 base = 0;
    if (lane == 0) base = atomicAdd(cursor, cnt);
    base = rdm_lane(base, 0);
    if (base + cnt > cap) {
      if (lane == 0) atomicOr(flags, kFlagOverflow);
      continue;
    }
    for (; m; m &= m - 1) {
      const int j = __ffsll((long long)m) - 1;
      const u64 D = rdm_lane(key, j), d = ch * kRdmEmitChunk + (u64)j;
      if (lane < ne) s_bit[wave][lane] = 1ULL << rdm_select(D, (unsigned)lane);
      wave_sync();  // read by this wavefront only, after its writes
      unsigned cls;
      for (unsigned t = (unsigned)lane; t < ntri; t += 64)
        recs[base + t] = rdm_emit_record(fm, d, D, s_bit[wave], s_tri, t, &cls);
      base += ntri;
      wave_sync();
    }
  }
}

// The subsets of one hash class of nbatch (all records of a subset are in one
// class, so that the sort buffers of a large state stay bounded): one
// wavefront per determinant, the kept records of the block staged in LDS and
// flushed as one run behind one cursor add.
__global__ void __launch_bounds__(kRdmEmitBlock)
k_rdm_emit_class(const u64* __restrict__ keys, const double* __restrict__ amps, u64 n, int ne, unsigned ntri,
                 RdmFmt fm, int nbatch, int batch, u64* __restrict__ recs, u64 cap, u64* __restrict__ cursor,
                 unsigned* __restrict__ flags) {
  extern __shared__ unsigned s_tri[];  // ntri
  __shared__ u64 s_rec[kRdmStage];
  __shared__ u64 s_bit[kRdmEmitBlock / 64][32];
  __shared__ unsigned s_cnt;
  __shared__ u64 s_base;
  rdm_triple_table(s_tri, ne, ntri);
  if (threadIdx.x == 0) s_cnt = 0;
  __syncthreads();
  const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
  constexpr int kW = kRdmEmitBlock / 64;
  const u64 step = (u64)gridDim.x * kW;
  auto flush = [&]() {  // called by every thread of the block
    __syncthreads();
    const unsigned cnt = s_cnt;
    if (threadIdx.x == 0) s_base = atomicAdd(cursor, (u64)cnt);
    __syncthreads();
    const u64 base = s_base;
    for (unsigned q = threadIdx.x; q < cnt; q += kRdmEmitBlock) {
      if (base + q < cap) recs[base + q] = s_rec[q];
      else atomicOr(flags, kFlagOverflow);
    }
    __syncthreads();
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
  };
  // Every wavefront of the block makes the same trips, so the flush after each
  // kRdmStage / kRdmEmitBlock rounds (a round adds at most one record per
  // thread) is met by the whole block.
  int round = 0;
  for (u64 d0 = (u64)blockIdx.x * kW; d0 < n; d0 += step) {
    const u64 d = d0 + (u64)wave;
    const bool live = d < n && !is_dead(amps[d < n ? d : 0]);
    const u64 D = live ? keys[d] : 0ULL;
    if (live && lane < ne) s_bit[wave][lane] = 1ULL << rdm_select(D, (unsigned)lane);
    wave_sync();  // read by this wavefront only, after its writes
    for (unsigned t0 = 0; t0 < ntri; t0 += 64) {
      const unsigned t = t0 + (unsigned)lane;
      bool put = live && t < ntri;
      u64 rec = 0;
      if (put) {
        unsigned cls;
        rec = rdm_emit_record(fm, d, D, s_bit[wave], s_tri, t, &cls);
        put = (int)(cls & (unsigned)(nbatch - 1)) == batch;
      }
      const u64 m = __ballot(put);
      if (m) {  // uniform over the wavefront
        unsigned b = 0;
        if (lane == 0) b = atomicAdd(&s_cnt, (unsigned)__popcll(m));
        b = (unsigned)__shfl((int)b, 0);
        if (put) s_rec[b + (unsigned)__popcll(m & ((1ULL << lane) - 1ULL))] = rec;
      }
      if (++round == kRdmStage / kRdmEmitBlock) {
        flush();
        round = 0;
      }
    }
    wave_sync();
  }
  flush();
}

// ---------------------------------------------------------------- count
// Sum over buckets (records of equal low sort bits) of m (m - 1) / 2: an upper
// bound on the pairs of the next pass.  The first record of a bucket finds its
// end by doubling steps and a bisection.
__global__ void __launch_bounds__(256)
k_rdm_count(const u64* __restrict__ recs, u64 R, int sort_bits, double* __restrict__ partial) {
  __shared__ double red[256];
  const u64 bmask = (1ULL << sort_bits) - 1ULL;
  double acc = 0.0;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 g = (u64)blockIdx.x * blockDim.x + threadIdx.x; g < R; g += stride) {
    const u64 b = recs[g] & bmask;
    if (g > 0 && (recs[g - 1] & bmask) == b) continue;
    u64 lo = g, hop = 1;  // recs[lo] is in the bucket
    while (lo + hop < R && (recs[lo + hop] & bmask) == b) {
      lo += hop;
      hop <<= 1;
    }
    while (hop > 1) {
      hop >>= 1;
      if (lo + hop < R && (recs[lo + hop] & bmask) == b) lo += hop;
    }
    const double m = (double)(lo - g + 1);
    acc += 0.5 * m * (m - 1.0);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------- pairs
// A record decoded: the subset, the canonical triple's block and index, and
// psi(D) with the sign of C_A |D>.  val = 0 for a record that names no entry.
struct RdmSide {
  u64 S;
  double val;
  int blk;
  unsigned idx;
};

__device__ inline RdmSide rdm_decode(u64 rec, const RdmFmt& fm, const RdmDims& dm, int ne,
                                     const unsigned* __restrict__ tri, unsigned ntri, const u64* __restrict__ keys,
                                     const double* __restrict__ amps, u64 n) {
  RdmSide o{0ULL, 0.0, 0, 0u};
  const u64 d = rdm_record_entry(fm, rec);
  const unsigned t = rdm_record_triple(fm, rec);
  if (d >= n || t >= ntri) return o;
  const double a = amps[d];
  if (is_dead(a)) return o;
  const u64 D = keys[d];
  const unsigned c = tri[t];
  const int x = rdm_select(D, c & 255u), y = rdm_select(D, (c >> 8) & 255u), z = rdm_select(D, c >> 16);
  int sgn;
  rdm_canonical(dm, D, x, y, z, &o.blk, &o.idx, &sgn);
  o.S = D ^ (1ULL << x) ^ (1ULL << y) ^ (1ULL << z);
  o.val = sgn ? -a : a;
  return o;
}

constexpr int kRdmPairBlock = 512;
constexpr int kRdmPairTile = 1024;
constexpr int kRdmPairHalo = 256;
constexpr int kRdmPairAll = kRdmPairTile + kRdmPairHalo;

// Every pair of records with one subset, once, into the triangle row <= column
// of Gamma (k_rdm_mirror writes the other one).  A block takes 1,024 sorted
// records and the 256 after them.  Most subsets belong to one entry only: the
// records with an equal hash ahead of or behind them in their bucket are
// listed, and only those are decoded (into LDS, full wavefronts) and paired; a
// record beyond the halo is decoded where it is met.
__global__ void __launch_bounds__(kRdmPairBlock)
k_rdm_pairs(const u64* __restrict__ recs, u64 R, RdmFmt fm, int sort_bits, int ne, unsigned ntri,
            const u64* __restrict__ keys, const double* __restrict__ amps, u64 n, RdmView V) {
  __shared__ u64 s_rec[kRdmPairAll];
  __shared__ u64 s_S[kRdmPairAll];
  __shared__ double s_val[kRdmPairAll];
  __shared__ unsigned s_idx[kRdmPairAll];
  __shared__ unsigned char s_hit[kRdmPairAll];
  __shared__ unsigned short s_list[kRdmPairAll];
  __shared__ unsigned s_nlist;
  extern __shared__ unsigned s_tri[];  // ntri
  rdm_triple_table(s_tri, ne, ntri);
  const u64 bmask = (1ULL << sort_bits) - 1ULL, hmask = (1ULL << fm.hb) - 1ULL;
  const u64 ntiles = (R + kRdmPairTile - 1) / kRdmPairTile;
  const int lane = (int)(threadIdx.x & 63u);
  for (u64 tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
    const u64 t0 = tl * kRdmPairTile;
    const int have = (int)((R - t0) < (u64)kRdmPairAll ? (R - t0) : (u64)kRdmPairAll);
    const int own = have < kRdmPairTile ? have : kRdmPairTile;
    __syncthreads();
    for (int i = threadIdx.x; i < have; i += kRdmPairBlock) {
      s_rec[i] = recs[t0 + i];
      s_hit[i] = 0;
    }
    if (threadIdx.x == 0) s_nlist = 0;
    __syncthreads();
    // the next equal hash of the bucket marks both records, so every member of
    // a group that is met within the tile is marked
    for (int i = threadIdx.x; i < have; i += kRdmPairBlock) {
      const u64 r = s_rec[i], b = r & bmask, h = r & hmask;
      int j = i + 1;
      while (j < have && (s_rec[j] & bmask) == b && (s_rec[j] & hmask) != h) ++j;
      if (j < have && (s_rec[j] & hmask) == h) {
        s_hit[i] = 1;
        s_hit[j] = 1;
      } else if (j == have && t0 + have < R) {
        s_hit[i] = 1;  // the bucket may go on past the halo
      }
    }
    __syncthreads();
    for (int i0 = 0; i0 < have; i0 += kRdmPairBlock) {  // same trips in every thread
      const int i = i0 + (int)threadIdx.x;
      const bool hit = i < have && s_hit[i];
      const u64 m = __ballot(hit);
      if (m) {
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(&s_nlist, (unsigned)__popcll(m));
        at = (unsigned)__shfl((int)at, 0);
        if (hit) s_list[at + (unsigned)__popcll(m & ((1ULL << lane) - 1ULL))] = (unsigned short)i;
      }
    }
    __syncthreads();
    const unsigned nlist = s_nlist;
    for (unsigned q = threadIdx.x; q < nlist; q += kRdmPairBlock) {
      const int i = s_list[q];
      const RdmSide o = rdm_decode(s_rec[i], fm, V.d, ne, s_tri, ntri, keys, amps, n);
      s_S[i] = o.S;
      s_val[i] = o.val;
      s_idx[i] = ((unsigned)o.blk << 28) | o.idx;
    }
    __syncthreads();
    for (unsigned q = threadIdx.x; q < nlist; q += kRdmPairBlock) {
      const int i = s_list[q];
      const double vi = s_val[i];
      if (i >= own || vi == 0.0) continue;
      const u64 b = s_rec[i] & bmask, h = s_rec[i] & hmask, S = s_S[i];
      const int blk = (int)(s_idx[i] >> 28);
      const unsigned A = s_idx[i] & 0x0fffffffu;
      double* __restrict__ g = V.g3 + V.d.off[blk];
      const u64 ld = V.d.ld[blk];
      for (u64 j = (u64)i + 1; t0 + j < R; ++j) {
        const u64 rj = j < (u64)have ? s_rec[j] : recs[t0 + j];
        if ((rj & bmask) != b) break;
        if ((rj & hmask) != h) continue;
        RdmSide o;
        if (j < (u64)have) {
          o.S = s_S[j];
          o.val = s_val[j];
          o.blk = (int)(s_idx[j] >> 28);
          o.idx = s_idx[j] & 0x0fffffffu;
        } else {
          o = rdm_decode(rj, fm, V.d, ne, s_tri, ntri, keys, amps, n);
        }
        if (o.val == 0.0 || o.S != S || o.blk != blk) continue;
        const unsigned lo = A < o.idx ? A : o.idx, hi = A < o.idx ? o.idx : A;
        unsafeAtomicAdd(&g[(u64)lo * ld + hi], vi * o.val);
      }
    }
  }
}

// ---------------------------------------------------------------- rows
// The pairs of a crowded state.  k_rdm_pairs adds every pair to Gamma in memory,
// 18 G/s whatever the size of Gamma: 14.4 of 16.2 ms for 2.6e8 pairs of 225,000
// determinants of 30 spin-orbitals.  Here a row of Gamma lies in LDS while its
// pairs are added (at most 15,872 doubles, 124 KB, at 32 orbitals):
//   members -- the sorted records, decoded, in the order (bucket, subset,
//              triple): a record's place is counted over its bucket in LDS
//              (1.2 ms for 3.7e7 records); one with others behind it is also
//              listed under its triple, which is its row;
//   sort    -- the list by row, two digits (0.5 ms);
//   rows    -- a block takes a range of the list; eight lanes add a record's
//              pairs with the members behind it, 16 bytes each, and the row
//              goes to memory when it is done (1.4 ms, bound by these reads).
// RdmMember.rem: members of the subset behind this one.
struct alignas(16) RdmMember {
  double val;
  unsigned idx, rem;
};

constexpr int kRdmRowBits = 16;  // block (2) and index (14) of a row
constexpr int kRdmMemTile = 1024;
constexpr int kRdmMemHalo = 1024;
constexpr int kRdmMemAll = kRdmMemTile + kRdmMemHalo;
constexpr int kRdmMemBlock = 512;
constexpr int kRdmMemPer = kRdmMemAll / kRdmMemBlock;

// A block takes the buckets that begin in its tile; one that goes on past the
// halo (more than 1,024 records) sets cursor[1], and the caller takes
// k_rdm_pairs.  cursor[0]: length of the list.
__global__ void __launch_bounds__(kRdmMemBlock)
k_rdm_members(const u64* __restrict__ recs, u64 R, RdmFmt fm, int sort_bits, int ne, unsigned ntri,
              const u64* __restrict__ keys, const double* __restrict__ amps, u64 n, RdmDims dm,
              RdmMember* __restrict__ mem, u64* __restrict__ list, u64* __restrict__ cursor) {
  constexpr unsigned kWords = kRdmMemAll / 64;
  __shared__ u64 s_S[kRdmMemAll];
  __shared__ unsigned s_b[kRdmMemAll + 1], s_idx[kRdmMemAll];
  __shared__ u64 s_head[kWords];  // one bit per record that begins a bucket
  __shared__ unsigned s_cnt;
  __shared__ u64 s_base;
  extern __shared__ unsigned s_tri[];  // ntri
  rdm_triple_table(s_tri, ne, ntri);
  const u64 bmask = (1ULL << sort_bits) - 1ULL;
  const u64 ntiles = (R + kRdmMemTile - 1) / kRdmMemTile;
  const int lane = (int)(threadIdx.x & 63u);
  // first bucket that begins at i or later (kRdmMemAll: none in the tile)
  auto next_head = [&](unsigned i) {
    unsigned w = i >> 6;
    if (w >= kWords) return (unsigned)kRdmMemAll;
    u64 m = s_head[w] & (~0ULL << (i & 63u));
    while (m == 0 && ++w < kWords) m = s_head[w];
    return m ? (w << 6) + (unsigned)__ffsll((long long)m) - 1u : (unsigned)kRdmMemAll;
  };
  for (u64 tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
    const u64 t0 = tl * kRdmMemTile;
    const unsigned have = (unsigned)((R - t0) < (u64)kRdmMemAll ? (R - t0) : (u64)kRdmMemAll);
    const unsigned own = have < (unsigned)kRdmMemTile ? have : (unsigned)kRdmMemTile;
    u64 rec[kRdmMemPer];
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k) {
      const u64 at = t0 + threadIdx.x + (u64)k * kRdmMemBlock;
      rec[k] = recs[at < R ? at : R - 1];
    }
    __syncthreads();  // the tile before is done with LDS
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k) s_b[1 + threadIdx.x + k * kRdmMemBlock] = (unsigned)(rec[k] & bmask);
    if (threadIdx.x == 0) {
      s_b[0] = t0 > 0 ? (unsigned)(recs[t0 - 1] & bmask) : ~s_b[1];  // bucket before the tile
      s_cnt = 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k) {
      const unsigned i = threadIdx.x + k * kRdmMemBlock;
      const u64 m = __ballot(i < have ? s_b[i] != s_b[i + 1] : t0 + have == R);  // past the end: a head
      if (lane == 0) s_head[i >> 6] = m;
    }
    __syncthreads();
    const unsigned begin = next_head(0);
    unsigned end = next_head(own);
    if (begin >= own) continue;  // inside a bucket of an earlier tile
    if (end == (unsigned)kRdmMemAll && t0 + (u64)kRdmMemAll != R) {
      // a head may still stand right behind the halo; it is not looked for
      if (threadIdx.x == 0) __hip_atomic_store(&cursor[1], (u64)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    double val[kRdmMemPer];
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k) {
      const unsigned i = threadIdx.x + k * kRdmMemBlock;
      val[k] = 0.0;
      if (i < begin || i >= end) continue;
      const RdmSide o = rdm_decode(rec[k], fm, dm, ne, s_tri, ntri, keys, amps, n);
      val[k] = o.val;
      s_S[i] = o.S;
      s_idx[i] = ((unsigned)o.blk << 14) | o.idx;
    }
    __syncthreads();
    unsigned slot[kRdmMemPer], at[kRdmMemPer];
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k) {
      const unsigned i = threadIdx.x + k * kRdmMemBlock;
      bool put = false;
      slot[k] = 0xffffffffu;
      at[k] = 0;
      if (i >= begin && i < end) {
        // bucket [lo, hi) of record i
        unsigned w = i >> 6;
        u64 m = s_head[w] & (~0ULL >> (63u - (i & 63u)));
        while (m == 0) m = s_head[--w];  // `begin` is a head
        const unsigned lo = (w << 6) + 63u - (unsigned)__clzll((long long)m);
        const unsigned hi = next_head(i + 1) < end ? next_head(i + 1) : end;
        // place within the bucket by (subset, triple); one subset's triples differ
        const unsigned id = s_idx[i];
        const u64 S = s_S[i];
        unsigned less = 0, rem = 0;
        for (unsigned j0 = lo; j0 < hi; j0 += 4) {
          u64 Sj[4];
          unsigned dj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned j = j0 + u < hi ? j0 + u : i;  // record i itself counts for nothing
            Sj[u] = s_S[j];
            dj[u] = s_idx[j];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const bool same = Sj[u] == S;
            less += (Sj[u] < S || (same && dj[u] < id)) ? 1u : 0u;
            rem += (same && dj[u] > id) ? 1u : 0u;
          }
        }
        at[k] = lo + less;
        mem[t0 + at[k]] = RdmMember{val[k], id, rem};
        put = rem != 0;
      }
      const u64 m = __ballot(put);
      if (m) {
        unsigned first = 0;
        if (lane == 0) first = atomicAdd(&s_cnt, (unsigned)__popcll(m));
        first = (unsigned)__shfl((int)first, 0);
        if (put) slot[k] = first + (unsigned)__popcll(m & ((1ULL << lane) - 1ULL));
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) s_base = atomicAdd((unsigned long long*)cursor, (unsigned long long)s_cnt);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRdmMemPer; ++k)
      if (slot[k] != 0xffffffffu)
        list[s_base + slot[k]] = ((t0 + at[k]) << kRdmRowBits) | s_idx[threadIdx.x + k * kRdmMemBlock];
  }
}

// End of every row that occurs in the sorted list.
__global__ void __launch_bounds__(256)
k_rdm_row_ends(const u64* __restrict__ list, u64 Q, unsigned* __restrict__ row_end) {
  const u64 stride = (u64)gridDim.x * blockDim.x, mask = (1ULL << kRdmRowBits) - 1ULL;
  for (u64 q = (u64)blockIdx.x * blockDim.x + threadIdx.x; q < Q; q += stride) {
    const u64 r = list[q] & mask;
    if (q + 1 == Q || (list[q + 1] & mask) != r) row_end[r] = (unsigned)(q + 1);
  }
}

constexpr int kRdmRowBlock = 512;
constexpr int kRdmRowLanes = 8;      // of a record: eight members are a cache line
// Records of the list per block: 8,192, fewer where that leaves the chip idle (a
// block writes out the rows of its range one after the other).
constexpr unsigned kRdmRowChunkMax = 8192, kRdmRowChunkMin = 512;

__global__ void __launch_bounds__(kRdmRowBlock)
k_rdm_rows(const u64* __restrict__ list, u64 Q, const unsigned* __restrict__ row_end,
           const RdmMember* __restrict__ mem, u64 R, unsigned width, unsigned chunk, RdmView V) {
  extern __shared__ double s_row[];  // width
  const u64 mask = (1ULL << kRdmRowBits) - 1ULL;
  const unsigned l = threadIdx.x % kRdmRowLanes, g = threadIdx.x / kRdmRowLanes;
  constexpr unsigned kStep = kRdmRowBlock / kRdmRowLanes;
  for (unsigned i = threadIdx.x; i < width; i += kRdmRowBlock) s_row[i] = 0.0;
  __syncthreads();
  const u64 q0 = (u64)blockIdx.x * chunk, q1 = q0 + chunk < Q ? q0 + chunk : Q;
  for (u64 q = q0; q < q1;) {
    const unsigned row = (unsigned)(list[q] & mask);
    const u64 e = row_end[row] < q1 ? row_end[row] : q1;
    u64 p = q + g < e ? list[q + g] >> kRdmRowBits : 0;
    for (u64 r = q + g; r < e; r += kStep) {
      const u64 next = list[r + kStep < e ? r + kStep : r];
      const RdmMember me = mem[p];
      // the first eight members behind, loaded before their number is known
      const u64 first = p + 1 + l;
      const RdmMember o = mem[first < R ? first : R - 1];
      if (l < me.rem) unsafeAtomicAdd(&s_row[o.idx & 0x3fffu], me.val * o.val);
      for (unsigned k = l + kRdmRowLanes; k < me.rem; k += kRdmRowLanes) {
        const RdmMember x = mem[p + 1 + k];
        unsafeAtomicAdd(&s_row[x.idx & 0x3fffu], me.val * x.val);
      }
      p = next >> kRdmRowBits;
    }
    __syncthreads();
    const int blk = (int)(row >> 14);
    const unsigned A = row & 0x3fffu, len = V.d.len[blk];
    double* __restrict__ gr = V.g3 + V.d.off[blk] + (u64)A * V.d.ld[blk];
    for (unsigned i = threadIdx.x; i < len; i += kRdmRowBlock) {
      const double v = s_row[i];
      if (v != 0.0) {
        s_row[i] = 0.0;
        unsafeAtomicAdd(&gr[i], v);
      }
    }
    __syncthreads();
    q = e;
  }
}

// Clears what the pair and diagonal passes add to and what the contraction
// reads but nothing writes: the columns from the diagonal on (padding
// included) and the zero row of each block.  k_rdm_mirror writes the rest.
__global__ void __launch_bounds__(256)
k_rdm_clear(RdmView V) {
  const int blk = (int)blockIdx.y;
  const unsigned len = V.d.len[blk], ld = V.d.ld[blk];
  double* __restrict__ g = V.g3 + V.d.off[blk];
  for (unsigned r = blockIdx.x; r <= len; r += gridDim.x) {
    double2* __restrict__ row = reinterpret_cast<double2*>(g + (u64)r * ld);  // ld is a multiple of 8
    for (unsigned c = (r < len ? r / 2 : 0u) + threadIdx.x; c < ld / 2; c += 256) row[c] = double2{0.0, 0.0};
  }
}

// The rows of Gamma below the diagonal from those above it, in 32 x 32 tiles
// through LDS (blockIdx.x: tile of the triangle, blockIdx.y: spin block).
__global__ void __launch_bounds__(256)
k_rdm_mirror(RdmView V) {
  __shared__ double s[32][33];
  const int blk = (int)blockIdx.y;
  const unsigned len = V.d.len[blk], nt = (len + 31) / 32;
  // tile (r, c), r <= c, at c (c + 1) / 2 + r
  const u64 t = blockIdx.x;
  u64 c = (u64)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while (c * (c + 1) / 2 > t) --c;
  while ((c + 1) * (c + 2) / 2 <= t) ++c;
  const u64 r = t - c * (c + 1) / 2;
  if (c >= nt) return;
  double* __restrict__ g = V.g3 + V.d.off[blk];
  const u64 ld = V.d.ld[blk];
  const unsigned x = threadIdx.x & 31u, y = threadIdx.x >> 5;
  for (unsigned k = y; k < 32; k += 8) {
    const u64 row = r * 32 + k, col = c * 32 + x;
    s[k][x] = (row < len && col < len) ? g[row * ld + col] : 0.0;
  }
  __syncthreads();
  for (unsigned k = y; k < 32; k += 8) {
    const u64 row = c * 32 + k, col = r * 32 + x;
    if (row < len && col < len && row > col) g[row * ld + col] = s[x][k];
  }
}

// ---------------------------------------------------------------- diagonal
__host__ __device__ inline unsigned rdm_diag_slices(unsigned len) { return (len + 7679u) / 7680u; }

// Gamma(A, A) = sum of psi(D)^2 over the D that hold A.  blockIdx.y is a slice
// of at most kRdmDiagLds triples of one spin block, summed in LDS and added to
// memory once per block.
constexpr int kRdmDiagBlock = 512;
constexpr unsigned kRdmDiagLds = 7680;  // with the orbital lists and pairs below 64 KB
__global__ void __launch_bounds__(kRdmDiagBlock)
k_rdm_diag(const u64* __restrict__ keys, const double* __restrict__ amps, u64 n, RdmView V) {
  __shared__ double s_diag[kRdmDiagLds];
  __shared__ int s_occ[kRdmDiagBlock / 64][2][32];
  __shared__ unsigned char s_px[496], s_py[496];  // pairs of at most 32 electrons
  int blk = 0;
  unsigned slice = blockIdx.y;
  while (blk < 3 && slice >= rdm_diag_slices(V.d.len[blk])) slice -= rdm_diag_slices(V.d.len[blk++]);
  const unsigned lo = slice * kRdmDiagLds;
  if (lo >= V.d.len[blk]) return;
  const unsigned len = V.d.len[blk] - lo < kRdmDiagLds ? V.d.len[blk] - lo : kRdmDiagLds;
  for (unsigned t = threadIdx.x; t < len; t += kRdmDiagBlock) s_diag[t] = 0.0;
  for (unsigned t = threadIdx.x; t < 496; t += kRdmDiagBlock) {
    int x, y;
    rdm_pair_split(t, &x, &y);
    s_px[t] = (unsigned char)x;
    s_py[t] = (unsigned char)y;
  }
  const bool one_spin = blk == 0 || blk == 3;
  const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
  constexpr int kW = kRdmDiagBlock / 64;
  const u64 amask = 0x5555555555555555ULL;
  // the spin with three or two of the triple's electrons
  const int sp = blk <= 1 ? 0 : 1;
  __syncthreads();
  // a wavefront loads 16 determinants at a time, the next 16 before it works
  // on these
  constexpr int kChunk = 16;
  const u64 nch = (n + kChunk - 1) / kChunk, cstep = (u64)gridDim.x * kW;
  u64 ch = (u64)blockIdx.x * kW + (u64)wave;
  u64 nk = 0, na_bits = kDeadBits;
  if (ch < nch && lane < kChunk && ch * kChunk + lane < n) {
    nk = keys[ch * kChunk + lane];
    na_bits = (u64)__double_as_longlong(amps[ch * kChunk + lane]);
  }
  for (; ch < nch; ch += cstep) {
  const u64 ck = nk, ca = na_bits;
  const u64 nx_ch = ch + cstep;
  na_bits = kDeadBits;
  if (nx_ch < nch && lane < kChunk && nx_ch * kChunk + lane < n) {
    nk = keys[nx_ch * kChunk + lane];
    na_bits = (u64)__double_as_longlong(amps[nx_ch * kChunk + lane]);
  }
  for (int j = 0; j < kChunk; ++j) {
    const double a = __longlong_as_double((long long)rdm_lane(ca, j));
    if (is_dead(a)) continue;  // uniform over the wavefront
    const u64 D = rdm_lane(ck, j);
    const double w = a * a;
    const int na = __popcll(D & amask), nb = __popcll(D & ~amask);
    if (lane < na) s_occ[wave][0][lane] = rdm_select(D & amask, (unsigned)lane) >> 1;
    if (lane < nb) s_occ[wave][1][lane] = rdm_select(D & ~amask, (unsigned)lane) >> 1;
    wave_sync();  // read by this wavefront only, after its writes
    const int* ox = s_occ[wave][sp];
    const int* oy = s_occ[wave][1 - sp];
    const int nx = sp ? nb : na, ny = sp ? na : nb;
    // two lanes per pair x < y, each taking every other third electron
    const int npair = nx * (nx - 1) / 2;
    for (int q = lane; q < 2 * npair; q += 64) {
      const int x = s_px[q >> 1], y = s_py[q >> 1];
      unsigned base;
      int end;
      const int* o;
      if (one_spin) {  // a < b < c: a below x
        base = rdm_c3((unsigned)ox[y]) + rdm_c2((unsigned)ox[x]);
        end = x;
        o = ox;
      } else {
        base = (rdm_c2((unsigned)ox[y]) + (unsigned)ox[x]) * (unsigned)V.d.n;
        end = ny;
        o = oy;
      }
      base -= lo;
      for (int e = q & 1; e < end; e += 2) {
        const unsigned id = base + (unsigned)o[e];
        if (id < len) atomicAdd(&s_diag[id], w);
      }
    }
    wave_sync();
  }
  }
  __syncthreads();
  double* g = V.g3 + V.d.off[blk];
  const u64 ld = V.d.ld[blk];
  for (unsigned t = threadIdx.x; t < len; t += kRdmDiagBlock) {
    const double v = s_diag[t];
    if (v != 0.0) unsafeAtomicAdd(&g[(u64)(lo + t) * ld + lo + t], v);
  }
}

// ---------------------------------------------------------------- two-body
// Gamma2(A2, B2) as the partial trace of Gamma over the orbitals x of one spin,
//   sum_x sgn(x A2) sgn(x B2) Gamma(x A2, x B2) / (electrons of that spin left),
// one block per (row A2, 256 columns B2) of the three spin blocks (aa, ab, bb),
// A2 and B2 canonical: pair index for equal spins, alpha n + beta for mixed.
// The rows x A2 of Gamma are the same for the block and listed in LDS.  The
// traced spin (spin[cls], factor inv[cls]) is beta where it can be: Gamma's
// columns then run along the threads.  Tracing both spins read twice the rows
// and, with 64-line gathers, took 250 us at 26 orbitals.
struct RdmTrace {
  int spin[3];
  double inv[3];
};
__global__ void __launch_bounds__(256)
k_rdm_two(RdmView V, RdmTrace tr, double* __restrict__ g2) {
  __shared__ const double* s_row[32];
  __shared__ int s_sg[32];  // 2 = no row
  const RdmDims& d = V.d;
  const unsigned np = d.np, nn = (unsigned)(d.n * d.n);
  unsigned A = blockIdx.x;
  int cls = 0;
  if (A >= np) {
    A -= np;
    cls = 1;
    if (A >= nn) {
      A -= nn;
      cls = 2;
    }
  }
  const unsigned ncol = cls == 1 ? nn : np;
  if (blockIdx.y * 256 >= ncol) return;
  const int sp = tr.spin[cls];
  if ((int)threadIdx.x < d.n) {
    int a0, a1, blk, sg;
    unsigned ia;
    rdm_pair_orbitals(d, cls, A, &a0, &a1);
    const bool ok = rdm_sorted(d, 2 * (int)threadIdx.x + sp, a0, a1, &blk, &ia, &sg);
    s_sg[threadIdx.x] = ok ? sg : 2;
    s_row[threadIdx.x] = ok ? V.g3 + d.off[blk] + (u64)ia * d.ld[blk] : V.g3;
  }
  __syncthreads();
  unsigned B = blockIdx.y * 256 + threadIdx.x;
  if (B >= ncol) return;
  // mixed columns with the alpha running fastest, as Gamma's columns do
  if (cls == 1) B = (B % (unsigned)d.n) * (unsigned)d.n + B / (unsigned)d.n;
  int b0, b1;
  rdm_pair_orbitals(d, cls, B, &b0, &b1);
  double acc = 0.0;
  // loads without branches (column 0 of a row with weight 0 where x is in the
  // pair already), so that several are in flight
#pragma unroll 4
  for (int x = 0; x < d.n; ++x) {
    const int sa = s_sg[x];
    int blk, sb = 0;
    unsigned ib = 0;
    const bool ok = rdm_sorted(d, 2 * x + sp, b0, b1, &blk, &ib, &sb) && sa <= 1;
    const double v = s_row[x][ok ? ib : 0u];
    acc += ok ? ((sa ^ sb) ? -v : v) : 0.0;
  }
  const u64 base = cls == 0 ? 0 : (cls == 1 ? (u64)np * np : (u64)np * np + (u64)nn * nn);
  g2[base + (u64)A * ncol + B] = acc * tr.inv[cls];
}

// ---------------------------------------------------------------- integrals
// V in the A-operand order of the FP64 16x16x4 matrix instruction: item
// (p, r) -- the np pairs p < r first, antisymmetrised for equal spins, then
// all (p, r) for opposite spins -- then row tile mt, k step ks, lane:
// P = 16 mt + lane % 16, s = 4 ks + lane / 16 (0 outside).
__global__ void __launch_bounds__(256)
k_rdm_vtab(Ints I, RdmDims d, int mt_n, int ks_n, double c, double* __restrict__ tab) {
  const u64 per = (u64)mt_n * ks_n * 64;
  const u64 total = ((u64)d.np + (u64)d.n * d.n) * per;
  const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const unsigned item = (unsigned)(t / per), in = (unsigned)(t % per);
  const int lane = (int)(in & 63u), ks = (int)((in >> 6) % (unsigned)ks_n), mt = (int)((in >> 6) / (unsigned)ks_n);
  const int P = 16 * mt + (lane & 15), s = 4 * ks + (lane >> 4);
  double v = 0.0;
  if (P < d.n && s < d.n) {
    int p, r;
    const bool same = item < d.np;
    if (same) {
      rdm_pair_split(item, &p, &r);
    } else {
      p = (int)((item - d.np) / (unsigned)d.n);
      r = (int)((item - d.np) % (unsigned)d.n);
    }
    v = eri_sp(I, p, P, r, s);
    if (r == s) v += c * I.h[p * d.n + P];
    if (same) {
      v -= eri_sp(I, r, P, p, s);
      if (p == s) v -= c * I.h[r * d.n + P];
    }
  }
  tab[t] = v;
}

// ---------------------------------------------------------------- contract
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kRdmNT = 2;  // column tiles of 16 per wavefront

// Work of one wavefront of k_rdm_contract: G(P; Q; col) for every P of one
// spin, one Q and 32 columns (annihilator pairs), over a chunk of the (p, r)
// items of one kind.
//
// As a matrix product the sum over (p, r, s) has 26 rows (P) and K = (p, r, s):
// per item (p, r) the A operand is V's 26 x 26 slice and the B operand 26 x 32
// values of one row of Gamma, gathered through column offsets that depend only
// on (s, column) and so stay in registers for the whole chunk: one load and one
// sign flip per B element, used for all P.  B elements that vanish (an index
// twice) read the zero column each row carries, rows that vanish the zero row
// behind the block.  Bound by the FP64 matrix rate and the reads of Gamma (each
// row once per spin, Q and kind); columns are ordered so that 16 lanes read
// neighbouring elements.  Chunks write partial sums that k_rdm_sum
// adds in order, which keeps the result free of scheduling order.
template <int KS>
__global__ void __launch_bounds__(256)
k_rdm_contract(RdmView V, const double* __restrict__ vtab, int chunks_same, int chunks_opp,
               double* __restrict__ part, u64 part_stride) {
  constexpr int MT = KS > 4 ? 2 : 1;
  constexpr int kPer = MT * KS * 64;
  __shared__ double s_a[2][kPer];
  const RdmDims d = V.d;
  const int n = d.n, lane = (int)(threadIdx.x & 63u), li = lane & 15, lk = lane >> 4;
  const int np = (int)d.np, nn = n * n;
  constexpr int kCols = 16 * kRdmNT;
  const int gs = (np + kCols - 1) / kCols, go = (nn + kCols - 1) / kCols;
  // Workgroups go to the eight XCDs in turn: each XCD takes a contiguous range
  // of the (chunk, wave group) list, so that the column groups of one Q, which
  // read the same rows of Gamma, share an L2.
  const unsigned per_q = (unsigned)(gs + go);
  const unsigned groups = (2u * (unsigned)n * per_q + 3) / 4;
  const unsigned nb = gridDim.x, xcd = blockIdx.x & 7u, nq = nb >> 3, nr = nb & 7u;
  const unsigned tile = xcd * nq + (xcd < nr ? xcd : nr) + (blockIdx.x >> 3);
  const int chunk = (int)(tile / groups);
  // wave -> (spin of P, Q, equal / opposite spin of Q, column group)
  // (uniform over the wavefront, so that everything derived from it and the
  // item's indices stays in scalar registers)
  unsigned w = (tile % groups) * 4 + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // a wavefront past the last one repeats it for the block's barriers
  const bool idle = w >= 2u * (unsigned)n * per_q;
  if (idle) w = 2u * (unsigned)n * per_q - 1u;
  const int sp = (int)(w / (per_q * (unsigned)n));
  w -= (unsigned)sp * per_q * (unsigned)n;
  const int q = (int)(w / per_q);
  w -= (unsigned)q * per_q;
  const bool q_same = (int)w < gs;  // Q has the spin of P
  const int col0 = (q_same ? (int)w : (int)w - gs) * kCols;
  const int ncol = q_same ? np : nn;
  const int Q = 2 * q + (q_same ? sp : 1 - sp);
  // chunk -> kind and item range
  const bool same = chunk < chunks_same;  // p, r, s: r and s have P's spin
  const int ch = same ? chunk : chunk - chunks_same;
  const int nch = same ? chunks_same : chunks_opp, items = same ? np : nn;
  const int i0 = (int)((long long)items * ch / nch), i1 = (int)((long long)items * (ch + 1) / nch);
  const int rs = same ? sp : 1 - sp;  // spin of r and s
  // Gamma block of the rows and columns: by the number of alphas among p, r, Q
  const int nalpha = (sp == 0) + (rs == 0) + ((Q & 1) == 0);
  const int blk = 3 - nalpha;
  const double* __restrict__ g3 = V.g3 + d.off[blk];
  const u64 ld = d.ld[blk];
  const unsigned zero_col = d.len[blk];
  // column offsets in bytes and sign bits
  unsigned off[KS][kRdmNT], neg[KS][kRdmNT];
  int S[kRdmNT], R[kRdmNT], outcol[kRdmNT];
#pragma unroll
  for (int t = 0; t < kRdmNT; ++t) {
    const int col = col0 + 16 * t + li;
    S[t] = R[t] = -1;
    outcol[t] = col;
    if (col < ncol) {
      if (q_same) {
        int x, y;
        rdm_pair_split((unsigned)col, &x, &y);
        S[t] = 2 * x + sp;
        R[t] = 2 * y + sp;
      } else {
        // the orbital that is alone of its spin in the column's triple runs
        // fastest: 16 lanes then read neighbouring elements for every s
        const bool fast_alpha = rs == 1;
        S[t] = 2 * (fast_alpha ? col % n : col / n);
        R[t] = 2 * (fast_alpha ? col / n : col % n) + 1;
        outcol[t] = (R[t] >> 1) * n + (S[t] >> 1);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int s = 4 * ks + lk;
      unsigned o = zero_col, sb = 0;
      if (s < n && S[t] >= 0) {
        int b, sg;
        unsigned id;
        if (rdm_sorted(d, 2 * s + rs, S[t], R[t], &b, &id, &sg)) {
          o = id;
          sb = (unsigned)sg << 31;
        }
      }
      off[ks][t] = o * 8u;
      neg[ks][t] = sb;
    }
  }
  // the d_sQ term: lanes of k step Q / 4 with s = Q read the two-body row
  const bool has_delta = rs == (Q & 1);
  const int dks = has_delta ? q >> 2 : -1;
  const bool dlane = has_delta && lk == (q & 3);
  const int cls2 = sp == rs ? (sp ? 2 : 0) : 1;
  const double* __restrict__ g2 = V.g2 + (cls2 == 0 ? 0 : (cls2 == 1 ? (u64)np * np : (u64)np * np + (u64)nn * nn));
  const int ld2 = cls2 == 1 ? nn : np;
  unsigned c2[kRdmNT];   // byte offset in the two-body row
  double w2[kRdmNT];     // +-1/2 in the lanes with s = Q, else 0
#pragma unroll
  for (int t = 0; t < kRdmNT; ++t) {
    c2[t] = 0;
    w2[t] = 0.0;
    if (dlane && S[t] >= 0) {
      int c, sg;
      unsigned id;
      rdm_sorted2(d, S[t], R[t], &c, &id, &sg);
      c2[t] = id * 8u;
      w2[t] = sg ? -0.5 : 0.5;
    }
  }
  f64x4 acc[MT][kRdmNT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < kRdmNT; ++t) acc[m][t] = f64x4{0.0, 0.0, 0.0, 0.0};
  const double* __restrict__ va = vtab + (u64)(same ? 0 : np) * kPer;
  // loads at a uniform base and a 32-bit lane offset: no address arithmetic in
  // the vector unit, which the FP64 matrix instructions keep busy
  auto at = [](const double* base, unsigned bytes) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + bytes);
  };
  // Item -> row of Gamma (the zero row if {p, r, Q} holds an index twice), sign
  // of the term, and the row and factor of the d_sQ term.
  auto item = [&](int p, int r, const double*& grow, unsigned& flip, const double*& drow, double& dfac) {
    const int so_p = 2 * p + sp, so_r = 2 * r + rs;
    // {p, r, Q} in the order a_Q a_r a_p, and the minus sign of the term
    int b, sg;
    unsigned row;
    const bool ok = rdm_sorted(d, Q, so_r, so_p, &b, &row, &sg);
    grow = g3 + (u64)(ok ? row : d.len[blk]) * ld;
    flip = (ok && !sg) ? 0x80000000u : 0u;
    int c, s2;
    unsigned row2 = 0;
    const bool ok2 = rdm_sorted2(d, so_r, so_p, &c, &row2, &s2);
    drow = g2 + (u64)(ok2 ? row2 : 0u) * ld2;
    dfac = ok2 ? (s2 ? -1.0 : 1.0) : 0.0;
  };
  // The B operands of the next item are loaded into each register as soon as
  // this item's value has been used, one whole item ahead of their use.  The A
  // operand is the same in the block's wavefronts: one copy in LDS, the next
  // item's behind it (each wavefront with its own loads of it read as much for A
  // as for B: 2.62 ms at 26 orbitals, 2.19 with the copy; matrix time 1.25).
  double bv[KS][kRdmNT], dv[kRdmNT];
  constexpr int kStage = (kPer + 255) / 256;
  auto stage_load = [&](const double* base, double (&v)[kStage]) {
#pragma unroll
    for (int j = 0; j < kStage; ++j) {
      const unsigned e = threadIdx.x + 256u * j;
      v[j] = at(base, (e < (unsigned)kPer ? e : (unsigned)kPer - 1u) * 8u);
    }
  };
  auto stage_store = [&](double* to, const double (&v)[kStage]) {
#pragma unroll
    for (int j = 0; j < kStage; ++j)
      if (threadIdx.x + 256u * j < (unsigned)kPer) to[threadIdx.x + 256u * j] = v[j];
  };
  const double *grow, *drow;
  unsigned flip;
  double dfac;
  int p = 0, r = 0;  // of the item loaded last
  if (same) {
    r = 1;
    while ((r + 1) * r / 2 <= i0) ++r;
    p = i0 - r * (r - 1) / 2;
  } else {
    p = i0 / n;
    r = i0 - p * n;
  }
  if (i0 < i1) {
    item(p, r, grow, flip, drow, dfac);
#pragma unroll
    for (int t = 0; t < kRdmNT; ++t) dv[t] = has_delta ? at(drow, c2[t]) : 0.0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int t = 0; t < kRdmNT; ++t) bv[ks][t] = at(grow, off[ks][t]);
    }
    double v[kStage];
    stage_load(va + (u64)i0 * kPer, v);
    stage_store(s_a[0], v);
  }
  lds_barrier();
  for (int it = i0; it < i1; ++it) {
    const int nx = it + 1 < i1 ? it + 1 : it;  // the last item is loaded again, unused
    if (nx != it) {
      if (same) {
        if (++p == r) {
          ++r;
          p = 0;
        }
      } else if (++r == n) {
        ++p;
        r = 0;
      }
    }
    // loaded ahead like the other operands and not touched before its use:
    // loads return in order, so a wait for it here would wait for all of them
    double dn[kRdmNT], fac_n;
    unsigned fn;
    item(p, r, grow, fn, drow, fac_n);
#pragma unroll
    for (int t = 0; t < kRdmNT; ++t) dn[t] = 0.0;
    if (has_delta) {  // uniform
#pragma unroll
      for (int t = 0; t < kRdmNT; ++t) dn[t] = at(drow, c2[t]);
    }
    double va_nx[kStage];
    stage_load(va + (u64)nx * kPer, va_nx);
    const double* a_now = s_a[(it - i0) & 1];
    double a[MT], a_nx[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = a_now[lane + m * KS * 64];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      double x[kRdmNT];
#pragma unroll
      for (int m = 0; m < MT; ++m) a_nx[m] = ks + 1 < KS ? a_now[lane + (m * KS + ks + 1) * 64] : 0.0;
#pragma unroll
      for (int t = 0; t < kRdmNT; ++t) {
        x[t] = __hiloint2double((int)((unsigned)__double2hiint(bv[ks][t]) ^ (neg[ks][t] ^ flip)),
                                __double2loint(bv[ks][t]));
        bv[ks][t] = at(grow, off[ks][t]);
      }
      if (ks == dks) {  // a branch (the asm keeps it one): one k step in KS, half of the waves
#pragma unroll
        for (int t = 0; t < kRdmNT; ++t) {
          asm volatile("" : "+v"(x[t]));
          x[t] += (w2[t] * dfac) * dv[t];
        }
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int t = 0; t < kRdmNT; ++t) acc[m][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], x[t], acc[m][t], 0, 0, 0);
        a[m] = a_nx[m];
      }
      // keeps the loads in this k step: moved behind the last product they
      // would be waited for at once
      __builtin_amdgcn_sched_barrier(0);
    }
    flip = fn;
    dfac = fac_n;
#pragma unroll
    for (int t = 0; t < kRdmNT; ++t) dv[t] = dn[t];
    // every wavefront is past the item whose copy this one takes the place of
    stage_store(s_a[(it - i0 + 1) & 1], va_nx);
    lds_barrier();
  }
  if (idle) return;
  // element i of lane l is row 4 i + l / 16, column l % 16 of the tile
  double* __restrict__ out = part + (u64)chunk * part_stride + rdm_g_offset(d, sp, q_same, q);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < kRdmNT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int P = 16 * m + 4 * i + lk;
        if (P < n && S[t] >= 0) out[(u64)P * ncol + outcol[t]] = acc[m][t][i];
      }
}

// out[t] = sum over the chunks of part[chunk][t], in order (out may be
// part itself).
__global__ void __launch_bounds__(256)
k_rdm_sum(double* part, u64 stride, int chunks, u64 len) {
  const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= len) return;
  double v = 0.0;
  for (int c = 0; c < chunks; ++c) v += part[(u64)c * stride + t];
  part[t] = v;
}

// ---------------------------------------------------------------- singles
// B(P; Q) for P, Q of one spin, one block each (blockIdx.x = (spin, P, Q)).
// Reads the full integral tensor, whose last index runs along the threads.
__global__ void __launch_bounds__(256)
k_rdm_singles(RdmView V, const double* __restrict__ h, const double* __restrict__ eri, double inv1,
              double* __restrict__ bs) {
  __shared__ double red[256];
  const int n = V.d.n;
  const int sp = (int)blockIdx.x / (n * n), P = ((int)blockIdx.x / n) % n, q = (int)blockIdx.x % n;
  const int Q = 2 * q + sp;
  const u64 np = V.d.np, nn = (u64)n * n;
  double acc = 0.0;
  // one thread per (r, s) of either spin, all p; h enters through the one-body
  // matrix, the partial trace r = s of the two-body one
  for (int t = threadIdx.x; t < 2 * n * n; t += 256) {
    const int s2 = t / (n * n), s = (t / n) % n, r = t % n;
    int ck, sk;
    unsigned ik;
    if (!rdm_sorted2(V.d, 2 * s + s2, Q, &ck, &ik, &sk)) continue;
    const u64 ldk = ck == 1 ? nn : np;
    // the two-body blocks are symmetric: the row of the ket, bra columns
    const double* __restrict__ row = V.g2 + (ck == 0 ? 0 : (ck == 1 ? np * np : np * np + nn * nn)) + (u64)ik * ldk;
    const double hw = r == s ? inv1 : 0.0;
    const bool same = s2 == sp;
#pragma unroll 4
    for (int p = 0; p < n; ++p) {
      // a_r a_p in canonical order
      const unsigned lo = (unsigned)(p < r ? p : r), hi = (unsigned)(p < r ? r : p);
      const unsigned ib = same ? rdm_c2(hi) + lo : (unsigned)(sp ? r * n + p : p * n + r);
      const bool sb = same ? r > p : sp == 0;
      const bool ok = !(same && p == r);
      const double v = row[ok ? ib : 0u] * (eri[((u64)(p * n + P) * n + s) * n + r] + hw * h[p * n + P]);
      acc += ok ? ((sb != (sk != 0)) ? -v : v) : 0.0;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) bs[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------- finish
// G(P; Q; S, R) from the summed products (annihilators in this order).
__device__ inline double rdm_g_value(const RdmDims& d, const double* __restrict__ g, int P, int Q, int S, int R) {
  const int sp = P & 1;
  const bool q_same = (Q & 1) == sp;
  double sg = 1.0;
  int col, ncol;
  if (q_same) {
    if (S > R) {
      const int t = S;
      S = R;
      R = t;
      sg = -1.0;
    }
    col = (int)rdm_c2((unsigned)(R >> 1)) + (S >> 1);
    ncol = (int)d.np;
  } else {
    if (S & 1) {
      const int t = S;
      S = R;
      R = t;
      sg = -1.0;
    }
    col = (R >> 1) * d.n + (S >> 1);
    ncol = d.n * d.n;
  }
  return sg * g[rdm_g_offset(d, sp, q_same, Q >> 1) + (u64)(P >> 1) * ncol + col];
}

__global__ void __launch_bounds__(256)
k_rdm_finish(RdmDims d, const double* __restrict__ g, const double* __restrict__ bs, const OpDesc* __restrict__ ops,
             const int* __restrict__ subset, long long count, const double* __restrict__ norm2,
             double* __restrict__ out) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const OpDesc op = ops[subset ? subset[t] : t];
  double v;
  if (op.R < 0) {
    const int sp = op.P & 1, n = d.n, p = op.P >> 1, q = op.Q >> 1;
    v = bs[(sp * n + p) * n + q] - bs[(sp * n + q) * n + p];
  } else {
    v = rdm_g_value(d, g, op.P, op.Q, op.S, op.R) - rdm_g_value(d, g, op.Q, op.P, op.S, op.R) -
        rdm_g_value(d, g, op.R, op.S, op.Q, op.P) + rdm_g_value(d, g, op.S, op.R, op.Q, op.P);
  }
  out[t] = (2.0 / norm2[0]) * v;
}

// ---------------------------------------------------------------- host
size_t rdm_gamma_elems(int n) {
  const RdmDims d = rdm_dims(n);
  size_t t = 0;
  for (int b = 0; b < 4; ++b) t += (size_t)(d.len[b] + 1) * d.ld[b];
  return t;
}

size_t rdm_two_elems(int n) {
  const RdmDims d = rdm_dims(n);
  return 2 * (size_t)d.np * d.np + (size_t)n * n * n * n;
}

static int rdm_ks(int n) { return (n + 3) / 4; }

size_t rdm_vtab_elems(int n) {
  const RdmDims d = rdm_dims(n);
  const int ks = rdm_ks(n), mt = ks > 4 ? 2 : 1;
  return ((size_t)d.np + (size_t)n * n) * mt * ks * 64;
}

// Chunks of the (p, r) items: about 80 items each at 26 orbitals, so that the
// 1,716 (spin, Q, column group) wavefronts become 20,592, and never more
// chunks than items.
void rdm_chunks(int n, int* same, int* opp) {
  const RdmDims d = rdm_dims(n);
  *same = std::max(1, std::min<int>((int)d.np, 4));
  *opp = std::max(1, std::min<int>(n * n, 8));
}

size_t rdm_part_elems(int n) {
  int a, b;
  rdm_chunks(n, &a, &b);
  return rdm_g_elems(rdm_dims(n)) * (size_t)(a + b);
}

hipError_t launch_rdm_emit(const DeviceState& st, u64 n, int ne, RdmFmt fm, int nbatch, int batch, u64 smask,
                           u64* recs, u64 cap, u64* cursor, int grid, hipStream_t stream) {
  if (ne < 3 || ne > kRdmMaxElectrons || (nbatch > 1 && smask)) return hipErrorInvalidValue;
  const unsigned ntri = (unsigned)(ne * (ne - 1) * (ne - 2) / 6);
  if (nbatch > 1)
    hipLaunchKernelGGL(k_rdm_emit_class, dim3(grid), dim3(kRdmEmitBlock), ntri * sizeof(unsigned), stream, st.keys,
                       st.amps, n, ne, ntri, fm, nbatch, batch, recs, cap, cursor, &st.ctr->flags);
  else
    hipLaunchKernelGGL(k_rdm_emit, dim3(grid), dim3(kRdmEmitBlock), ntri * sizeof(unsigned), stream, st.keys, st.amps,
                       n, ne, ntri, fm, smask, recs, cap, cursor, &st.ctr->flags);
  return hipGetLastError();
}

hipError_t launch_rdm_count(const u64* recs, u64 R, int sort_bits, double* partial, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_rdm_count, dim3(grid), dim3(256), 0, stream, recs, R, sort_bits, partial);
  return hipGetLastError();
}

hipError_t launch_rdm_pairs(const DeviceState& st, u64 n, int n_spatial, int ne, RdmFmt fm, int sort_bits,
                            const u64* recs, u64 R, double* g3, int grid, hipStream_t stream) {
  if (R == 0) return hipSuccess;
  const unsigned ntri = (unsigned)(ne * (ne - 1) * (ne - 2) / 6);
  const RdmView V{rdm_dims(n_spatial), g3, nullptr};
  hipLaunchKernelGGL(k_rdm_pairs, dim3(grid), dim3(kRdmPairBlock), ntri * sizeof(unsigned), stream, recs, R, fm, sort_bits, ne, ntri,
                     st.keys, st.amps, n, V);
  return hipGetLastError();
}

size_t rdm_member_bytes() { return sizeof(RdmMember); }
int rdm_row_bits() { return kRdmRowBits; }

hipError_t launch_rdm_members(const DeviceState& st, u64 n, int n_spatial, int ne, RdmFmt fm, int sort_bits,
                              const u64* recs, u64 R, void* mem, u64* list, u64* cursor, int grid,
                              hipStream_t stream) {
  const unsigned ntri = (unsigned)(ne * (ne - 1) * (ne - 2) / 6);
  hipError_t e = launch_fill_u32(cursor, 0u, 4, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rdm_members, dim3(grid), dim3(kRdmMemBlock), ntri * sizeof(unsigned), stream, recs, R, fm,
                     sort_bits, ne, ntri, st.keys, st.amps, n, rdm_dims(n_spatial), (RdmMember*)mem, list, cursor);
  return hipGetLastError();
}

// list sorted by row; row_end: 2^16 words.
hipError_t launch_rdm_rows(int n_spatial, const u64* list, u64 Q, unsigned* row_end, const void* mem, u64 R, double* g3,
                           hipStream_t stream) {
  if (Q == 0) return hipSuccess;
  if (Q >= (1ULL << 32)) return hipErrorInvalidValue;
  const RdmView V{rdm_dims(n_spatial), g3, nullptr};
  const unsigned width = std::max(V.d.len[0], V.d.len[1]);
  if (width > (1u << 14)) return hipErrorInvalidValue;
  const int bytes = (int)(width * sizeof(double));
  hipError_t e = hipFuncSetAttribute((const void*)k_rdm_rows, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rdm_row_ends, dim3((unsigned)std::min<u64>((Q + 255) / 256, 4096)), dim3(256), 0, stream, list, Q,
                     row_end);
  const u64 even = (Q + 4095) / 4096;  // sixteen blocks a CU
  const unsigned chunk = (unsigned)std::min<u64>(kRdmRowChunkMax, std::max<u64>(kRdmRowChunkMin, even));
  const unsigned blocks = (unsigned)((Q + chunk - 1) / chunk);
  hipLaunchKernelGGL(k_rdm_rows, dim3(blocks), dim3(kRdmRowBlock), (size_t)bytes, stream, list, Q, row_end,
                     (const RdmMember*)mem, R, width, chunk, V);
  return hipGetLastError();
}

hipError_t launch_rdm_diag(const DeviceState& st, u64 n, int n_spatial, double* g3, int grid, hipStream_t stream) {
  const RdmView V{rdm_dims(n_spatial), g3, nullptr};
  unsigned slices = 0;
  for (int b = 0; b < 4; ++b) slices += rdm_diag_slices(V.d.len[b]);
  if (slices == 0) return hipSuccess;
  hipLaunchKernelGGL(k_rdm_diag, dim3(grid, slices), dim3(kRdmDiagBlock), 0, stream, st.keys, st.amps, n, V);
  return hipGetLastError();
}

hipError_t launch_rdm_clear(int n_spatial, double* g3, hipStream_t stream) {
  const RdmView V{rdm_dims(n_spatial), g3, nullptr};
  hipLaunchKernelGGL(k_rdm_clear, dim3(2048, 4), dim3(256), 0, stream, V);
  return hipGetLastError();
}

template <int KS>
static void contract_ks(const RdmView& V, const double* vtab, int a, int b, double* part, u64 stride, unsigned blocks,
                        hipStream_t stream) {
  hipLaunchKernelGGL(k_rdm_contract<KS>, dim3(blocks * (unsigned)(a + b)), dim3(256), 0, stream, V, vtab, a, b, part,
                     stride);
}

// Two-body matrix, integrals, contraction and the asked gradients; g3 complete.
hipError_t launch_rdm_gradients(const Ints& I, const double* eri, int na, int nb, double* g3, double* g2, double* vtab, double* part, double* bs,
                                const OpDesc* ops, const int* subset, long long count, const double* norm2,
                                double* out, hipStream_t stream) {
  const int n = I.n, ne = na + nb;
  if (n < 1 || n > 32 || ne < 3) return hipErrorInvalidValue;
  const RdmView V{rdm_dims(n), g3, g2};
  const u64 vt = rdm_vtab_elems(n);
  // the spin whose electrons beside the pair are traced out: beta if it has any
  const int beside[3][2] = {{na - 2, nb}, {na - 1, nb - 1}, {na, nb - 2}};
  RdmTrace tr;
  for (int cls = 0; cls < 3; ++cls) {
    tr.spin[cls] = beside[cls][1] >= 1 ? 1 : 0;
    // a class without electrons for its pair has a zero matrix
    tr.inv[cls] = 1.0 / std::max(1, beside[cls][tr.spin[cls]]);
  }
  unsigned mt_tiles = 0;
  for (int b = 0; b < 4; ++b) {
    const unsigned nt = (V.d.len[b] + 31) / 32;
    mt_tiles = std::max(mt_tiles, nt * (nt + 1) / 2);
  }
  if (mt_tiles)
    hipLaunchKernelGGL(k_rdm_mirror, dim3(mt_tiles, 4), dim3(256), 0, stream, V);
  const unsigned pairs2 = V.d.np, mixed2 = (unsigned)(n * n);
  hipLaunchKernelGGL(k_rdm_two, dim3(2 * pairs2 + mixed2, (std::max(pairs2, mixed2) + 255) / 256), dim3(256), 0, stream,
                     V, tr, g2);
  const int ks = rdm_ks(n), mt = ks > 4 ? 2 : 1;
  hipLaunchKernelGGL(k_rdm_vtab, dim3((unsigned)((vt + 255) / 256)), dim3(256), 0, stream, I, V.d, mt, ks,
                     1.0 / (ne - 1.5), vtab);
  int a, b;
  rdm_chunks(n, &a, &b);
  const u64 stride = rdm_g_elems(V.d);
  const unsigned cols = 16 * kRdmNT, np = V.d.np, nn = (unsigned)(n * n);
  const unsigned waves = 2u * (unsigned)n * ((np + cols - 1) / cols + (nn + cols - 1) / cols);
  const unsigned blocks = (waves + 3) / 4;
  switch (ks) {
    case 1: contract_ks<1>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 2: contract_ks<2>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 3: contract_ks<3>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 4: contract_ks<4>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 5: contract_ks<5>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 6: contract_ks<6>(V, vtab, a, b, part, stride, blocks, stream); break;
    case 7: contract_ks<7>(V, vtab, a, b, part, stride, blocks, stream); break;
    default: contract_ks<8>(V, vtab, a, b, part, stride, blocks, stream); break;
  }
  hipLaunchKernelGGL(k_rdm_sum, dim3((unsigned)((stride + 255) / 256)), dim3(256), 0, stream, part, stride, a + b,
                     stride);
  hipLaunchKernelGGL(k_rdm_singles, dim3((unsigned)(2 * n * n)), dim3(256), 0, stream, V, I.h, eri,
                     1.0 / (ne - 1), bs);
  hipLaunchKernelGGL(k_rdm_finish, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, V.d, part, bs, ops,
                     subset, count, norm2, out);
  return hipGetLastError();
}

}  // namespace swcs
