// sigma_P of large states by spin strings.
//
// Two determinants have a nonzero Slater-Condon element only if they differ in
// at most two electrons, so their spin strings (the alpha and the beta
// occupation) differ by
//   (0, 1), (0, 2) electrons: one alpha string -- members of one alpha group;
//   (1, 0), (2, 0):           one beta string  -- members of one beta group;
//   (1, 1):                   alpha strings one excitation apart, and betas too.
// The entries are sorted once by alpha string and once by beta string, one
// record each (hole-pair grouping sorts C(N_e, 2) = 120 records per determinant
// at 16 electrons).  Within a group every pair is tested by a popcount of the
// other strings; for (1, 1) a wavefront probes a table of the strings that occur
// for the na (n - na) single excitations of its rows' string and tests the
// members of the groups it finds.  A test is four instructions and one 4-byte
// load shared by eight rows; matrix elements are formed only for the pairs that
// pass, queued in LDS so that they run on full wavefronts.
//
// 983,489 determinants of 52 spin-orbitals and 16 electrons: 161,043 alpha
// strings, 8.2e8 (1, 1) tests for 8.5e6 pairs.  Both sorts take 0.3 ms, the
// groups 0.08, the spin that leads the (1, 1) pairs 1.44 (bound by the
// dependent table probes and the tests' instructions) and the other 0.24; hole
// pairs took 0.43 to emit, 4.2 to sort and 5.95 to scan their records.
#include <algorithm>

#include "swcs_internal.h"

namespace swcs {

// Compact string of one spin of an interleaved key.
__device__ inline unsigned str_compact(u64 D, int spin) {
  u64 x = (D >> spin) & 0x5555555555555555ULL;
  x = (x | (x >> 1)) & 0x3333333333333333ULL;
  x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0FULL;
  x = (x | (x >> 4)) & 0x00FF00FF00FF00FFULL;
  x = (x | (x >> 8)) & 0x0000FFFF0000FFFFULL;
  x = (x | (x >> 16)) & 0x00000000FFFFFFFFULL;
  return (unsigned)x;
}

// One record per entry and spin: the string in the low n bits, bit n for dead
// entries (they sort behind the alive ones), the entry index from bit `shift`
// on, a whole number of the sort's 8-bit digits, so that no pass sees it.
__global__ void __launch_bounds__(256)
k_str_emit(const u64* __restrict__ keys, const double* __restrict__ amps, u64 cnt, int n, int shift,
           u64* __restrict__ ra,
           u64* __restrict__ rb) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride) {
    const u64 D = keys[i], top = (i << shift) | (is_dead(amps[i]) ? 1ULL << n : 0ULL);
    ra[i] = top | str_compact(D, 0);
    rb[i] = top | str_compact(D, 1);
  }
}

// Table slot of an occurring string: its group [lo, hi) in the sorted order.
// key = string + 1 (a string may be empty), 0 = free.
struct StrSlot {
  u64 key;
  unsigned lo, hi;
};

__device__ inline u64 str_hash(unsigned s, u64 mask) { return mix64((u64)s + 0x632be59bd9b4e019ULL) & mask; }

__device__ inline bool str_find(const StrSlot* __restrict__ tab, u64 mask, unsigned s, unsigned* lo, unsigned* hi) {
  u64 h = str_hash(s, mask);
  for (u64 probes = 0; probes <= mask; ++probes) {
    const StrSlot t = tab[h];
    if (t.key == (u64)s + 1) {
      *lo = t.lo;
      *hi = t.hi;
      return true;
    }
    if (t.key == 0) return false;
    h = (h + 1) & mask;
  }
  return false;
}

// Pairs of sampled determinants that share a string: every sampled row against
// this block's 256 columns, both spread evenly over the entries (at the limit
// of what AUTO takes, 1e7 determinants still give some 200 such pairs).  A
// block's line of out: pairs with one alpha string, with one beta string (an
// entry and itself excluded), columns alive, rows alive, pairs of one entry.
constexpr int kStrRowSample = 256;
constexpr u64 kStrColSample = 16384;
static_assert((kStrColSample + 255) / 256 <= kStrSampleBlocks, "lines of out");

__global__ void __launch_bounds__(256)
k_str_sample(const u64* __restrict__ keys, const double* __restrict__ amps, u64 cnt, unsigned rows, unsigned cols,
             unsigned* __restrict__ out) {
  __shared__ uint2 s_row[kStrRowSample];
  __shared__ unsigned s_at[kStrRowSample];
  __shared__ unsigned s_sum[5], s_n;
  if (threadIdx.x < 5) s_sum[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  for (unsigned r = threadIdx.x; r < rows; r += 256) {
    const u64 i = (u64)r * cnt / rows;
    if (is_dead(amps[i])) continue;
    const u64 D = keys[i];
    const unsigned at = atomicAdd(&s_n, 1u);
    s_row[at] = make_uint2(str_compact(D, 0), str_compact(D, 1));
    s_at[at] = (unsigned)i;
  }
  __syncthreads();
  const unsigned n = s_n, c = blockIdx.x * 256 + threadIdx.x;
  unsigned sum[4] = {0, 0, 0, 0};
  const u64 j = c < cols ? (u64)c * cnt / cols : 0;
  if (c < cols && !is_dead(amps[j])) {
    const u64 D = keys[j];
    const unsigned a = str_compact(D, 0), b = str_compact(D, 1);
    sum[2] = 1;
    for (unsigned r = 0; r < n; ++r) {
      const uint2 o = s_row[r];
      const unsigned self = s_at[r] == (unsigned)j ? 1u : 0u;
      sum[0] += (o.x == a ? 1u : 0u) - self;
      sum[1] += (o.y == b ? 1u : 0u) - self;
      sum[3] += self;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    unsigned v = sum[q];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63u) == 0) atomicAdd(&s_sum[q < 3 ? q : 4], v);
  }
  __syncthreads();
  if (threadIdx.x < 5) out[5 * blockIdx.x + threadIdx.x] = threadIdx.x == 3 ? n : s_sum[threadIdx.x];
}

// Sorted records of one spin -> keys, amplitudes and the other spin's strings
// in this order, and the table of this spin's strings (load at most 1/2; each
// string is inserted once, by the first record of its group, which finds the
// end by doubling steps and a bisection).
__global__ void __launch_bounds__(256)
k_str_groups(const u64* __restrict__ rec, u64 alive, int n, int shift, int spin, const u64* __restrict__ keys,
             const double* __restrict__ amps, u64* __restrict__ skey, double* __restrict__ sval,
             unsigned* __restrict__ oth, StrSlot* __restrict__ tab, u64 mask) {
  const u64 smask = (1ULL << n) - 1ULL;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 p = (u64)blockIdx.x * blockDim.x + threadIdx.x; p < alive; p += stride) {
    const u64 r = rec[p], i = r >> shift;
    const unsigned s = (unsigned)(r & smask);
    const u64 D = keys[i];
    skey[p] = D;
    sval[p] = amps[i];
    oth[p] = str_compact(D, 1 - spin);
    if (p > 0 && (unsigned)(rec[p - 1] & smask) == s) continue;
    u64 lo = p, hop = 1;  // rec[lo] is in the group
    while (lo + hop < alive && (unsigned)(rec[lo + hop] & smask) == s) {
      lo += hop;
      hop <<= 1;
    }
    while (hop > 1) {
      hop >>= 1;
      if (lo + hop < alive && (unsigned)(rec[lo + hop] & smask) == s) lo += hop;
    }
    u64 h = str_hash(s, mask);
    for (u64 probes = 0; probes <= mask; ++probes) {  // at most half the slots are ever taken
      if (atomicCAS((unsigned long long*)&tab[h].key, 0ULL, (unsigned long long)s + 1ULL) == 0ULL) {
        tab[h].lo = (unsigned)p;
        tab[h].hi = (unsigned)(lo + 1);
        break;
      }
      h = (h + 1) & mask;
    }
  }
}

// <X|H|D> of distinct determinants of one sector that differ in one or two
// electrons.
__device__ inline double str_element(const Ints& I, u64 X, u64 D) {
  const u64 diff = X ^ D, holes = D & diff, parts = X & diff;
  const int h0 = __ffsll((long long)holes) - 1, p0 = __ffsll((long long)parts) - 1;
  if (__popcll(diff) == 2) return single_element(I, D, h0, p0);
  return double_element(I, D, h0, 63 - __clzll((long long)holes), p0, 63 - __clzll((long long)parts));
}

constexpr int kStrBlock = 256;
constexpr int kStrWaves = kStrBlock / 64;
constexpr int kStrRows = 8;         // rows per wavefront
constexpr int kStrAdj = 257;        // 16 x 16 single excitations at most, and the group itself
constexpr int kStrQueue = 64 + 64;  // pairs waiting for their element

struct StrWave {
  unsigned lo[kStrAdj];       // start of each candidate group
  unsigned off[kStrAdj + 1];  // prefix sums of their sizes
  unsigned qj[kStrQueue];     // queued pairs: candidate position,
  unsigned char qr[kStrQueue];  // row within the wavefront
  unsigned char occ[32], vir[32];
  double sum[kStrRows];
};

// sigma of eight consecutive rows (sorted positions) per wavefront: the pairs
// within their own group, and with ADJ those with the groups one excitation
// away.  Each row is owned by one wavefront, which adds its sum to sigma.
template <bool ADJ>
__global__ void __launch_bounds__(kStrBlock)
k_str_sigma(const u64* __restrict__ rec, u64 alive, int n, int shift, int nocc, const u64* __restrict__ skey,
            const double* __restrict__ sval, const unsigned* __restrict__ oth, const StrSlot* __restrict__ tab,
            u64 mask, Ints I, double* __restrict__ sigma) {
  __shared__ StrWave s_w[kStrWaves];
  const int lane = (int)(threadIdx.x & 63u);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  StrWave& W = s_w[wave];
  const u64 smask = (1ULL << n) - 1ULL, below = (1ULL << lane) - 1ULL;
  const u64 nch = (alive + kStrRows - 1) / kStrRows;
  // all LDS use is per wavefront (wave_sync)
  for (u64 ch = (u64)blockIdx.x * kStrWaves + (u64)wave; ch < nch; ch += (u64)gridDim.x * kStrWaves) {
    const u64 row0 = ch * kStrRows;
    const int rows = (int)((alive - row0) < (u64)kStrRows ? (alive - row0) : (u64)kStrRows);
    // lane r < rows: string and other string of row r
    const u64 rr = rec[row0 + (lane < rows ? lane : 0)];
    const unsigned my_str = (unsigned)(rr & smask), my_oth = oth[row0 + (lane < rows ? lane : 0)];
    if (lane < kStrRows) W.sum[lane] = 0.0;
    unsigned nq = 0;  // queued pairs (uniform)
    auto drain = [&](unsigned take) {
      wave_sync();
      if ((unsigned)lane < take) {
        const unsigned r = W.qr[lane], j = W.qj[lane];
        atomicAdd(&W.sum[r], str_element(I, skey[j], skey[row0 + r]) * sval[j]);
      }
      wave_sync();
      // the rest moves to the front
      const unsigned left = nq - take;
      unsigned j = 0;
      unsigned char r = 0;
      if ((unsigned)lane < left) {
        j = W.qj[take + lane];
        r = W.qr[take + lane];
      }
      wave_sync();
      if ((unsigned)lane < left) {
        W.qj[lane] = j;
        W.qr[lane] = r;
      }
      nq = left;
      wave_sync();
    };
    for (int r0 = 0; r0 < rows;) {
      // run [r0, r1) of rows with one string
      const unsigned str = (unsigned)__builtin_amdgcn_readlane((int)my_str, r0);
      const u64 same = __ballot(lane < rows && my_str == str);
      const int r1 = r0 + __popcll(same);  // sorted: the run is contiguous
      unsigned nadj = 1;
      {
        unsigned lo = 0, hi = 0;
        if (lane == 0) {
          (void)str_find(tab, mask, str, &lo, &hi);
          W.lo[0] = lo;
          W.off[0] = 0;
          W.off[1] = hi - lo;
        }
      }
      if (ADJ) {
        const int nvir = n - nocc;
        if (lane < n) {
          const unsigned b = (1u << lane) - 1u;
          if ((str >> lane) & 1u) W.occ[__popc(str & b)] = (unsigned char)lane;
          else W.vir[__popc(~str & b)] = (unsigned char)lane;
        }
        wave_sync();
        for (int q0 = 0; q0 < nocc * nvir; q0 += 64) {
          const int q = q0 + lane;
          unsigned lo = 0, hi = 0;
          bool hit = false;
          if (q < nocc * nvir) {
            const int i = q / nvir, a = q - i * nvir;
            hit = str_find(tab, mask, str ^ (1u << W.occ[i]) ^ (1u << W.vir[a]), &lo, &hi);
          }
          const u64 m = __ballot(hit);
          // inclusive prefix sum of the sizes over the wavefront
          unsigned inc = hit ? hi - lo : 0u;
          for (int off = 1; off < 64; off <<= 1) {
            const unsigned v = __shfl_up(inc, off);
            if (lane >= off) inc += v;
          }
          const unsigned base = W.off[nadj];
          if (hit) {
            const unsigned k = nadj + (unsigned)__popcll(m & below);
            W.lo[k] = lo;
            W.off[k + 1] = base + inc;
          }
          nadj += (unsigned)__popcll(m);
          wave_sync();
        }
      }
      wave_sync();
      const unsigned total = W.off[nadj], own = W.off[1];
      unsigned orow[kStrRows];
#pragma unroll
      for (int r = 0; r < kStrRows; ++r) {
        const int at = r0 + r < r1 ? r0 + r : r0;
        orow[r] = (unsigned)__builtin_amdgcn_readlane((int)my_oth, at);
      }
      const int nr = r1 - r0;
      for (unsigned f0 = 0; f0 < total; f0 += 64) {
        const unsigned f = f0 + (unsigned)lane;
        unsigned j = 0, mask8 = 0;
        if (f < total) {
          unsigned k = 0;
          if (ADJ) {  // group of flat candidate f
            unsigned hi = nadj;
            while (hi - k > 1) {
              const unsigned mid = (k + hi) >> 1;
              if (W.off[mid] <= f) k = mid;
              else hi = mid;
            }
          }
          j = W.lo[k] + (f - W.off[k]);
          const unsigned o = oth[j];
          const int most = f < own ? 4 : 2;
#pragma unroll
          for (int r = 0; r < kStrRows; ++r) {
            const int pc = __popc(o ^ orow[r]);
            // 2 for a single excitation of the other string; 4 only within the group
            if (r < nr && pc >= 2 && pc <= most) mask8 |= 1u << r;
          }
        }
        while (true) {
          const u64 m = __ballot(mask8 != 0);
          if (m == 0) break;
          if (mask8) {
            const unsigned at = nq + (unsigned)__popcll(m & below);
            const int r = __ffs((int)mask8) - 1;
            mask8 &= mask8 - 1;
            W.qj[at] = j;
            W.qr[at] = (unsigned char)(r0 + r);
          }
          nq += (unsigned)__popcll(m);
          if (nq >= 64) drain(64);
        }
      }
      r0 = r1;
    }
    if (nq) drain(nq);
    if (lane < rows) sigma[rr >> shift] += W.sum[lane];
    wave_sync();
  }
}

size_t str_slot_bytes() { return sizeof(StrSlot); }

unsigned str_sample_blocks(u64 cnt) { return (unsigned)((std::min<u64>(cnt, kStrColSample) + 255) / 256); }

hipError_t launch_str_sample(const DeviceState& st, u64 cnt, unsigned* out, hipStream_t stream) {
  if (cnt == 0 || cnt >= (1ULL << 31)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_str_sample, dim3(str_sample_blocks(cnt)), dim3(256), 0, stream, st.keys, st.amps, cnt,
                     (unsigned)std::min<u64>(cnt, kStrRowSample), (unsigned)std::min<u64>(cnt, kStrColSample), out);
  return hipGetLastError();
}

hipError_t launch_str_emit(const DeviceState& st, u64 cnt, int n, int shift, u64* ra, u64* rb, int grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_str_emit, dim3(grid), dim3(256), 0, stream, st.keys, st.amps, cnt, n, shift, ra, rb);
  return hipGetLastError();
}

hipError_t launch_str_groups(const DeviceState& st, const u64* rec, u64 alive, int n, int shift, int spin, u64* skey,
                             double* sval, unsigned* oth, void* tab, u64 slots, int grid, hipStream_t stream) {
  hipError_t e = launch_fill_u32(tab, 0u, slots * sizeof(StrSlot) / 4, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_str_groups, dim3(grid), dim3(256), 0, stream, rec, alive, n, shift, spin, st.keys, st.amps, skey, sval,
                     oth, (StrSlot*)tab, slots - 1);
  return hipGetLastError();
}

hipError_t launch_str_sigma(const Ints& I, const u64* rec, u64 alive, int shift, int nocc, const u64* skey,
                            const double* sval, const unsigned* oth, const void* tab, u64 slots, bool adj,
                            double* sigma, int grid, hipStream_t stream) {
  if (nocc * (I.n - nocc) > kStrAdj - 1) return hipErrorInvalidValue;
  if (adj)
    hipLaunchKernelGGL(k_str_sigma<true>, dim3(grid), dim3(kStrBlock), 0, stream, rec, alive, I.n, shift, nocc, skey,
                       sval, oth, (const StrSlot*)tab, slots - 1, I, sigma);
  else
    hipLaunchKernelGGL(k_str_sigma<false>, dim3(grid), dim3(kStrBlock), 0, stream, rec, alive, I.n, shift, nocc, skey,
                       sval, oth, (const StrSlot*)tab, slots - 1, I, sigma);
  return hipGetLastError();
}

}  // namespace swcs
