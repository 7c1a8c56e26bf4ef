// Index and sign rules of the three-body density matrix (k_rdm.hip), shared by
// its kernels and host code.
//
// Annihilator triples and pairs are kept in one order: alphas ascending, then
// betas ascending.  Triples of one spin pattern form one block of Gamma:
//   0  three alphas       C(c,3) + C(b,2) + a           (a < b < c)
//   1  two alphas, a beta pair(a, b) n + beta
//   2  an alpha, two betas pair(b, c) n + alpha
//   3  three betas        as 0
// with np = C(n, 2) and pair(a, b) = C(b, 2) + a.  A block of len triples is a
// (len + 1) x ld matrix, ld > len: its last row and the columns from len on
// stay zero and stand for triples with an index twice.
#pragma once

#include "swcs_internal.h"

namespace swcs {

constexpr int kRdmMaxElectrons = 32;
constexpr unsigned kRdmMaxTriples = 4960;  // C(32, 3)

__host__ __device__ inline unsigned rdm_c2(unsigned m) { return (m * m - m) >> 1; }
__host__ __device__ inline unsigned rdm_c3(unsigned m) { return m < 3 ? 0u : m * (m - 1) * (m - 2) / 6; }

struct RdmDims {
  int n;
  unsigned np;
  unsigned len[4], ld[4];
  u64 off[4];
};

__host__ __device__ inline RdmDims rdm_dims(int n) {
  RdmDims d;
  d.n = n;
  d.np = rdm_c2((unsigned)n);
  d.len[0] = d.len[3] = rdm_c3((unsigned)n);
  d.len[1] = d.len[2] = d.np * (unsigned)n;
  u64 at = 0;
  for (int b = 0; b < 4; ++b) {
    d.ld[b] = (d.len[b] + 8u) & ~7u;
    d.off[b] = at;
    at += (u64)(d.len[b] + 1) * d.ld[b];
  }
  return d;
}

// Record: hash of the subset in the low hb bits, the triple's code in bt bits,
// the entry index above.
struct RdmFmt {
  int hb, bt;
};
__host__ __device__ inline u64 rdm_record(const RdmFmt& f, u64 d, unsigned t, u64 h) {
  return (d << (f.hb + f.bt)) | ((u64)t << f.hb) | h;
}
__host__ __device__ inline u64 rdm_record_entry(const RdmFmt& f, u64 r) { return r >> (f.hb + f.bt); }
__host__ __device__ inline unsigned rdm_record_triple(const RdmFmt& f, u64 r) {
  return (unsigned)((r >> f.hb) & ((1ULL << f.bt) - 1ULL));
}

// Orbitals a < b of pair index i.
__host__ __device__ inline void rdm_pair_split(unsigned i, int* a, int* b) {
  unsigned y = (unsigned)((1.0f + sqrtf(1.0f + 8.0f * (float)i)) * 0.5f);
  while (y * (y - 1) / 2 > i) --y;
  while ((y + 1) * y / 2 <= i) ++y;
  *b = (int)y;
  *a = (int)(i - y * (y - 1) / 2);
}

// Spin-orbitals of pair index i of spin class cls (0 aa, 1 ab, 2 bb).
__host__ __device__ inline void rdm_pair_orbitals(const RdmDims& d, int cls, unsigned i, int* x, int* y) {
  if (cls == 1) {
    *x = 2 * (int)(i / (unsigned)d.n);
    *y = 2 * (int)(i % (unsigned)d.n) + 1;
    return;
  }
  const int s = cls == 2 ? 1 : 0;
  int a, b;
  rdm_pair_split(i, &a, &b);
  *x = 2 * a + s;
  *y = 2 * b + s;
}

// a_x a_y in canonical order: spin class, index, and sign (1 = minus); false
// when x = y.
__host__ __device__ inline bool rdm_sorted2(const RdmDims& d, int x, int y, int* cls, unsigned* id, int* sg) {
  if (x == y) return false;
  // order by (spin, orbital)
  const int kx = ((x & 1) << 6) | (x >> 1), ky = ((y & 1) << 6) | (y >> 1);
  *sg = kx > ky;
  const int lo = kx > ky ? y : x, hi = kx > ky ? x : y;
  const unsigned a = (unsigned)(lo >> 1), b = (unsigned)(hi >> 1);
  if ((lo & 1) != (hi & 1)) {
    *cls = 1;
    *id = a * (unsigned)d.n + b;
  } else {
    *cls = (lo & 1) ? 2 : 0;
    *id = rdm_c2(b) + a;
  }
  return true;
}

// a_x a_y a_z in canonical order: block, index, sign; false when two agree.
__host__ __device__ inline bool rdm_sorted(const RdmDims& d, int x, int y, int z, int* blk, unsigned* id, int* sg) {
  int k0 = ((x & 1) << 6) | (x >> 1), k1 = ((y & 1) << 6) | (y >> 1), k2 = ((z & 1) << 6) | (z >> 1);
  if (k0 == k1 || k0 == k2 || k1 == k2) return false;
  int s = 0, t;
  if (k0 > k1) { t = k0; k0 = k1; k1 = t; s ^= 1; }
  if (k1 > k2) { t = k1; k1 = k2; k2 = t; s ^= 1; }
  if (k0 > k1) { t = k0; k0 = k1; k1 = t; s ^= 1; }
  *sg = s;
  const unsigned a = (unsigned)(k0 & 63), b = (unsigned)(k1 & 63), c = (unsigned)(k2 & 63);
  const int nb = (k0 >> 6) + (k1 >> 6) + (k2 >> 6);
  *blk = nb;
  if (nb == 0 || nb == 3) *id = rdm_c3(c) + rdm_c2(b) + a;
  else if (nb == 1) *id = (rdm_c2(b) + a) * (unsigned)d.n + c;
  else *id = (rdm_c2(c) + b) * (unsigned)d.n + a;
  return true;
}

// C_A |D> for the occupied spin-orbitals x < y < z of D: block, index and sign
// (1 = minus) of the canonical product, the rightmost annihilator acting first
// (betas from the highest, then alphas from the highest).
__host__ __device__ inline void rdm_canonical(const RdmDims& d, u64 D, int x, int y, int z, int* blk, unsigned* id,
                                              int* sg) {
#if defined(__HIP_DEVICE_COMPILE__)
  int s = __popcll(D & ((1ULL << x) - 1ULL)) + __popcll(D & ((1ULL << y) - 1ULL)) +
          __popcll(D & ((1ULL << z) - 1ULL));
#else
  int s = __builtin_popcountll(D & ((1ULL << x) - 1ULL)) + __builtin_popcountll(D & ((1ULL << y) - 1ULL)) +
          __builtin_popcountll(D & ((1ULL << z) - 1ULL));
#endif
  // a beta below an alpha leaves first and lowers the alpha's count by one
  s += ((x & 1) && !(y & 1)) + ((x & 1) && !(z & 1)) + ((y & 1) && !(z & 1));
  int order;
  (void)rdm_sorted(d, x, y, z, blk, id, &order);
  *sg = s & 1;
}

// Position of G(.; Q; .) for P of spin sp: per spin, the n matrices [P][pair]
// of Q with P's spin, then the n matrices [P][beta n + alpha] of Q with the
// other one.
__host__ __device__ inline u64 rdm_g_offset(const RdmDims& d, int sp, bool q_same, int q) {
  const u64 nn = (u64)d.n * d.n, per_s = (u64)d.n * d.np, per_o = (u64)d.n * nn;
  const u64 spin = (u64)d.n * (per_s + per_o);
  return (u64)sp * spin + (q_same ? (u64)q * per_s : (u64)d.n * per_s + (u64)q * per_o);
}
__host__ __device__ inline u64 rdm_g_elems(const RdmDims& d) {
  return 2 * (u64)d.n * ((u64)d.n * d.np + (u64)d.n * d.n * d.n);
}

}  // namespace swcs
