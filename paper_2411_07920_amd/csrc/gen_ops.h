// Per-entry logic of one gate exp(theta G) of a spin-complemented generator whose
// rows overlap (shapes, ownership and formulas: k_generator.hip), shared by the
// multi-block kernels in HBM and the single-workgroup kernels in LDS.  A thread
// that looks up a key which another one appends in the same gate takes the same
// decision either way: it owns nothing of that component.
#pragma once

#include "gate_ops.h"

namespace swcs {

// +1: T acts on D; -1: T^dagger acts on D; 0: neither.
__device__ inline int op_acts(const OpDesc& op, u64 D) {
  if (((D & op.ann) == op.ann) && ((D & op.cre) == 0)) return 1;
  if (((D & op.cre) == op.cre) && ((D & op.ann) == 0)) return -1;
  return 0;
}

// <Y|f A|D> for the row acting on D as `act` (Y its image): +f <Y|T|D>, or
// -f <Y|T^dagger|D> = -f <D|T|Y>.
__device__ inline double op_coef(const OpDesc& op, int act, u64 D, double f) {
  const u64 Y = D ^ (op.ann | op.cre);
  return act > 0 ? f * (double)phase_of_T(op, D) : -f * (double)phase_of_T(op, Y);
}

struct GenOut {
  int napp;
  u64 key[2];
  double val[2];
  long long dalive;
  int kind;  // 0 nothing to log, 1 pair, 2 star
  PairRec pr;
  StarRec sr;
};

__device__ inline unsigned rec_index(long long j) { return j >= 0 ? (unsigned)j : 0xffffffffu; }

template <class Store>
__device__ inline void gen_pair(Store& S, double eps, u64 src, long long js, u64 dst, long long jd, int s,
                                double c, double snr, double sg, GenOut& o) {
  const double araw = js >= 0 ? S.amp((u64)js) : dead_value();
  const double braw = jd >= 0 ? S.amp((u64)jd) : dead_value();
  const bool aliveS = !is_dead(araw), aliveD = !is_dead(braw);
  if (!aliveS && !aliveD) return;
  const double sp = (double)s;
  const double a = aliveS ? araw : 0.0, b = aliveD ? braw : 0.0;
  const double ns = c * a - sp * (snr * b);
  const double nd = c * b + sp * (snr * a);
  const bool keepS = !(fabs(ns) < eps), keepD = !(fabs(nd) < eps);
  if (js >= 0) S.set_amp((u64)js, keepS ? ns : dead_value());
  else if (keepS) { o.key[o.napp] = src; o.val[o.napp++] = ns; }
  if (jd >= 0) S.set_amp((u64)jd, keepD ? nd : dead_value());
  else if (keepD) { o.key[o.napp] = dst; o.val[o.napp++] = nd; }
  o.dalive = (long long)keepS - (long long)aliveS + (long long)keepD - (long long)aliveD;
  o.kind = 1;
  o.pr.iD = rec_index(js);
  o.pr.iX = rec_index(jd);
  o.pr.s = (int)(sp * sg);  // the second row turns by s theta: its sign folded in
  o.pr.pad = 0;
  o.pr.a_old = araw;
  o.pr.b_old = braw;
}

template <class Store>
__device__ inline void gen_star(Store& S, const GenGate& g, double eps, u64 C, long long jc, u64 L1,
                                long long j1, u64 L2, long long j2, double al, double be, GenOut& o) {
  const double craw = jc >= 0 ? S.amp((u64)jc) : dead_value();
  const double r1 = j1 >= 0 ? S.amp((u64)j1) : dead_value();
  const double r2 = j2 >= 0 ? S.amp((u64)j2) : dead_value();
  const bool aC = !is_dead(craw), a1 = !is_dead(r1), a2 = !is_dead(r2);
  if (!aC && !a1 && !a2) return;
  const double xc = aC ? craw : 0.0, x1 = a1 ? r1 : 0.0, x2 = a2 ? r2 : 0.0;
  const double u = (al * x1 + be * x2) * g.rt;
  const double nc = g.c2 * xc - g.s2 * u;
  const double nu = g.s2 * xc + g.c2 * u;
  const double du = nu - u;
  const double n1 = x1 + al * (g.rt * du);
  const double n2 = x2 + be * (g.rt * du);
  const bool kC = !(fabs(nc) < eps), k1 = !(fabs(n1) < eps), k2 = !(fabs(n2) < eps);
  if (jc >= 0) S.set_amp((u64)jc, kC ? nc : dead_value());
  else if (kC) { o.key[o.napp] = C; o.val[o.napp++] = nc; }
  if (j1 >= 0) S.set_amp((u64)j1, k1 ? n1 : dead_value());
  else if (k1) { o.key[o.napp] = L1; o.val[o.napp++] = n1; }
  if (j2 >= 0) S.set_amp((u64)j2, k2 ? n2 : dead_value());
  else if (k2) { o.key[o.napp] = L2; o.val[o.napp++] = n2; }
  o.dalive = (long long)kC - (long long)aC + (long long)k1 - (long long)a1 + (long long)k2 - (long long)a2;
  o.kind = 2;
  o.sr.iC = rec_index(jc);
  o.sr.i1 = rec_index(j1);
  o.sr.i2 = rec_index(j2);
  o.sr.al = (signed char)(al > 0.0 ? 1 : -1);
  o.sr.be = (signed char)(be > 0.0 ? 1 : -1);
  o.sr.xc = craw;
  o.sr.x1 = r1;
  o.sr.x2 = r2;
}

// The update of stored entry i (see the ownership rule above).  At most one
// absent member of a pair, or two of a star, is returned for appending.
template <class Store>
__device__ inline GenOut gen_entry(Store& S, u64 i, const GenGate& g, double eps) {
  GenOut o;
  o.napp = 0;
  o.dalive = 0;
  o.kind = 0;
  const u64 D = S.key(i);
  const int a1 = op_acts(g.op1, D), a2 = op_acts(g.op2, D);
  if (!a1 && !a2) return o;
  const u64 m1 = g.op1.ann | g.op1.cre, m2 = g.op2.ann | g.op2.cre;
  if (a1 && a2) {
    const u64 L1 = D ^ m1, L2 = D ^ m2;
    gen_star(S, g, eps, D, (long long)i, L1, S.find(L1), L2, S.find(L2), op_coef(g.op1, a1, D, 1.0),
             op_coef(g.op2, a2, D, g.sg), o);
    return o;
  }
  const bool one = a1 != 0;
  const OpDesc& op = one ? g.op1 : g.op2;
  const OpDesc& ot = one ? g.op2 : g.op1;
  const u64 P = D ^ (one ? m1 : m2);
  const int ao = op_acts(ot, P);
  if (ao) {
    // D is a leaf of the star centred at P
    if (S.find(P) >= 0) return o;  // the centre owns it
    const u64 Lo = P ^ (one ? m2 : m1);
    const long long jo = S.find(Lo);
    if (jo >= 0 && Lo < D) return o;  // the other leaf owns it
    const int ar = op_acts(op, P);
    const double al = one ? op_coef(g.op1, ar, P, 1.0) : op_coef(g.op1, ao, P, 1.0);
    const double be = one ? op_coef(g.op2, ao, P, g.sg) : op_coef(g.op2, ar, P, g.sg);
    if (one) gen_star(S, g, eps, P, -1, D, (long long)i, Lo, jo, al, be, o);
    else gen_star(S, g, eps, P, -1, Lo, jo, D, (long long)i, al, be, o);
    return o;
  }
  const int a = one ? a1 : a2;
  const double snr = one ? g.sn : g.sn2;
  const double sg = one ? 1.0 : g.sg;
  if (a > 0) {
    gen_pair(S, eps, D, (long long)i, P, S.find(P), phase_of_T(op, D), g.c, snr, sg, o);
  } else {
    if (S.find(P) >= 0) return o;  // the source owns the pair
    gen_pair(S, eps, P, -1, D, (long long)i, phase_of_T(op, P), g.c, snr, sg, o);
  }
  return o;
}

}  // namespace swcs
