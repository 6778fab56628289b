// One-sided (Hestenes) Jacobi sweeps over a block, by one workgroup, in
// float64.  Internal linkage: included by the eigensolver.
//
// A group of G lanes holds two blocks of NB columns (X: left, Y: right) in
// registers, their rows in pieces of PE elements spread over its lanes, and
// rotates the NB^2 cross pairs in NB steps of NB disjoint pairs.  A column is
// kept scaled, a = sqrt(D) x: a rotation by t = tan(angle) is, in place,
//   x <- x - (t d_b / d_a) y,            D_a <- D_a / (1 + t^2),
//   y <- y + (t d_a / d_b) / (1 + t^2) x, D_b <- D_b (1 + t^2)
// (d = sqrt(D)), two multiply-adds per element pair where cos and sin take
// four operations.  Squared norms are carried along (|a|^2 - t g, |b|^2 + t g
// with g = a'b) and formed afresh at every sweep, so one inner product per
// pair remains.  The scalars of pair q sit in the lanes with lane % NB == q,
// so the NB pairs' rotations cost one evaluation.  The angle, the test whether
// a pair is rotated and the measures that end the sweeps are formed in the
// data's own type (Sc; any t gives an orthogonal rotation, an inexact one
// leaves a little more for the next sweep); 1 / (1 + t^2) is formed to working
// precision.  In float32 for float64 data they would save 2.5 %.
//
// Blocks stand in a row of positions; a sweep is one odd-even transposition
// pass: the blocks at positions (0,1), (2,3), .. are rotated and change
// places, then (1,2), (3,4), .. -- after as many phases as blocks every pair
// has met once and the row is reversed.  A block moves on in one direction,
// so per phase a group keeps one block in registers and passes the other to
// its neighbour through LDS: one block written, one read and one barrier for
// NB^2 rotations.  Slot i of the exchange buffer belongs to group i after
// every second phase: a group passes its left-moving block on in its own slot
// and its right-moving one in the next group's, which it alone has read last,
// so half of the block's storage and one barrier a phase are enough.  Slots
// are interleaved lane by lane: every access of a wave is one contiguous row.
//
// Sweeps start from columns in descending order of their norms until the
// couplings are small (ORDER2): equal eigenvalues then stand side by side,
// without which the couplings of a cluster to the rest fall by a factor of a
// few per sweep only, not quadratically.  Sweeps that a float32 solve of
// order 160 takes, with and without: 10 and 14 with a quarter of the
// eigenvalues equal, 8 and 9 for a Gaussian matrix; at order 60: 8 and 12, 7
// and 8.
//
// What bounds it: the issue of 3 multiply-adds per element pair on the few
// waves one block occupies (a wave issues a vector instruction every four
// cycles), about as many instructions again for the reduction, the rotation
// and the broadcasts, and their latency; above order 128, two waves to a
// SIMD, also the LDS traffic of the exchange (320 KB a phase at order 200,
// 2500 of its 10900 cycles).  Measured per sweep: 10 us at order 30, 24 us at
// 60 (NB = 2), 56 us at 100, 73 us at 128, 150 us at 160, 230 us at 200 (NB =
// 4); with float64 angles 11, 24, 58 and 75 us, 134 us at 140.  Reading and writing both columns of every pair in LDS for each
// rotation (the circle schedule, which this replaces) took 1542 us for the
// projection of an order-100 float64 block, this 500 us; two-column blocks at
// order 100 (twice the exchanges, two waves per SIMD) 64 us per sweep.
#pragma once

#include <type_traits>

#include "cosmo_internal.h"

namespace cosmo {
namespace {

// Cross-lane moves inside rows of 16 lanes (DPP).
template <int CTRL, int BANKS = 0xF> __device__ __forceinline__ double dpp_mov(double x, double old = 0.0) {
  const long long b = __double_as_longlong(x), o = __double_as_longlong(old);
  const int lo = __builtin_amdgcn_update_dpp((int)o, (int)b, CTRL, 0xF, BANKS, BANKS == 0xF);
  const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, 0xF, BANKS, BANKS == 0xF);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E;        // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int DPP_ROR8 = 0x128;                        // rotate a row of 16 lanes by 8: lane i ^ 8
constexpr int DPP_SHL4 = 0x104, DPP_SHR4 = 0x114;      // lane i reads lane i + 4, i - 4
constexpr int quad_perm(int a, int b, int c, int d) { return a | b << 2 | c << 4 | d << 6; }

// Sums of NB values over aligned groups of G lanes: value q's total in the
// lanes with lane % NB == q.  Every step adds a lane and its partner (lane ^
// 1, 2, 4, 8), so the lanes holding one total hold the same bits: the rows of
// a column must be rotated by the same angle in all of them.
template <int G, int NB> __device__ __forceinline__ double group_sums(const double (&v)[NB]) {
  static_assert((G == 8 || G == 16) && (NB == 2 || NB == 4), "group of 8 or 16 lanes, 2 or 4 values");
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
  double s;
  if constexpr (NB == 2) {
    s = (b0 ? v[1] : v[0]) + dpp_mov<DPP_XOR1>(b0 ? v[0] : v[1]);
    s += dpp_mov<DPP_XOR2>(s);
  } else {
    const double lo = (b0 ? v[1] : v[0]) + dpp_mov<DPP_XOR1>(b0 ? v[0] : v[1]);
    const double hi = (b0 ? v[3] : v[2]) + dpp_mov<DPP_XOR1>(b0 ? v[2] : v[3]);
    s = (b1 ? hi : lo) + dpp_mov<DPP_XOR2>(b1 ? lo : hi);
  }
  // lane i ^ 4: quads 0 and 2 of a row read upwards, 1 and 3 downwards
  s += dpp_mov<DPP_SHR4, 0xA>(s, dpp_mov<DPP_SHL4, 0x5>(s));
  if constexpr (G == 16) s += dpp_mov<DPP_ROR8>(s);
  return s;
}

// The value held by the lanes of index Q, in every lane of their quad.
template <int NB, int Q> __device__ __forceinline__ double from_lane(double x) {
  if constexpr (NB == 4) return dpp_mov<quad_perm(Q, Q, Q, Q)>(x);
  else return dpp_mov<quad_perm(Q, Q, 2 + Q, 2 + Q)>(x);
}
template <int NB> __device__ __forceinline__ double lane_value(double x, int q) {   // q: known after unrolling
  return q == 0 ? from_lane<NB, 0>(x) : q == 1 ? from_lane<NB, 1>(x) : q == 2 ? from_lane<NB, 2 % NB>(x)
                                                                                : from_lane<NB, 3 % NB>(x);
}
// Lane q receives lane (q + 1) % NB's value.
template <int NB> __device__ __forceinline__ double next_lane(double x) {
  return dpp_mov<NB == 4 ? quad_perm(1, 2, 3, 0) : DPP_XOR1>(x);
}

// 1 / x to working precision: two Newton steps on the hardware's reciprocal.
__device__ __forceinline__ double full_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// 1 / x and 1 / sqrt(x) for the angles: the hardware's in float32; in float64
// one Newton step on it (47 bits or more).
__device__ __forceinline__ float angle_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double angle_rcp(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ float angle_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double angle_rsq(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// What a sweep has seen: the largest squared cosine of a column pair and the
// largest squared tangent of a rotation.
template <typename Sc> struct SweepMax {
  Sc cos2, tan2;
};
// The same over the workgroup, three sweeps in turn (non-negative numbers
// order like their bits), and whether the columns were put in another order.
template <typename Sc> struct SweepShared {
  using Bits = std::conditional_t<sizeof(Sc) == 8, unsigned long long, unsigned int>;
  Bits cos2[3], tan2[3];
  int moved;
  __device__ __forceinline__ void clear() {   // by the first threads, before a barrier
    if (threadIdx.x < 3) cos2[threadIdx.x] = tan2[threadIdx.x] = 0;
    if (threadIdx.x == 3) moved = 0;
  }
  static __device__ __forceinline__ Bits bits(Sc x) { return __builtin_bit_cast(Bits, x); }
  static __device__ __forceinline__ Sc value(Bits b) { return __builtin_bit_cast(Sc, b); }
};

// Rotates NB disjoint pairs (a[q], b[q]); al, da, be, db: squared norms and D
// of pair q's columns in the lanes of index q.
template <int G, int NB, int E, typename Sc>
__device__ __forceinline__ void rotate_pairs(double *const (&a)[NB], double *const (&b)[NB], double &al, double &da,
                                             double &be, double &db, Sc tol2, SweepMax<Sc> &mx) {
  double dots[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) dots[q] = a[q][0] * b[q][0];
#pragma unroll
  for (int e = 1; e < E; ++e)
#pragma unroll
    for (int q = 0; q < NB; ++q) dots[q] = fma(a[q][e], b[q][e], dots[q]);
  const double g = group_sums<G, NB>(dots);
  const double P = da * db, Pg = P * g;
  const Sc gs = (Sc)g, g2 = gs * (Sc)Pg;   // (a'b)^2
  const Sc ab = (Sc)al * (Sc)be;
  const bool rot = g2 > tol2 * ab;
  if constexpr (E * NB >= 20) {
    if (__ballot(rot) == 0) return;   // nothing to rotate in this wave
  }
  const Sc d = (Sc)(be - al);
  const Sc r2 = fma((Sc)4, g2, d * d);
  Sc tau = 2 * gs * angle_rcp(fma(r2, angle_rsq(r2), fabs(d)));
  tau = rot ? copysign((Sc)1, d) * tau : (Sc)0;   // t / (d_a d_b); 0 where r2 = 0
  const double cx = (double)tau * db, cy = (double)tau * da;
  const double t2 = cx * cy, sec2 = 1.0 + t2, k = (double)tau * Pg;
  const double cs2 = rot ? full_rcp(sec2) : 1.0;
  const double cz = cy * cs2;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const double u = lane_value<NB>(cx, q);
#pragma unroll
    for (int e = 0; e < E; ++e) a[q][e] = fma(-u, b[q][e], a[q][e]);
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const double u = lane_value<NB>(cz, q);
#pragma unroll
    for (int e = 0; e < E; ++e) b[q][e] = fma(u, a[q][e], b[q][e]);
  }
  al -= k;
  be += k;
  da *= cs2;
  db *= sec2;
  mx.cos2 = fmax(mx.cos2, g2 * angle_rcp(ab));   // (a zero column's NaN is dropped)
  mx.tan2 = fmax(mx.tan2, (Sc)t2);
}

template <int NB, int E> struct JacobiRegs {
  double x[NB][E], y[NB][E];
  double al, da;   // column X_q (q: lane index): squared norm, D
  double be, db;   // column Y_q
};

// The cross pairs of blocks X and Y: step S pairs (x_q, y_(q+S)).
template <int G, int NB, int E, int S, typename Sc>
__device__ __forceinline__ void cross_step(JacobiRegs<NB, E> &R, Sc tol2, SweepMax<Sc> &mx) {
  double *a[NB], *b[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    a[q] = R.x[q];
    b[q] = R.y[(q + S) % NB];
  }
  rotate_pairs<G, NB, E>(a, b, R.al, R.da, R.be, R.db, tol2, mx);
  R.be = next_lane<NB>(R.be);
  R.db = next_lane<NB>(R.db);
}
template <int G, int NB, int E, typename Sc>
__device__ __forceinline__ void cross_pairs(JacobiRegs<NB, E> &R, Sc tol2, SweepMax<Sc> &mx) {
  cross_step<G, NB, E, 0>(R, tol2, mx);
  cross_step<G, NB, E, 1>(R, tol2, mx);
  if constexpr (NB == 4) {
    cross_step<G, NB, E, 2>(R, tol2, mx);
    cross_step<G, NB, E, 3>(R, tol2, mx);
  }
}

// The pairs (I0, J0), (I1, J1) of X and of Y at once (NB = 4); lanes 0 and 1
// of a quad take X's scalars, lanes 2 and 3 Y's.
template <int G, int E, int I0, int J0, int I1, int J1, typename Sc>
__device__ __forceinline__ void inside_step4(JacobiRegs<4, E> &R, Sc tol2, SweepMax<Sc> &mx) {
  const int m = threadIdx.x & 3;
  const bool hi = m >= 2;
  auto gather_a = [&](double fx, double fy) {
    const double u = dpp_mov<quad_perm(I0, I1, I0, I1)>(fx), w = dpp_mov<quad_perm(I0, I1, I0, I1)>(fy);
    return hi ? w : u;
  };
  auto gather_b = [&](double fx, double fy) {
    const double u = dpp_mov<quad_perm(J0, J1, J0, J1)>(fx), w = dpp_mov<quad_perm(J0, J1, J0, J1)>(fy);
    return hi ? w : u;
  };
  double al = gather_a(R.al, R.be), da = gather_a(R.da, R.db), be = gather_b(R.al, R.be), db = gather_b(R.da, R.db);
  double *a[4] = {R.x[I0], R.x[I1], R.y[I0], R.y[I1]};
  double *b[4] = {R.x[J0], R.x[J1], R.y[J0], R.y[J1]};
  rotate_pairs<G, 4, E>(a, b, al, da, be, db, tol2, mx);
  // column m is the first or second member of pair 0 or 1
  constexpr int P0 = 0, P1 = (1 == I0 || 1 == J0) ? 0 : 1, P2 = (2 == I0 || 2 == J0) ? 0 : 1,
                P3 = (3 == I0 || 3 == J0) ? 0 : 1;
  const bool second = m == J0 || m == J1;
  auto scatter = [&](double fa, double fb, double &ox, double &oy) {
    const double xa = dpp_mov<quad_perm(P0, P1, P2, P3)>(fa), xb = dpp_mov<quad_perm(P0, P1, P2, P3)>(fb);
    const double ya = dpp_mov<quad_perm(2 + P0, 2 + P1, 2 + P2, 2 + P3)>(fa);
    const double yb = dpp_mov<quad_perm(2 + P0, 2 + P1, 2 + P2, 2 + P3)>(fb);
    ox = second ? xb : xa;
    oy = second ? yb : ya;
  };
  scatter(al, be, R.al, R.be);
  scatter(da, db, R.da, R.db);
}

// The pairs inside the blocks, once per sweep.
template <int G, int NB, int E, typename Sc>
__device__ __forceinline__ void inside_pairs(JacobiRegs<NB, E> &R, Sc tol2, SweepMax<Sc> &mx) {
  if constexpr (NB == 4) {
    inside_step4<G, E, 0, 1, 2, 3>(R, tol2, mx);
    inside_step4<G, E, 0, 2, 1, 3>(R, tol2, mx);
    inside_step4<G, E, 0, 3, 1, 2>(R, tol2, mx);
  } else {
    // even lanes: (x0, x1), odd lanes: (y0, y1)
    const bool odd = threadIdx.x & 1;
    const double al2 = dpp_mov<DPP_XOR1>(R.al), da2 = dpp_mov<DPP_XOR1>(R.da);
    const double be2 = dpp_mov<DPP_XOR1>(R.be), db2 = dpp_mov<DPP_XOR1>(R.db);
    double al = odd ? be2 : R.al, da = odd ? db2 : R.da, be = odd ? R.be : al2, db = odd ? R.db : da2;
    double *a[2] = {R.x[0], R.y[0]}, *b[2] = {R.x[1], R.y[1]};
    rotate_pairs<G, 2, E>(a, b, al, da, be, db, tol2, mx);
    const double pa = dpp_mov<DPP_XOR1>(al), pda = dpp_mov<DPP_XOR1>(da), pb = dpp_mov<DPP_XOR1>(be), pdb = dpp_mov<DPP_XOR1>(db);
    R.al = odd ? pb : al;
    R.da = odd ? pdb : da;
    R.be = odd ? be : pa;
    R.db = odd ? db : pda;
  }
}

// A block whose scale became small or large is rescaled by a power of two (exact).
template <int NB, int E> __device__ __forceinline__ void rescale(double (&col)[NB][E], double &D) {
  const bool low = D < 0.0009765625, high = D > 1024.0;   // 2^-10, 2^10
  if (__ballot(low || high) == 0) return;
  const double f = low ? 0.03125 : high ? 32.0 : 1.0;
  D = low ? D * 1024.0 : high ? D * 0.0009765625 : D;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const double fq = lane_value<NB>(f, q);
#pragma unroll
    for (int e = 0; e < E; ++e) col[q][e] *= fq;
  }
}

// When a solve's sweeps end.  tol2: pairs with a squared cosine below it are
// not rotated.  A sweep that rotated nothing ends them; so does one after
// which the couplings left are below stop: they are no larger than the
// largest that it met (max|cos|), nor than what its rotations can have left
// behind, p max|tan| max|cos| (they mix a rotated pair's remainder with
// another pair's coupling).  (Sweeping on until nothing is rotated took 12 %
// longer in an unroll of order-20 float64 blocks, 3 % at orders up to 100, for
// the same errors against 80-bit arithmetic.)  At most max_sweeps sweeps, or, with coarse2 > 0,
// max_sweeps until the largest squared cosine is below coarse2 and then up to
// max_fine more.
template <typename Sc> struct SweepRule {
  Sc tol2, stop, coarse2;
  int max_sweeps, max_fine;
};
struct SweepCount {
  int sweeps, fine;
  bool converged;
};

template <int NB> __host__ __device__ constexpr int jacobi_cols(int p) { return (p + 2 * NB - 1) / (2 * NB) * (2 * NB); }

// Sweeps that met no squared cosine above this leave the order as it is: the
// norms are the eigenvalues to half the digits by then.
constexpr float ORDER2 = 1e-6f;

// Exchange buffer for blocks of E pieces per lane in a class of orders up to
// PMAX: groups, lanes that hold a last piece, elements.
template <int G, int NB, int E, int PMAX> struct Exchange {
  static constexpr int NG = (G * E < PMAX ? jacobi_cols<NB>(G * E) : jacobi_cols<NB>(PMAX)) / (2 * NB);
  static constexpr int TW = PMAX - G * (E - 1) < G ? PMAX - G * (E - 1) : G;
  static constexpr int elems = NB * NG * (G * (E - 1) + TW);
};

// This thread's place: group, lane in it, whether its group holds columns.
// busy is the same in a whole wave; waves past the last group only keep the
// barriers.
template <int G, int NB> struct JacobiPlace {
  int ng, grp, gl;
  bool act, busy;
  __device__ __forceinline__ explicit JacobiPlace(int p) {
    ng = jacobi_cols<NB>(p) / (2 * NB);
    grp = threadIdx.x / G;
    gl = threadIdx.x % G;
    act = grp < ng;
    busy = __builtin_amdgcn_readfirstlane(grp) < ng;
  }
};

// First columns of the blocks that this group holds between sweeps.
struct BlockCols {
  int x, y;
};
template <int G, int NB> __device__ __forceinline__ BlockCols block_cols(const JacobiPlace<G, NB> &at, int rev) {
  const int bx = rev ? 2 * at.ng - 1 - 2 * at.grp : 2 * at.grp;
  return {NB * bx, NB * (rev ? bx - 1 : bx + 1)};
}

// Sweeps over the order-p block whose columns 2 NB g .. 2 NB g + NB - 1 are
// group g's X and the next NB its Y, zero past the block, column norms of
// order one; idle groups hold zeros.  Ends with column blocks at their
// positions, reversed after an odd number of sweeps (rev).  xb:
// Exchange::elems, sc: jacobi_cols<NB>(p) elements, rk: as many, mx_s:
// cleared; all are free to use from the first barrier on, which is the
// first thing.  put(column, row, value) and get(column, row) reach a store of
// jacobi_cols<NB>(p) columns and p rows in which columns are put in order
// (put past column p - 1 may be dropped, get gives zeros there); it may
// overlap xb.  ordered: the columns start in order (a warm start's).
template <int NT, int G, int NB, int E, int PMAX, typename Sc, typename Put, typename Get>
__device__ __forceinline__ SweepCount jacobi_sweeps(JacobiRegs<NB, E> &R, const JacobiPlace<G, NB> &at, double *xb,
                                                    double *sc, short *rk, int p, const SweepRule<Sc> &rule, bool ordered,
                                                    SweepShared<Sc> &mx_s, int &rev, Put put, Get get) {
  using X = Exchange<G, NB, E, PMAX>;
  const int tid = threadIdx.x, q = tid % NB, grp = at.grp, gl = at.gl, ng = at.ng;
  const bool act = at.act, busy = at.busy, last = grp == ng - 1;
  const bool tail = G * (E - 1) + gl < p;   // this lane's last piece lies inside the block
  double *xf = xb + tid, *xt = xb + NB * X::NG * G * (E - 1) + grp * X::TW + gl;   // whole pieces, last pieces
  auto load = [&](int shift, double (&dst)[NB][E]) {   // from this group's slot or (shift = 1) the next
#pragma unroll
    for (int k = 0; k < NB; ++k) {
#pragma unroll
      for (int c = 0; c < E - 1; ++c) dst[k][c] = xf[(k * (E - 1) + c) * X::NG * G + shift * G];
      dst[k][E - 1] = tail ? xt[k * X::NG * X::TW + shift * X::TW] : 0.0;
    }
  };
  auto store = [&](int shift, const double (&src)[NB][E]) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
#pragma unroll
      for (int c = 0; c < E - 1; ++c) xf[(k * (E - 1) + c) * X::NG * G + shift * G] = src[k][c];
      if (tail) xt[k * X::NG * X::TW + shift * X::TW] = src[k][E - 1];
    }
  };
  auto norms = [&](const double (&v)[NB][E]) {
    double s[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      s[k] = v[k][0] * v[k][0];
#pragma unroll
      for (int e = 1; e < E; ++e) s[k] = fma(v[k][e], v[k][e], s[k]);
    }
    return group_sums<G, NB>(s);
  };
  double *sc_mine = sc + 2 * NB * grp + q, *sc_next = sc_mine + 2 * NB;   // squared norms, then D
  R.da = R.db = 1;
  R.al = R.be = 0;
  __syncthreads();
  SweepCount n{0, 0, p == 1};
  bool fine = false, coarse_ok = true;
  bool order = !ordered;
  int total = 0;
  rev = 0;
  while (!n.converged && (fine ? n.fine < rule.max_fine : n.sweeps < rule.max_sweeps)) {
    SweepMax<Sc> mx{0, 0};
    if (busy) {
      R.al = R.da * norms(R.x);
      R.be = R.db * norms(R.y);
    }
    if (order) {   // the columns in descending order of their norms, in float32
      const BlockCols b = block_cols<G, NB>(at, rev);
      float *key = reinterpret_cast<float *>(sc);
      if (act && gl < NB) {
        key[b.x + q] = (float)R.al;
        key[b.y + q] = (float)R.be;
      }
      __syncthreads();
      // TPC threads to a column, each counting a part of those before it
      constexpr int TPC = NT / jacobi_cols<NB>(PMAX) >= 4 ? 4 : 2;
      static_assert(NT >= 2 * jacobi_cols<NB>(PMAX), "two threads to a column");
      const int nc = 2 * NB * ng, col = tid / TPC;
      if (col < nc) {
        const int mine = __float_as_int(key[col]);   // (non-negative floats order like their bits)
        int rank = 0;
        for (int j = 4 * (tid % TPC); j < nc; j += 4 * TPC) {
          const int4 other = *reinterpret_cast<const int4 *>(key + j);
          rank += (other.x >= mine + (j >= col)) + (other.y >= mine + (j + 1 >= col)) +
                  (other.z >= mine + (j + 2 >= col)) + (other.w >= mine + (j + 3 >= col));
        }
        rank += __builtin_amdgcn_update_dpp(0, rank, DPP_XOR1, 0xF, 0xF, true);
        if constexpr (TPC == 4) rank += __builtin_amdgcn_update_dpp(0, rank, DPP_XOR2, 0xF, 0xF, true);
        if (tid % TPC == 0) {
          rk[col] = (short)rank;
          if (rank != col) mx_s.moved = total + 1;
        }
      }
      __syncthreads();
      if (mx_s.moved == total + 1) {
        if (act) {
          auto move = [&](int col0, const double (&v)[NB][E], double D, double norm) {
            const double f = sqrt(D);
#pragma unroll
            for (int k = 0; k < NB; ++k) {
              const int to = rk[col0 + k];
              const double fk = lane_value<NB>(f, k);
#pragma unroll
              for (int c = 0; c < E; ++c)
                if (c < E - 1 || tail) put(to, G * c + gl, v[k][c] * fk);
            }
            if (gl < NB) sc[rk[col0 + q]] = norm;
          };
          move(b.x, R.x, R.da, R.al);
          move(b.y, R.y, R.db, R.be);
        }
        __syncthreads();
        if (act) {
          const int col0 = 2 * NB * grp;
          auto fetch = [&](int col, double (&v)[NB][E]) {
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
              for (int c = 0; c < E; ++c) v[k][c] = c < E - 1 || tail ? get(col + k, G * c + gl) : 0.0;
          };
          fetch(col0, R.x);
          fetch(col0 + NB, R.y);
          R.al = sc[col0 + q];
          R.be = sc[col0 + NB + q];
          R.da = R.db = 1;
        }
        rev = 0;
        __syncthreads();
      }
    }
    if (busy) inside_pairs<G, NB, E>(R, rule.tol2, mx);
    for (int ph = 0; ph < ng; ++ph) {
      if (busy) {
        cross_pairs<G, NB, E>(R, rule.tol2, mx);
        // the former right block moves left, to the group before
        rescale<NB, E>(R.y, R.db);
      }
      if (act) {
        store(0, R.y);
        if (gl < NB) {
          sc_mine[0] = R.be;
          sc_mine[NB] = R.db;
        }
      }
      __syncthreads();
      if (act) {
        if (last) {   // the right end: no partner in this phase
#pragma unroll
          for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e) R.y[k][e] = 0;
          R.be = 0;
          R.db = 1;
        } else {
          load(1, R.y);
          R.be = sc_next[0];
          R.db = sc_next[NB];
        }
      }
      if (busy) {
        cross_pairs<G, NB, E>(R, rule.tol2, mx);
        // the former left block moves right, to the group after
        rescale<NB, E>(R.x, R.da);
      }
      if (act && !last) {
        store(1, R.x);
        if (gl < NB) {
          sc_next[0] = R.al;
          sc_next[NB] = R.da;
        }
      }
      __syncthreads();
      if (act) {
        if (last) {   // it turns round at the right end
#pragma unroll
          for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e) R.y[k][e] = R.x[k][e];
          R.be = R.al;
          R.db = R.da;
        }
        // the left end takes back its own block of the phase before
        load(0, R.x);
        R.al = sc_mine[0];
        R.da = sc_mine[NB];
      }
    }
    rev ^= 1;
    // the sweep's maxima over the workgroup
    using Shared = SweepShared<Sc>;
    const int slot = total % 3, next = (total + 1) % 3;
    if (busy) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        mx.cos2 = fmax(mx.cos2, __shfl_xor(mx.cos2, off, 64));
        mx.tan2 = fmax(mx.tan2, __shfl_xor(mx.tan2, off, 64));
      }
      if (tid % 64 == 0) {
        atomicMax(&mx_s.cos2[slot], Shared::bits(mx.cos2));
        atomicMax(&mx_s.tan2[slot], Shared::bits(mx.tan2));
      }
    }
    if (tid == 0) mx_s.cos2[next] = mx_s.tan2[next] = 0;
    __syncthreads();
    const Sc c2 = Shared::value(mx_s.cos2[slot]), t2 = Shared::value(mx_s.tan2[slot]);
    order = c2 > ORDER2;
    ++total;
    if (fine) ++n.fine;
    else ++n.sweeps;
    n.converged = t2 == 0 || fmin((Sc)1, (Sc)p * sqrt(t2)) * sqrt(c2) <= rule.stop;
    if (!fine && rule.coarse2 > 0 && (c2 <= rule.coarse2 || n.sweeps >= rule.max_sweeps)) {
      fine = true;
      coarse_ok = n.converged || c2 <= rule.coarse2;
    }
  }
  if (fine) n.converged = coarse_ok;
  return n;
}

// The swept columns to unit length; their norms in the lanes of index q.
struct ColumnNorms {
  double x, y;
};
template <int G, int NB, int E> __device__ __forceinline__ ColumnNorms unit_columns(JacobiRegs<NB, E> &R) {
  auto unit = [&](double (&v)[NB][E]) {
    double s[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      s[k] = v[k][0] * v[k][0];
#pragma unroll
      for (int e = 1; e < E; ++e) s[k] = fma(v[k][e], v[k][e], s[k]);
    }
    const double n2 = group_sums<G, NB>(s), n = sqrt(n2), f = n2 > 0.0 ? 1.0 / n : 0.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const double fk = lane_value<NB>(f, k);
#pragma unroll
      for (int e = 0; e < E; ++e) v[k][e] *= fk;
    }
    return n;
  };
  const double nx = unit(R.x), ny = unit(R.y);
  return {sqrt(R.da) * nx, sqrt(R.db) * ny};
}

// The sweeps over a block that lies in LDS, with as many pieces per lane as
// order p needs: W has jacobi_cols<NB>(p) columns of leading dimension ld,
// rows p .. ld - 1 and columns from p on zero; scale brings its column norms
// to order one.  Leaves in W the normalised columns and in lamd their norms
// times scale.  W also holds the exchange buffer, lamd the moving scalars
// (jacobi_cols<NB>(p) elements).  Starts and ends with a barrier.
template <int NT, int G, int NB, int E, int EMAX, int PMAX, typename Sc>
__device__ __forceinline__ SweepCount sweep_lds(double *W, double scale, int p, int ld, const SweepRule<Sc> &rule,
                                                bool ordered, double *lamd, short *rk, SweepShared<Sc> &mx_s) {
  if constexpr (E < EMAX) {
    if (p > G * E) return sweep_lds<NT, G, NB, E + 1, EMAX, PMAX>(W, scale, p, ld, rule, ordered, lamd, rk, mx_s);
  }
  const JacobiPlace<G, NB> at(p);
  const int q = threadIdx.x % NB;
  const bool tail = G * (E - 1) + at.gl < p;
  JacobiRegs<NB, E> R;
  __syncthreads();
  auto load = [&](const double *src, double (&dst)[NB][E]) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int c = 0; c < E; ++c)
        dst[k][c] = at.act && (c < E - 1 || tail) ? src[k * ld + at.gl + G * c] * scale : 0.0;
  };
  load(W + 2 * NB * at.grp * ld, R.x);
  load(W + (2 * NB * at.grp + NB) * ld, R.y);
  int rev;
  const SweepCount n = jacobi_sweeps<NT, G, NB, E, PMAX>(
      R, at, W, lamd, rk, p, rule, ordered, mx_s, rev, [&](int col, int row, double v) { W[col * ld + row] = v; },
      [&](int col, int row) { return W[col * ld + row]; });
  __syncthreads();
  if (at.busy) {
    const ColumnNorms nm = unit_columns<G, NB, E>(R);
    if (at.act) {
      const BlockCols b = block_cols<G, NB>(at, rev);
      auto store = [&](double *dst, const double (&src)[NB][E]) {
#pragma unroll
        for (int k = 0; k < NB; ++k)
#pragma unroll
          for (int c = 0; c < E; ++c)
            if (c < E - 1 || tail) dst[k * ld + at.gl + G * c] = src[k][c];
      };
      store(W + b.x * ld, R.x);
      store(W + b.y * ld, R.y);
      if (at.gl < NB) {
        if (b.x + q < p) lamd[b.x + q] = nm.x;
        if (b.y + q < p) lamd[b.y + q] = nm.y;
      }
    }
  }
  __syncthreads();
  return n;
}

}  // namespace
}  // namespace cosmo
