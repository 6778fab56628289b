// One-sided (Hestenes) Jacobi sweeps over a block held in LDS, by one
// workgroup.  Internal linkage: included by the eigensolver.
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
// so the NB pairs' rotations cost one evaluation.  The angle is computed in
// float32 (any t gives an orthogonal rotation; an inexact one leaves a little
// more for the next sweep); 1 / (1 + t^2) is formed to working precision.
//
// Blocks stand in a row of positions; a sweep is one odd-even transposition
// pass: the blocks at positions (0,1), (2,3), .. are rotated and change
// places, then (1,2), (3,4), .. -- after as many phases as blocks every pair
// has met once and the row is reversed.  A block moves on in one direction,
// so per phase a group keeps one block in registers and passes the other to
// its neighbour through LDS: one block written, one read and one barrier for
// NB^2 rotations.  The block's own storage is the exchange buffer (left half:
// Y blocks moving left, right half: X blocks moving right).
//
// What bounds it: the issue of 3 multiply-adds per element pair on the few
// waves one block occupies (a wave issues a vector instruction every four
// cycles), about as many instructions again for the reduction, the rotation
// and the broadcasts, and their latency.  Measured per sweep in float64:
// 51 us at order 100 (NB = 4, G = 16: one wave per SIMD), 24 us at 64 and
// 10 us at 32 (NB = 2).  Reading and writing both columns of every pair in
// LDS for each rotation (the circle schedule, which this replaces) took
// 1542 us for the projection of an order-100 float64 block, this 690 us.
// Two-column blocks at order 100 (twice the exchanges, two waves per SIMD)
// took 64 us per sweep.
#pragma once

#include "cosmo_internal.h"

namespace cosmo {
namespace {

// Cross-lane moves inside rows of 16 lanes (DPP).
template <int CTRL, int BANKS = 0xF> __device__ __forceinline__ float dpp_mov(float x, float old = 0.f) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, 0xF, BANKS, BANKS == 0xF));
}
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
template <int G, int NB, typename T> __device__ __forceinline__ T group_sums(const T (&v)[NB]) {
  static_assert((G == 8 || G == 16) && (NB == 2 || NB == 4), "group of 8 or 16 lanes, 2 or 4 values");
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
  T s;
  if constexpr (NB == 2) {
    s = (b0 ? v[1] : v[0]) + dpp_mov<DPP_XOR1>(b0 ? v[0] : v[1]);
    s += dpp_mov<DPP_XOR2>(s);
  } else {
    const T lo = (b0 ? v[1] : v[0]) + dpp_mov<DPP_XOR1>(b0 ? v[0] : v[1]);
    const T hi = (b0 ? v[3] : v[2]) + dpp_mov<DPP_XOR1>(b0 ? v[2] : v[3]);
    s = (b1 ? hi : lo) + dpp_mov<DPP_XOR2>(b1 ? lo : hi);
  }
  // lane i ^ 4: quads 0 and 2 of a row read upwards, 1 and 3 downwards
  s += dpp_mov<DPP_SHR4, 0xA>(s, dpp_mov<DPP_SHL4, 0x5>(s));
  if constexpr (G == 16) s += dpp_mov<DPP_ROR8>(s);
  return s;
}

// The value held by the lanes of index Q, in every lane of their quad.
template <int NB, int Q, typename T> __device__ __forceinline__ T from_lane(T x) {
  if constexpr (NB == 4) return dpp_mov<quad_perm(Q, Q, Q, Q)>(x);
  else return dpp_mov<quad_perm(Q, Q, 2 + Q, 2 + Q)>(x);
}
template <int NB, typename T> __device__ __forceinline__ T lane_value(T x, int q) {   // q: known after unrolling
  return q == 0 ? from_lane<NB, 0>(x) : q == 1 ? from_lane<NB, 1>(x) : q == 2 ? from_lane<NB, 2 % NB>(x)
                                                                                : from_lane<NB, 3 % NB>(x);
}
// Lane q receives lane (q + 1) % NB's value.
template <int NB, typename T> __device__ __forceinline__ T next_lane(T x) {
  return dpp_mov<NB == 4 ? quad_perm(1, 2, 3, 0) : DPP_XOR1>(x);
}

// 1 / x to working precision: the hardware's float32 reciprocal, or two
// Newton steps on its float64 one.
__device__ __forceinline__ float full_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double full_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// What a sweep has seen: the largest squared cosine of a column pair and the
// largest squared tangent of a rotation.
struct SweepMax {
  float cos2, tan2;
};

// Rotates NB disjoint pairs (a[q], b[q]); al, da, be, db: squared norms and D
// of pair q's columns in the lanes of index q.
template <int G, int NB, int E, typename C>
__device__ __forceinline__ void rotate_pairs(C *const (&a)[NB], C *const (&b)[NB], C &al, C &da, C &be, C &db, float tol2,
                                    SweepMax &mx) {
  C dots[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) dots[q] = a[q][0] * b[q][0];
#pragma unroll
  for (int e = 1; e < E; ++e)
#pragma unroll
    for (int q = 0; q < NB; ++q) dots[q] = fma(a[q][e], b[q][e], dots[q]);
  const C g = group_sums<G, NB>(dots);
  const C P = da * db, Pg = P * g;
  const float gf = (float)g, g2 = gf * (float)Pg;   // (a'b)^2
  const float ab = (float)al * (float)be;
  const bool rot = g2 > tol2 * ab;
  if constexpr (E * NB >= 20) {
    if (__ballot(rot) == 0) return;   // nothing to rotate in this wave
  }
  const float d = (float)(be - al);
  const float r2 = fmaf(4.f, g2, d * d);
  float tau = 2.f * gf * __builtin_amdgcn_rcpf(fmaf(r2, __builtin_amdgcn_rsqf(r2), fabsf(d)));
  tau = rot ? copysignf(1.f, d) * tau : 0.f;   // t / (d_a d_b); 0 where r2 = 0
  const C cx = (C)tau * db, cy = (C)tau * da;
  const C t2 = cx * cy, sec2 = (C)1 + t2, k = (C)tau * Pg;
  const C cs2 = rot ? full_rcp(sec2) : (C)1;
  const C cz = cy * cs2;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const C u = lane_value<NB>(cx, q);
#pragma unroll
    for (int e = 0; e < E; ++e) a[q][e] = fma(-u, b[q][e], a[q][e]);
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const C u = lane_value<NB>(cz, q);
#pragma unroll
    for (int e = 0; e < E; ++e) b[q][e] = fma(u, a[q][e], b[q][e]);
  }
  al -= k;
  be += k;
  da *= cs2;
  db *= sec2;
  mx.cos2 = fmaxf(mx.cos2, g2 * __builtin_amdgcn_rcpf(ab));   // (a zero column's NaN is dropped)
  mx.tan2 = fmaxf(mx.tan2, (float)t2);
}

template <typename C, int NB, int E> struct JacobiRegs {
  C x[NB][E], y[NB][E];
  C al, da;   // column X_q (q: lane index): squared norm, D
  C be, db;   // column Y_q
};

// The cross pairs of blocks X and Y: step S pairs (x_q, y_(q+S)).
template <int G, int NB, int E, int S, typename C>
__device__ __forceinline__ void cross_step(JacobiRegs<C, NB, E> &R, float tol2, SweepMax &mx) {
  C *a[NB], *b[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    a[q] = R.x[q];
    b[q] = R.y[(q + S) % NB];
  }
  rotate_pairs<G, NB, E>(a, b, R.al, R.da, R.be, R.db, tol2, mx);
  R.be = next_lane<NB>(R.be);
  R.db = next_lane<NB>(R.db);
}
template <int G, int NB, int E, typename C>
__device__ __forceinline__ void cross_pairs(JacobiRegs<C, NB, E> &R, float tol2, SweepMax &mx) {
  cross_step<G, NB, E, 0>(R, tol2, mx);
  cross_step<G, NB, E, 1>(R, tol2, mx);
  if constexpr (NB == 4) {
    cross_step<G, NB, E, 2>(R, tol2, mx);
    cross_step<G, NB, E, 3>(R, tol2, mx);
  }
}

// The pairs (I0, J0), (I1, J1) of X and of Y at once (NB = 4); lanes 0 and 1
// of a quad take X's scalars, lanes 2 and 3 Y's.
template <int G, int E, int I0, int J0, int I1, int J1, typename C>
__device__ __forceinline__ void inside_step4(JacobiRegs<C, 4, E> &R, float tol2, SweepMax &mx) {
  const int m = threadIdx.x & 3;
  const bool hi = m >= 2;
  auto gather_a = [&](C fx, C fy) {
    const C u = dpp_mov<quad_perm(I0, I1, I0, I1)>(fx), w = dpp_mov<quad_perm(I0, I1, I0, I1)>(fy);
    return hi ? w : u;
  };
  auto gather_b = [&](C fx, C fy) {
    const C u = dpp_mov<quad_perm(J0, J1, J0, J1)>(fx), w = dpp_mov<quad_perm(J0, J1, J0, J1)>(fy);
    return hi ? w : u;
  };
  C al = gather_a(R.al, R.be), da = gather_a(R.da, R.db), be = gather_b(R.al, R.be), db = gather_b(R.da, R.db);
  C *a[4] = {R.x[I0], R.x[I1], R.y[I0], R.y[I1]};
  C *b[4] = {R.x[J0], R.x[J1], R.y[J0], R.y[J1]};
  rotate_pairs<G, 4, E>(a, b, al, da, be, db, tol2, mx);
  // column m is the first or second member of pair 0 or 1
  constexpr int P0 = 0, P1 = (1 == I0 || 1 == J0) ? 0 : 1, P2 = (2 == I0 || 2 == J0) ? 0 : 1,
                P3 = (3 == I0 || 3 == J0) ? 0 : 1;
  const bool second = m == J0 || m == J1;
  auto scatter = [&](C fa, C fb, C &ox, C &oy) {
    const C xa = dpp_mov<quad_perm(P0, P1, P2, P3)>(fa), xb = dpp_mov<quad_perm(P0, P1, P2, P3)>(fb);
    const C ya = dpp_mov<quad_perm(2 + P0, 2 + P1, 2 + P2, 2 + P3)>(fa);
    const C yb = dpp_mov<quad_perm(2 + P0, 2 + P1, 2 + P2, 2 + P3)>(fb);
    ox = second ? xb : xa;
    oy = second ? yb : ya;
  };
  scatter(al, be, R.al, R.be);
  scatter(da, db, R.da, R.db);
}

// The pairs inside the blocks, once per sweep.
template <int G, int NB, int E, typename C>
__device__ __forceinline__ void inside_pairs(JacobiRegs<C, NB, E> &R, float tol2, SweepMax &mx) {
  if constexpr (NB == 4) {
    inside_step4<G, E, 0, 1, 2, 3>(R, tol2, mx);
    inside_step4<G, E, 0, 2, 1, 3>(R, tol2, mx);
    inside_step4<G, E, 0, 3, 1, 2>(R, tol2, mx);
  } else {
    // even lanes: (x0, x1), odd lanes: (y0, y1)
    const bool odd = threadIdx.x & 1;
    const C al2 = dpp_mov<DPP_XOR1>(R.al), da2 = dpp_mov<DPP_XOR1>(R.da);
    const C be2 = dpp_mov<DPP_XOR1>(R.be), db2 = dpp_mov<DPP_XOR1>(R.db);
    C al = odd ? be2 : R.al, da = odd ? db2 : R.da, be = odd ? R.be : al2, db = odd ? R.db : da2;
    C *a[2] = {R.x[0], R.y[0]}, *b[2] = {R.x[1], R.y[1]};
    rotate_pairs<G, 2, E>(a, b, al, da, be, db, tol2, mx);
    const C pa = dpp_mov<DPP_XOR1>(al), pda = dpp_mov<DPP_XOR1>(da), pb = dpp_mov<DPP_XOR1>(be), pdb = dpp_mov<DPP_XOR1>(db);
    R.al = odd ? pb : al;
    R.da = odd ? pdb : da;
    R.be = odd ? be : pa;
    R.db = odd ? db : pda;
  }
}

// A block whose scale became small or large is rescaled by a power of two (exact).
template <int NB, int E, typename C> __device__ __forceinline__ void rescale(C (&col)[NB][E], C &D) {
  const bool low = D < (C)0.0009765625, high = D > (C)1024;   // 2^-10, 2^10
  if (__ballot(low || high) == 0) return;
  const C f = low ? (C)0.03125 : high ? (C)32 : (C)1;
  D = low ? D * (C)1024 : high ? D * (C)0.0009765625 : D;
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const C fq = lane_value<NB>(f, q);
#pragma unroll
    for (int e = 0; e < E; ++e) col[q][e] *= fq;
  }
}

// When a solve's sweeps end.  tol2: pairs with a squared cosine below it are
// not rotated.  A sweep that rotated nothing ends them; so does one after
// which the couplings that its rotations can have left behind, at most
// p max|tan| max|cos|, are below stop (they mix a rotated pair's remainder
// with another pair's coupling).  At most max_sweeps sweeps, or, with
// coarse2 > 0, max_sweeps until the largest squared cosine is below coarse2
// and then up to max_fine more.
struct SweepRule {
  float tol2, stop, coarse2;
  int max_sweeps, max_fine;
};
struct SweepCount {
  int sweeps, fine;
  bool converged;
};

// Sweeps over the order-p block in W (jacobi_cols<NB>(p) columns of leading
// dimension ld, rows p .. ld - 1 and columns from p on zero; scale brings its
// column norms to order one); leaves in W the normalised columns and in lamd
// their norms times scale.  scal: 2 * jacobi_cols<NB>(p) elements (may be
// lamd), mx_s: 6 zeroed ints.  Starts and ends with a barrier.
template <int NB> __host__ __device__ constexpr int jacobi_cols(int p) { return (p + 2 * NB - 1) / (2 * NB) * (2 * NB); }

template <typename C, int G, int NB, int PE, int NCH>
__device__ __forceinline__ SweepCount jacobi_sweeps(C *W, C *scal, C scale, int p, int ld, const SweepRule &rule, double *lamd,
                                    int *mx_s) {
  constexpr int E = PE * NCH;
  typedef C V __attribute__((ext_vector_type(PE)));
  const int tid = threadIdx.x, grp = tid / G, gl = tid % G, q = tid % NB;
  const int ng = jacobi_cols<NB>(p) / (2 * NB);
  const bool act = grp < ng, first = grp == 0, last = grp == ng - 1;
  const bool busy = __builtin_amdgcn_readfirstlane(grp) < ng;   // waves past the last group only keep the barriers
  const int pe = (p + PE - 1) / PE * PE;
  const int row0 = PE * gl;
  const bool tail = row0 + PE * G * (NCH - 1) < pe;   // this lane's last piece lies inside the block
  C *bufL = W, *bufR = W + NB * ng * ld;              // ng slots of NB columns each
  C *scL = scal, *scR = scal + 2 * NB * ng;           // per slot: squared norms of its columns, then their D
  JacobiRegs<C, NB, E> R;
  auto load = [&](const C *src, C (&dst)[NB][E]) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        V t = 0;
        if (c < NCH - 1 || tail) t = *reinterpret_cast<const V *>(src + k * ld + row0 + PE * G * c);
#pragma unroll
        for (int e = 0; e < PE; ++e) dst[k][PE * c + e] = t[e];
      }
  };
  auto store = [&](C *dst, const C (&src)[NB][E]) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        if (c < NCH - 1 || tail) {
          V t;
#pragma unroll
          for (int e = 0; e < PE; ++e) t[e] = src[k][PE * c + e];
          *reinterpret_cast<V *>(dst + k * ld + row0 + PE * G * c) = t;
        }
  };
  auto set_all = [&](C (&dst)[NB][E], C f) {   // times f; f = 0 clears
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int e = 0; e < E; ++e) dst[k][e] = f == (C)0 ? (C)0 : dst[k][e] * f;
  };
  auto norms = [&](const C (&v)[NB][E]) {
    C s[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      s[k] = v[k][0] * v[k][0];
#pragma unroll
      for (int e = 1; e < E; ++e) s[k] = fma(v[k][e], v[k][e], s[k]);
    }
    return group_sums<G, NB>(s);
  };
  R.da = R.db = 1;
  R.al = R.be = 0;
  __syncthreads();
  if (act) {
    load(W + 2 * NB * grp * ld, R.x);
    load(W + (2 * NB * grp + NB) * ld, R.y);
    set_all(R.x, scale);
    set_all(R.y, scale);
  } else {
    set_all(R.x, 0);
    set_all(R.y, 0);
  }
  C *myL = bufL + NB * grp * ld, *myR = bufR + NB * grp * ld;
  __syncthreads();   // every column is in registers before the buffers are written
  SweepCount n{0, 0, p == 1};
  bool fine = false, coarse_ok = true;
  int rev = 0, total = 0;
  while (!n.converged && (fine ? n.fine < rule.max_fine : n.sweeps < rule.max_sweeps)) {
    SweepMax mx{0.f, 0.f};
    if (busy) {
      R.al = R.da * norms(R.x);
      R.be = R.db * norms(R.y);
      inside_pairs<G, NB, E>(R, rule.tol2, mx);
    }
    for (int ph = 0; ph < ng; ++ph) {
      if (busy) {
        cross_pairs<G, NB, E>(R, rule.tol2, mx);
        // the former right block moves left, to the group before
        rescale<NB, E>(R.y, R.db);
      }
      if (act) {
        store(myL, R.y);
        if (gl < NB) {
          scL[2 * NB * grp + q] = R.be;
          scL[2 * NB * grp + NB + q] = R.db;
        }
      }
      __syncthreads();
      if (act) {
        if (last) {   // the right end: no partner in this phase
          set_all(R.y, 0);
          R.be = 0;
          R.db = 1;
        } else {
          load(myL + NB * ld, R.y);
          R.be = scL[2 * NB * (grp + 1) + q];
          R.db = scL[2 * NB * (grp + 1) + NB + q];
        }
      }
      if (busy) {
        cross_pairs<G, NB, E>(R, rule.tol2, mx);
        // the former left block moves right, to the group after
        rescale<NB, E>(R.x, R.da);
      }
      if (act) {
        store(myR, R.x);
        if (gl < NB) {
          scR[2 * NB * grp + q] = R.al;
          scR[2 * NB * grp + NB + q] = R.da;
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
        const C *src = first ? bufL : myR - NB * ld;
        const C *ssc = first ? scL : scR + 2 * NB * (grp - 1);
        load(src, R.x);
        R.al = ssc[q];
        R.da = ssc[NB + q];
      }
    }
    rev ^= 1;
    // the sweep's maxima over the workgroup (non-negative floats order like their bits)
    int *slot = mx_s + 2 * (total % 3), *next = mx_s + 2 * ((total + 1) % 3);
    if (busy) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        mx.cos2 = fmaxf(mx.cos2, __shfl_xor(mx.cos2, off, 64));
        mx.tan2 = fmaxf(mx.tan2, __shfl_xor(mx.tan2, off, 64));
      }
      if (tid % 64 == 0) {
        atomicMax(&slot[0], __float_as_int(mx.cos2));
        atomicMax(&slot[1], __float_as_int(mx.tan2));
      }
    }
    if (tid == 0) next[0] = next[1] = 0;
    __syncthreads();
    const float c2 = __int_as_float(slot[0]), t2 = __int_as_float(slot[1]);
    ++total;
    if (fine) ++n.fine;
    else ++n.sweeps;
    n.converged = t2 == 0.f || (float)p * sqrtf(c2) * sqrtf(t2) <= rule.stop;
    if (!fine && rule.coarse2 > 0.f && (c2 <= rule.coarse2 || n.sweeps >= rule.max_sweeps)) {
      fine = true;
      coarse_ok = n.converged || c2 <= rule.coarse2;
    }
  }
  if (fine) n.converged = coarse_ok;
  __syncthreads();
  // normalised columns and their norms
  auto norms64 = [&](const C (&v)[NB][E]) {
    double s[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      s[k] = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) s[k] = fma((double)v[k][e], (double)v[k][e], s[k]);
    }
    return group_sums<G, NB>(s);
  };
  if (busy) {
    const double sx = norms64(R.x), sy = norms64(R.y);
    const double nx = sqrt(sx), ny = sqrt(sy);
    const double ix = sx > 0.0 ? 1.0 / nx : 0.0, iy = sy > 0.0 ? 1.0 / ny : 0.0;
    auto mul = [&](C (&v)[NB][E], double f) {
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const double fk = lane_value<NB>(f, k);
#pragma unroll
        for (int e = 0; e < E; ++e) v[k][e] = (C)((double)v[k][e] * fk);
      }
    };
    mul(R.x, ix);
    mul(R.y, iy);
    if (act) {
      // position i holds block i, or block 2 ng - 1 - i after an odd number of sweeps
      const int bx = rev ? 2 * ng - 1 - 2 * grp : 2 * grp, by = rev ? bx - 1 : bx + 1;
      store(W + NB * bx * ld, R.x);
      store(W + NB * by * ld, R.y);
      if (gl < NB) {
        if (NB * bx + q < p) lamd[NB * bx + q] = sqrt((double)R.da) * nx;
        if (NB * by + q < p) lamd[NB * by + q] = sqrt((double)R.db) * ny;
      }
    }
  }
  __syncthreads();
  return n;
}

// The sweeps with as many column pieces per lane as order p needs.
template <typename C, int G, int NB, int PE, int NCH, int NMAX>
__device__ __forceinline__ SweepCount run_sweeps(C *W, C *scal, C scale, int p, int ld, const SweepRule &rule, double *lamd,
                                        int *mx_s) {
  if constexpr (NCH < NMAX) {
    if (p > PE * G * NCH)
      return run_sweeps<C, G, NB, PE, NCH + 1, NMAX>(W, scal, scale, p, ld, rule, lamd, mx_s);
  }
  return jacobi_sweeps<C, G, NB, PE, NCH>(W, scal, scale, p, ld, rule, lamd, mx_s);
}

}  // namespace
}  // namespace cosmo
