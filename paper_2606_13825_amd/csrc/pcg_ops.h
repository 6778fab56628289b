// Building blocks of the CG kernels (per instance, cooperative and team
// forms): workgroup sums, CSR row passes, the fused dense sub-block product
// and the epilogue of a solve.  Internal linkage.
#pragma once

#include "cosmo_internal.h"
#include "wave_ops.h"

namespace cosmo {
namespace {

constexpr int NRESTART = 4;          // restarts from a float64 residual, at most
constexpr double ROUND_DROP2 = 1e-4;  // a restarted round lowers its residual by 1e-2 (squared here)
constexpr double STALL2 = 0.25;       // a true residual that fell by less than 2x ends the refinement

template <typename T> __device__ inline T sub_sum(T v, int L) {
  for (int off = L >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Deterministic workgroup sum of two values (red holds 2 NTH / 64 entries).
template <int NTH, typename T> __device__ inline void wg_sum2(T &a, T &b, T *red) {
  a = sub_sum(a, 64);
  b = sub_sum(b, 64);
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  __syncthreads();
  if (l == 0) {
    red[w] = a;
    red[NTH / 64 + w] = b;
  }
  __syncthreads();
  T ta = 0, tb = 0;
  for (int i = 0; i < NTH / 64; ++i) {
    ta += red[i];
    tb += red[NTH / 64 + i];
  }
  a = ta;
  b = tb;
}

// ---- CSR row passes ------------------------------------------------------------
//
// Rows rows[r0..r1) of one length class, handled by row groups of L lanes:
// group g of a pass takes row r0 + g + j nsub (j = 0, 1, ...).  Sums are
// accumulated in AT; each row's sum goes to emit(row, sum) on its first lane.
// active(row) skips rows (of instances that are done).

// Short rows (at most 4 nonzeros, one lane each): four rows per lane per
// pass, all entries read with clamped indices and masks so the whole gather is
// in flight at once.
template <typename AT, typename CT, typename T, typename VIN, typename Act, typename F>
__device__ inline void short_rows(const int32_t *__restrict__ rows, const RowSpan *__restrict__ span, int64_t first,
                                  int64_t r1, int64_t stride, const CT *__restrict__ col,
                                  const T *__restrict__ val, VIN vin, Act active, F emit) {
  for (int64_t base = first; base < r1; base += 4 * stride) {
    int32_t rw[4];
    int64_t k0[4], nk[4];
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t ri = base + u * stride;
      ok[u] = ri < r1;
      rw[u] = ok[u] ? rows[ri] : 0;
      const RowSpan sp = ok[u] ? span[ri] : RowSpan{0, 0};
      k0[u] = sp.kb;
      nk[u] = sp.k1 - sp.kb;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ok[u] = ok[u] && active(rw[u]);
      if (!ok[u]) nk[u] = 0;
    }
    AT acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc[u] = 0;
      if (nk[u] > 0) {
        // indices clamped to the row's last entry; surplus terms masked
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t k = k0[u] + (q < nk[u] ? q : nk[u] - 1);
          const AT prod = (AT)val[k] * (AT)vin[col[k]];
          acc[u] += q < nk[u] ? prod : (AT)0;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ok[u]) emit(rw[u], acc[u]);
  }
}

// Pieces of a row: VE = 16 / sizeof(T) values and VE column indices.
template <typename T> struct alignas(16) ValPiece {
  T v[16 / sizeof(T)];
};
template <typename CT, int N> struct alignas(sizeof(CT) * N) ColPiece {
  CT c[N];
};

// L lanes per row.  The row's entries are read in 16-byte pieces (the CSR
// arrays are 16-byte aligned): entries before its first aligned piece and
// after its last full piece one per lane, the full pieces U per lane per
// pass (the surplus clamped and masked), so that 2 U 16-byte loads and U VE
// gathers are in flight per lane.  The next row's id and entry range are
// loaded while the current row is summed, so the index loads are off the
// critical path.  gsub / nsub: this thread's row group and the number of row
// groups of the pass.
template <int L, typename AT, int U = 2, typename CT, typename T, typename VIN, typename Act, typename F>
__device__ inline void row_pass(const int32_t *__restrict__ rows, const RowSpan *__restrict__ span, int64_t r0,
                                int64_t r1, int64_t gsub, int64_t nsub, const CT *__restrict__ col,
                                const T *__restrict__ val, VIN vin, Act active, F emit) {
  if constexpr (L == 1) {
    short_rows<AT>(rows, span, r0 + gsub, r1, nsub, col, val, vin, active, emit);
  } else {
    constexpr int VE = 16 / sizeof(T);
    static_assert(L >= VE - 1, "a lane for each entry before the first whole piece");
    using VP = ValPiece<T>;
    using CP = ColPiece<CT, VE>;
    const int lane = threadIdx.x % L;
    int64_t ri = r0 + gsub;
    int32_t nrow = 0;
    RowSpan nsp{0, 0};
    if (ri < r1) {
      nrow = rows[ri];
      nsp = span[ri];
    }
    for (int64_t base = r0; base < r1; base += nsub, ri += nsub) {
      const int32_t row = nrow;
      const RowSpan sp = nsp;
      const bool in = ri < r1;
      if (ri + nsub < r1) {
        nrow = rows[ri + nsub];
        nsp = span[ri + nsub];
      }
      bool ok = false;
      AT a0 = 0, a1 = 0;
      if (in) {
        ok = active(row);
        if (ok) {
          const int64_t kb = sp.kb, k1 = sp.k1;
          int64_t ka = (kb + VE - 1) / VE * VE;
          if (ka > k1) ka = k1;
          const int64_t np = (k1 - ka) / VE, kt = ka + np * VE;
          if (lane < ka - kb) a0 += (AT)val[kb + lane] * (AT)vin[col[kb + lane]];
          if (lane < k1 - kt) a1 += (AT)val[kt + lane] * (AT)vin[col[kt + lane]];
          const VP *vp = reinterpret_cast<const VP *>(val + ka);
          const CP *cp = reinterpret_cast<const CP *>(col + ka);
          for (int64_t q = lane; q < np; q += U * L) {
            VP vv[U];
            CP cc[U];
            bool has[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              has[u] = q + u * L < np;
              const int64_t qu = has[u] ? q + u * L : q;
              vv[u] = vp[qu];
              cc[u] = cp[qu];
            }
            AT gv[U][VE];   // every gather of the pass before the first use
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int e = 0; e < VE; ++e) gv[u][e] = (AT)vin[cc[u].c[e]];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int e = 0; e < VE; ++e) {
                const AT pr = (AT)vv[u].v[e] * gv[u][e];
                if (u % 2 == 0) a0 += has[u] ? pr : (AT)0;
                else a1 += has[u] ? pr : (AT)0;
              }
          }
        }
      }
      const AT acc = sub_sum(a0 + a1, L);   // every lane of the row group takes part
      if (ok && lane == 0) emit(row, acc);
    }
  }
}

// All three length classes of A (cls_off = View::instA) or A' (instAt) over
// the rows of instances [b0, b1): per-instance passes use b1 = b0 + 1, grid
// passes b0 = 0, b1 = B.
template <int NTH, bool GRID, typename AT, typename T, typename VIN, typename Act, typename F>
__device__ inline void class_passes(const int32_t *rows, const RowSpan *span, const int64_t *cls_off, int64_t B1,
                                    int b0, int b1, const int32_t *col, const T *val, VIN vin, Act active, F emit) {
  auto sub = [&](int L, int64_t &g, int64_t &n) {
    if (GRID) {
      g = (int64_t)blockIdx.x * (NTH / L) + threadIdx.x / L;
      n = (int64_t)gridDim.x * (NTH / L);
    } else {
      g = threadIdx.x / L;
      n = NTH / L;
    }
  };
  int64_t g, n;
  sub(1, g, n);
  row_pass<1, AT>(rows, span, cls_off[b0], cls_off[b1], g, n, col, val, vin, active, emit);
  sub(8, g, n);
  row_pass<8, AT>(rows, span, cls_off[B1 + b0], cls_off[B1 + b1], g, n, col, val, vin, active, emit);
  sub(64, g, n);
  row_pass<64, AT>(rows, span, cls_off[2 * B1 + b0], cls_off[2 * B1 + b1], g, n, col, val, vin, active, emit);
}

// ---- dense sub-blocks inside one instance's workgroup ----------------------------
//
// Rows of A covered by a dense placement hold only their CSR part in t after
// the row passes.  Per row r of each dense block G of instance b, one wave
// forms d = G_r . vin, turns every placement's row i = row0_p + r of t into
// rho_hat_i (t_i + scale_p d), and adds w_r G_r, w_r = sum_p scale_p t_i, to
// its partial of G'w -- so G is read once per operator application.  The
// waves' partials are added in wave order into ec (the column passes add
// ec to the CSR part of A' t).  MP: 16-byte pieces of a row per lane.
//
// Rows [rb, re) of the block (a slice of it, or all of it); vin(c): the
// vector's entry of the block's column c; row((A p)_i, new t_i) is called once
// per row of A, on one lane.
struct NoTerm {
  template <typename AT> __device__ void operator()(AT, AT) const {}
};
template <int NTH, int MP, typename AT, typename TG, typename T, typename TT, typename VIN, typename Row = NoTerm>
__device__ inline void dense_block_fused(const DenseDesc &d, int rb, int re, const T *__restrict__ rho_hat, VIN vin,
                                         TT *__restrict__ t, AT *__restrict__ lds, double *__restrict__ ec,
                                         Row row = NoTerm{}) {
  constexpr int VE = 16 / sizeof(TG);
  constexpr int NW = NTH / 64;
  // rows in flight per wave: four while a row spans at most two pieces per
  // lane, two for wider rows (register budget); the block read is bound by
  // the bytes each CU keeps in flight
  constexpr int U = MP <= 2 ? 4 : 2;
  static_assert(COSMO_DENSE_MAX_PLACEMENTS == 4, "one lane per (row, placement): four placements per row");
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int npieces = (d.cols + VE - 1) / VE;
  AT xv[MP][VE], acc[MP][VE];
#pragma unroll
  for (int q = 0; q < MP; ++q)
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const int c = (lane + 64 * q) * VE + e;
      xv[q][e] = c < d.cols ? (AT)vin(c) : (AT)0;
      acc[q][e] = (AT)0;
    }
  // Lane 4u + p of a pass handles placement p of the pass's row u: it loads
  // that entry of t and rho_hat (two vector loads per pass instead of one
  // per row and placement), forms and stores the new entry, and the four
  // lanes of the row sum their scale * entry into the row's weight.  Lanes
  // of placements the block does not have take scale 0 and store nothing.
  const int lu = (lane >> 2) & (U - 1), lp = lane & 3;
  const bool lplace = lp < d.nplace;
  int64_t lrow0 = d.row0[0];
  AT lsc = (AT)d.scale[0];
#pragma unroll
  for (int q = 1; q < COSMO_DENSE_MAX_PLACEMENTS; ++q)
    if (lp == q && lplace) {
      lrow0 = d.row0[q];
      lsc = (AT)d.scale[q];
    }
  if (!lplace) lsc = (AT)0;
  // (the block's address comes out of memory: said to be global memory, its
  // loads do not also wait for the LDS)
  typedef TG Piece __attribute__((ext_vector_type(VE)));
  typedef const __attribute__((address_space(1))) Piece *GlobalPieces;
  GlobalPieces G = (GlobalPieces)d.val;
  const int64_t ldp = d.ld / VE;
  for (int r0 = rb + wave; r0 < re; r0 += U * NW) {
    Piece g[U][MP];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(r0 + u * NW, re - 1);   // clamped; surplus rows change nothing
#pragma unroll
      for (int q = 0; q < MP; ++q) {
        // lanes past the row's end re-read its last piece (their terms are
        // masked below), so every load of the pass is issued unconditionally
        const int pc = min(lane + 64 * q, npieces - 1);
        g[u][q] = G[(int64_t)r * ldp + pc];
      }
    }
    const int lr = r0 + lu * NW;
    const int lrc = min(lr, re - 1);
    const AT tl = (AT)t[lrow0 + lrc], rl = (AT)rho_hat[lrow0 + lrc];
    // the U rows' dot products, summed over the wave together
    AT dots[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      dots[u] = 0;
#pragma unroll
      for (int q = 0; q < MP; ++q)
#pragma unroll
        for (int e = 0; e < VE; ++e) dots[u] += (AT)g[u][q][e] * xv[q][e];   // xv is 0 past the row's end
    }
    wave_sums<U>(dots);
    AT dl = dots[0];
#pragma unroll
    for (int u = 1; u < U; ++u) dl = lu == u ? dots[u] : dl;
    const AT ap = tl + lsc * dl, ti = rl * ap;
    if (lane < 4 * U && lplace && lr < re) {
      t[lrow0 + lr] = (TT)ti;
      row(ap, ti);
    }
    AT wl = lsc * ti;
    wl += __shfl_xor(wl, 1, 64);
    wl += __shfl_xor(wl, 2, 64);   // lane 4u: row u's weight
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u * NW < re) {
        const AT w = read_lane(wl, 4 * u);
#pragma unroll
        for (int q = 0; q < MP; ++q)
#pragma unroll
          for (int e = 0; e < VE; ++e) acc[q][e] += w * (AT)g[u][q][e];   // entries past cols are never read
      }
    }
  }
  // partials of the waves, added in wave order
#pragma unroll
  for (int q = 0; q < MP; ++q)
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const int c = (lane + 64 * q) * VE + e;
      if (c < d.cols) lds[wave * d.cols + c] = acc[q][e];
    }
  __syncthreads();
  for (int c = threadIdx.x; c < d.cols; c += NTH) {
    AT sum = 0;
    for (int w = 0; w < NW; ++w) sum += lds[w * d.cols + c];
    ec[d.coff + c] = (double)sum;
  }
  __syncthreads();   // the partials are read before the next block overwrites them
}

// Epilogue shared by both forms, over instance b's columns.
template <int NTH, typename T>
__device__ inline void finish(const View<T> &v, int b, bool fail, int it, int passes, double rrt, double thr, T *x,
                              const T *alpha_k, const T *xold, T *xnew, const T *gx_in, T *gx_out, int32_t mode,
                              cosmo_stats *stats) {
  const int64_t n0 = v.n_off[b], n1 = v.n_off[b + 1];
  if (fail)   // a non-finite system marks its solution, never a finite warm start
    for (int64_t j = n0 + threadIdx.x; j < n1; j += NTH) x[j] = (T)NAN;
  const T al = alpha_k ? alpha_k[b] : (T)1;
  if (mode == 0) {
    if (xnew)
      for (int64_t j = n0 + threadIdx.x; j < n1; j += NTH) xnew[j] = al * x[j] + ((T)1 - al) * xold[j];
  } else {
    for (int64_t j = n0 + threadIdx.x; j < n1; j += NTH) gx_out[j] = ((T)1 - al) * gx_in[j] + v.sigma * x[j];
  }
  if (stats && threadIdx.x == 0) {
    atomicMax(&stats[b].cg_iters_max, it);
    atomicAdd(&stats[b].cg_iters_total, it);
    atomicAdd(&stats[b].cg_passes_total, passes);
    if (!(rrt <= thr)) atomicAdd(&stats[b].cg_not_converged, 1);
  }
}

}  // namespace
}  // namespace cosmo
