// PSD-cone blocks: projection by eigendecomposition (eq:psd-proj) and the
// Daleckii-Krein vector-Jacobian product (eq:psd-cotangent-dk, eq:lowner).
//
// Eigensolver: one-sided (Hestenes) cyclic Jacobi on the shifted block
// G = S + c I, c = 1.1 min(||S||_F, ||S||_inf) >= 1.1 ||S||_2, so G is
// positive definite with condition number below 21.  Column pairs of W
// (initially G) are rotated until every pair is orthogonal to the tolerance;
// then W = G V with V orthogonal and W'W diagonal, hence the normalised
// columns of W are eigenvectors of S and the column norms minus c are its
// eigenvalues.  Rotations never mix columns that are already orthogonal, so
// exactly or nearly repeated eigenvalues need no special treatment: the
// eigenvectors come out orthonormal to working precision regardless of
// gaps.  The sweeps are in jacobi_sweeps.h.
//
// Reconstruction Pi = U diag(max(lam, 0)) U' and the four products of the DK
// rule U (L o (U' T U)) U' run on the matrix cores (v_mfma 16x16x4, FP32 or
// FP64; helpers in mma_tiles.h), on 16 x 16 output tiles, one wave per tile.
#include <algorithm>
#include <type_traits>

#include "cosmo_internal.h"
#include "jacobi_sweeps.h"
#include "mma_tiles.h"

namespace cosmo {
namespace {

template <typename T> struct Unit;
template <> struct Unit<float> { static constexpr float eps = 5.96e-8f; };
template <> struct Unit<double> { static constexpr double eps = 1.11e-16; };

constexpr int MAXP = COSMO_MAX_PSD_ORDER_F32;

template <typename T, int NT> __device__ inline T wg_max(T v, T *red) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  T t = red[0];
  for (int w = 1; w < NT / 64; ++w) t = fmax(t, red[w]);
  return t;
}

// A p x p block in LDS is column-major; its columns are padded to whole pairs
// of Jacobi blocks (zero columns).  The leading dimension makes the groups of
// a wave, which work on consecutive column blocks, hit different LDS banks:
// 4 modulo 8 doubles (8 modulo 16 for two-column blocks of 16-lane groups).
// Rows p to ld - 1 are zero.  p * ld does not decrease with p.
template <int G, int NB> __host__ __device__ constexpr int eig_ld(int p) {
  return NB == 4 || G == 8 ? ((p + 3) & ~7) + 4 : ((p + 7) & ~15) + 8;
}

// Runs comp(t) for the tiles t = wave, wave + nw, ... below ntiles and stores
// each result with wr(t, result).  A wave keeps all its results in registers
// until every wave has finished computing (one barrier), so wr may overwrite
// what comp reads; HOLD must cover the tiles of one wave.  Ends with a barrier.
template <int HOLD, typename Fc, typename Fw>
__device__ inline void tile_pass(int ntiles, int wave, int nw, Fc comp, Fw wr) {
  decltype(comp(0)) hold[HOLD];
#pragma unroll
  for (int h = 0; h < HOLD; ++h) {
    const int t = wave + h * nw;
    if (t < ntiles) hold[h] = comp(t);
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < HOLD; ++h) {
    const int t = wave + h * nw;
    if (t < ntiles) wr(t, hold[h]);
  }
  __syncthreads();
}

// What the eigensolver kernels share.  mode 0: COSMO step on the block (s+
// and y+ rows); mode 1: projection only.  rscratch: per block 3 p^2 doubles,
// the first p^2 for the float64 eigenvectors; a warm start reads those of the
// previous step there (warm_read), and leaves its own (warm_write).
template <typename T> struct EigArgs {
  const PsdDesc *descs;
  int32_t max_sweeps;
  double tol;
  int32_t mode;
  const T *rho_hat, *vin, *sh, *y;
  T *s_new, *y_new, *U, *lam;
  cosmo_stats *stats;
  int32_t refine;
  double *rscratch;
  int32_t warm_read, warm_write;
};

// When the sweeps end (jacobi_sweeps.h).  tol is the column cosine that
// counts as orthogonal: the caller's, or 4 eps sqrt(p) of the data's type.  A
// refined float32 solve sweeps to a cosine of 1e-3 within max_sweeps, then on
// until what is left is below 2e-8, a third of float32's unit roundoff.
// Repeated eigenvalues, which float32 data hold as clusters 1e-8 wide, are
// what sets this: with a quarter of them equal at order 138, the couplings
// left after sweeps 7 to 11 are 1.4e-7, 1.7e-8, 3.7e-9, 1.7e-11 and 7e-15.
template <typename T> __device__ __forceinline__ SweepRule<T> sweep_rule(const EigArgs<T> &a, int p) {
  const double tol = a.tol > 0.0 ? a.tol : 4.0 * (double)Unit<T>::eps * sqrt((double)p);
  SweepRule<T> rule{(T)(tol * tol), (T)tol, 0, a.max_sweeps, 0};
  if (std::is_same<T, float>::value && a.refine > 0) {
    const float fine = (float)fmin(a.tol > 0.0 ? a.tol : 1.0, 2e-8);
    rule = SweepRule<T>{(T)fmaxf(1e-30f, 1e-4f * fine * fine), (T)fine, (T)1e-6f, a.max_sweeps, 8};
  }
  return rule;
}

// Power of two that brings the columns of a block shifted by c to order one,
// whatever c is: the sweeps judge a pair of columns by the product of their
// squared norms, which for larger or smaller columns leaves the range it is
// formed in.
__device__ __forceinline__ double column_scale(double c) {
  int e = 0;
  (void)frexp(c, &e);
  return ldexp(1.0, -e);   // c is positive and finite, the root of a float64 sum at most: |e| < 540
}

// A non-finite block yields a non-finite projection (never a clipped one).
template <typename T, int NT> __device__ inline void put_nan(const EigArgs<T> &a, const PsdDesc &d) {
  const int p = d.p;
  for (int idx = threadIdx.x; idx < p * (p + 1) / 2; idx += NT) {
    a.s_new[d.row0 + idx] = (T)NAN;
    if (a.mode == 0) a.y_new[d.row0 + idx] = (T)NAN;
  }
  if (a.lam)
    for (int i = threadIdx.x; i < p; i += NT) a.lam[d.loff + i] = (T)NAN;
  for (int e = threadIdx.x; e < p * p; e += NT) {
    if (a.U) a.U[d.uoff + e] = (T)NAN;
    if (a.warm_write) a.rscratch[3 * (size_t)d.uoff + e] = NAN;
  }
}

// svec entry (row, col), row <= col, of the projection, and the y+ row.
template <typename T> struct PutEntry {
  const EigArgs<T> &a;
  int64_t row0;
  T rh;
  __device__ __forceinline__ PutEntry(const EigArgs<T> &args, const PsdDesc &d)
      : a(args), row0(d.row0), rh(args.mode == 0 ? args.rho_hat[d.row0] : (T)0) {}
  __device__ __forceinline__ void operator()(int row, int col, double val) const {
    const int64_t idx = row0 + col * (col + 1) / 2 + row;
    const T o = (T)((row == col) ? val : val * SQRT2);
    a.s_new[idx] = o;
    if (a.mode == 0) a.y_new[idx] = a.y[idx] + rh * (a.sh[idx] - o);
  }
};

template <typename T> __device__ inline void count_sweeps(const EigArgs<T> &a, const PsdDesc &d, const SweepCount &sw) {
  if (!a.stats) return;
  atomicMax(&a.stats[d.inst].eig_sweeps_max, sw.sweeps);
  atomicAdd(&a.stats[d.inst].eig_sweeps_total, sw.sweeps);
  atomicAdd(&a.stats[d.inst].eig_solves, 1);
  if (!sw.converged) atomicAdd(&a.stats[d.inst].eig_not_converged, 1);
  if (sw.fine) atomicAdd(&a.stats[d.inst].eig_refine_steps_total, sw.fine);
}

// Indices of the positive eigenvalues, in order, by the first wave; the list
// is padded to whole groups of 16 with the last column.
__device__ inline void list_positive(const double *lamd, int p, short *pos_idx, int *npos) {
  const int lane = threadIdx.x;
  if (lane >= 64) return;
  int np = 0;
  for (int base = 0; base < p; base += 64) {
    const int i = base + lane;
    const bool on = i < p && lamd[i] > 0.0;
    const unsigned long long m = __ballot(on);
    if (on) pos_idx[np + __popcll(m & ((1ull << lane) - 1))] = (short)i;
    np += __popcll(m);
  }
  if (lane < 16) pos_idx[np + lane] = (short)(p - 1);
  if (lane == 0) *npos = np;
}

// Blocks of order up to 128: the block lies in LDS before and after the
// sweeps.  float32 data sweep in float64 too: the vector units issue float64
// multiply-adds at the rate of (unpacked) float32 ones, a sweep costs about a
// quarter more (LDS traffic, cross-lane moves), and the eigenpairs need no
// refinement afterwards (245 us of 979 at order 100 when they were swept in
// float32).
// Static LDS of the kernels that follow: eigenvalues (the scalars that travel
// with the columns during the sweeps), positive indices, sums.
template <typename T, int NT, int PMAX> struct EigShared {
  __attribute__((aligned(16))) double lamd[PMAX];   // (a multiple of whole pairs of column blocks)
  double red[NT / 64];
  short pos_idx[PMAX + 16];
  SweepShared<T> mx_s;
  int npos;
};

template <typename T, int NT, int G, int NB, int PMAX, int SMAX>
__device__ __forceinline__ void eig_block(const EigArgs<T> &a, const PsdDesc &d, double *W, EigShared<T, NT, SMAX> &sm) {
  static_assert(jacobi_cols<NB>(PMAX) == PMAX && PMAX <= SMAX, "one scalar per column");
  double *lamd = sm.lamd, *red = sm.red;
  short *pos_idx = sm.pos_idx;
  const int p = d.p;
  const int ld = eig_ld<G, NB>(p), nc = jacobi_cols<NB>(p);
  const int nrows = p * (p + 1) / 2;
  const T *v = a.vin + d.row0;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  constexpr int NWv = NT / 64;
  double *Ut = a.rscratch + 3 * (size_t)d.uoff;   // used when a warm start reads or leaves it: row-major

  // S = smat(v) into W (column-major, full).  Four entries in flight per thread.
  for (int base = tid; base < nrows; base += 4 * NT) {
    T val[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) val[u] = v[min(base + u * NT, nrows - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = base + u * NT;
      if (idx < nrows) {
        const int j = svec_col(idx);
        const int i = idx - j * (j + 1) / 2;
        double x = (double)val[u];
        if (i != j) x *= RSQRT2;
        W[i + j * ld] = x;
        W[j + i * ld] = x;
      }
    }
  }
  {   // zero rows p .. ld - 1 and columns p .. nc - 1
    const int npad = ld - p;
    for (int e = tid; e < npad * p; e += NT) {
      const int j = e / npad;
      W[p + (e - j * npad) + j * ld] = 0.0;
    }
    for (int e = p * ld + tid; e < nc * ld; e += NT) W[e] = 0.0;
  }
  sm.mx_s.clear();
  __syncthreads();   // W complete
  // Largest column sum of |S| and ||S||_F^2, 16 lanes per column.  The sums of
  // squares are then added in an order that depends on p alone: a block has
  // the same bits whatever workgroup it is solved in, by itself or in a
  // launch with other classes.
  double colmax = 0;
  for (int j = tid / 16; j < (p + NT / 16 - 1) / (NT / 16) * (NT / 16); j += NT / 16) {
    double part[2] = {0, 0};
    if (j < p)
      for (int i = tid % 16; i < p; i += 16) {
        const double x = W[i + j * ld];
        part[0] += fabs(x);
        part[1] = fma(x, x, part[1]);
      }
    const double sum = group_sums<16, 2>(part);   // of the magnitudes in even lanes, of the squares in odd ones
    if (tid % 2 == 0) colmax = fmax(colmax, sum);
    if (j < p && tid % 16 == 1) lamd[j] = sum;
  }
  const double inf = wg_max<double, NT>(colmax, red);   // contains a barrier: lamd complete after this
  double fro2 = 0;
  for (int j = lane; j < p; j += 64) fro2 += lamd[j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) fro2 += __shfl_xor(fro2, off, 64);
  if (!isfinite((T)fro2)) {
    put_nan<T, NT>(a, d);
    return;   // fro2 is the same in every thread: the whole workgroup leaves
  }
  double c = 1.1 * fmin(sqrt(fro2), inf);
  if (!(c > 0.0)) c = 1;
  // Warm start: W = (S + c I) U_prev, with U_prev the eigenvectors of the same
  // block at the previous unrolled step.  One-sided Jacobi on W computes the
  // same decomposition (W = G V with V orthogonal, W'W diagonal at the end);
  // a nearly diagonalising start only shortens the sweeps.
  const int nt = (p + 15) / 16;
  constexpr int NTMAX = (PMAX + 15) / 16;
  constexpr int HOLD = (NTMAX * NTMAX + NWv - 1) / NWv;
  if (a.warm_read) {
    // S is in W, so the products are held in registers until all are done
    tile_pass<HOLD>(
        nt * nt, wave, NWv,
        [&](int t) {
          const int I = t / nt, J = t % nt;
          return tile_mma<double>(
              I * 16, J * 16, p, [&](int i, int k) -> double { return W[min(i, ld - 1) + min(k, p - 1) * ld]; },
              [&](int k, int j) -> double { return (k < p && j < p) ? Ut[k * p + j] : 0.0; });
        },
        [&](int t, const Mma<double>::v4 &acc) {
          const int I = t / nt, J = t % nt;
          const int col = J * 16 + (lane & 15);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = I * 16 + Mma<double>::row(lane, e);
            if (row < p && col < p) W[row + col * ld] = acc[e] + c * Ut[row * p + col];
          }
        });
  } else {
    for (int i = tid; i < p; i += NT) W[i + i * ld] += c;
  }

  const double scale = column_scale(c);
  constexpr int PMIN = PMAX <= 32 ? 1 : (PMAX <= 64 ? 33 : 65);   // smallest order of the class
  constexpr int EMIN = (PMIN + G - 1) / G, EMAX = (PMAX + G - 1) / G;
  const SweepCount sw = sweep_lds<NT, G, NB, EMIN, EMAX, PMAX>(W, scale, p, ld, sweep_rule(a, p), a.warm_read != 0,
                                                                   lamd, pos_idx, sm.mx_s);
  // eigenvalues: column norms minus the shift
  for (int i = tid; i < p; i += NT) lamd[i] = lamd[i] / scale - c;
  __syncthreads();

  // Pi = sum_{lam_k > 0} lam_k u_k u_k' (upper-triangle tiles)
  const int ntiles = nt * (nt + 1) / 2;
  const PutEntry<T> put(a, d);
  if (a.lam)
    for (int i = tid; i < p; i += NT) a.lam[d.loff + i] = (T)lamd[i];
  if (a.U)
    for (int e = tid; e < p * p; e += NT) {
      const int j = e / p, i = e - j * p;
      a.U[d.uoff + e] = (T)W[i + j * ld];
    }
  if (a.warm_write)
    for (int e = tid; e < p * p; e += NT) {
      const int i = e / p, j = e - i * p;
      Ut[e] = W[i + j * ld];
    }
  list_positive(lamd, p, pos_idx, &sm.npos);
  if (tid == 0) count_sweeps(a, d, sw);
  __syncthreads();
  const int npos = sm.npos;
  for (int t = wave; t < ntiles; t += NWv) {
    int I, J;
    upper_tile(t, I, J);
    // rows past the block's end read the padding or its last row: only
    // entries of the result that are not stored depend on them
    const Mma<double>::v4 acc = tile_mma<double>(
        I * 16, J * 16, npos,
        [&](int i, int k) -> double {
          const int c2 = pos_idx[k];
          return W[min(i, ld - 1) + c2 * ld] * (k < npos ? lamd[c2] : 0.0);
        },
        [&](int k, int j) -> double { return W[min(j, ld - 1) + pos_idx[k] * ld]; });
    const int col = J * 16 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = I * 16 + Mma<double>::row(lane, e);
      if (row <= col && col < p) put(row, col, acc[e]);
    }
  }
}

template <typename T, int NT, int G, int NB, int PMAX>
__global__ __launch_bounds__(NT) void k_psd_eig(const EigArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ EigShared<T, NT, PMAX> sm;
  const PsdDesc d = a.descs[blockIdx.x];
  eig_block<T, NT, G, NB, PMAX>(a, d, reinterpret_cast<double *>(smem_raw), sm);
}

// Blocks of several of those classes in one launch, all with the threads of
// the largest (the smaller ones' sweeps leave waves at the barriers).  For
// calls whose blocks do not fill the device: class after class, such a launch
// takes as long as its largest block, three times over (48 float64 blocks of
// orders 20 to 100: 82 + 214 + 502 us; together 502, and 510 with float64
// angles).
template <typename T>
__global__ __launch_bounds__(512) void k_psd_eig_mixed(const EigArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ EigShared<T, 512, 128> sm;
  const PsdDesc d = a.descs[blockIdx.x];
  double *W = reinterpret_cast<double *>(smem_raw);
  if (d.p <= 32) eig_block<T, 512, 8, 2, 32>(a, d, W, sm);
  else if (d.p <= 64) eig_block<T, 512, 16, 2, 64>(a, d, W, sm);
  else eig_block<T, 512, 16, 4, 128>(a, d, W, sm);
}

// Blocks of order above 128 (float32 to 200, float64 to 140).  In float64
// such a block does not fit the LDS, but it fits the registers of seven waves
// (sixteen lanes and eight columns to a group, 16 E rows, 4 E doubles a lane
// for each of X and Y: 208 registers of 256 at E = 13), and the sweeps need
// LDS only for the half of it that moves.  Before the sweeps LDS holds the
// svec entries of S as they came, in the data's own type (off the diagonal
// S is 1 / sqrt(2) times them, formed in float64 where they are used); after them the eigenvectors go to the scratch,
// column-major, and the products read them from the L2.  The warm start's
// product lands in the registers that the sweeps want it in: result rows of
// the matrix cores' 16 x 16 x 4 are the columns of one block of the four
// groups of a wave, result columns the sixteen lanes of a group.
// Sixteen float32 blocks of orders 129 to 200: 2.1 to 2.3 ms; float32 sweeps with an
// Ogita-Aishima refinement of the eigenpairs in float64 products (two to
// three passes over global scratch, about 515 us each at order 200) took 3.6.
constexpr int LARGE_NT = 448;

// LDS elements in the data's type: S, its leading dimension a multiple of four.
__host__ __device__ constexpr int large_ld(int p) { return (p + 3) & ~3; }

template <typename T, int E, int PMAX>
__device__ __forceinline__ void eig_large(const EigArgs<T> &a, const PsdDesc &d, unsigned char *smem, double *lamd,
                                          short *pos_idx, double *red, SweepShared<T> &mx_s, int *npos_s) {
  constexpr int G = 16, NB = 4, NT = LARGE_NT;
  typedef Mma<double>::v4 v4;
  const int p = d.p, ld = large_ld(p);
  const int nrows = p * (p + 1) / 2;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, kk = lane >> 4;
  T *S = reinterpret_cast<T *>(smem);
  double *Ut = a.rscratch + 3 * (size_t)d.uoff;   // eigenvectors, column-major
  const T *v = a.vin + d.row0;

  double fro2 = 0;
  for (int base = tid; base < nrows; base += 4 * NT) {
    T val[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) val[u] = v[min(base + u * NT, nrows - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = base + u * NT;
      if (idx < nrows) {
        const int j = svec_col(idx);
        const int i = idx - j * (j + 1) / 2;
        const double x = (double)val[u];
        fro2 += x * x;
        S[i + j * ld] = val[u];
        S[j + i * ld] = val[u];
      }
    }
  }
  for (int j = tid; j < p; j += NT)
    for (int i = p; i < ld; ++i) S[i + j * ld] = (T)0;
  mx_s.clear();
  fro2 = wg_sum<double, NT>(fro2, red);   // contains barriers: S complete after this
  if (!isfinite((T)fro2)) {
    put_nan<T, NT>(a, d);
    return;   // the same in every thread
  }
  double colmax = 0;
  for (int j = tid / 16; j < (p + NT / 16 - 1) / (NT / 16) * (NT / 16); j += NT / 16) {
    double sum = 0;
    if (j < p)
      for (int i = r; i < p; i += 16) sum += fabs((double)S[i + j * ld]) * (i == j ? 1.0 : RSQRT2);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    colmax = fmax(colmax, sum);
  }
  const double inf = wg_max<double, NT>(colmax, red);
  double c = 1.1 * fmin(sqrt(fro2), inf);
  if (!(c > 0.0)) c = 1;
  const double scale = column_scale(c);

  const JacobiPlace<G, NB> at(p);
  JacobiRegs<NB, E> R;
  const bool tail = G * (E - 1) + r < p;
  if (a.warm_read) {
    // columns col0 .. col0 + 3 of (S + c I) U: operand row m = g + 4 e is
    // column e of group g's block
    auto product = [&](int side, double (&dst)[NB][E]) {
      const int mcol = 2 * NB * (4 * wave + (r & 3)) + NB * side + (r >> 2);   // column of operand row r
      const bool in = mcol < p;
      const double *u = Ut + (size_t)min(mcol, p - 1) * p;
      v4 acc[E];
#pragma unroll
      for (int t = 0; t < E; ++t) acc[t] = v4{0, 0, 0, 0};
      for (int k0 = 0; k0 < p; k0 += 16) {
        // lane quarter kk takes the k's k0 + 4 kk .. + 3, one per product
        const int k = k0 + 4 * kk, ks = min(k, ld - 4);
        double uk[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) uk[w] = in && k + w < p ? u[min(k + w, p - 1)] : 0.0;
#pragma unroll
        for (int t = 0; t < E; ++t) {
          const T *sc = S + min(16 * t + r, p - 1) * ld + ks;
          T sv[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) sv[w] = sc[w];
#pragma unroll
          for (int w = 0; w < 4; ++w) acc[t] = Mma<double>::op(uk[w], (double)sv[w], acc[t]);
        }
      }
      const int col0 = 2 * NB * at.grp + NB * side;
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int t = 0; t < E; ++t) {
          const int row = 16 * t + r, col = col0 + k;
          const bool on = row < p && col < p;
          const double uu = Ut[(on ? row : 0) + (size_t)(on ? col : 0) * p];
          // S = svec entries / sqrt(2) + (1 - 1 / sqrt(2)) diagonal
          const double dc = fma(1.0 - RSQRT2, (double)S[(on ? row : 0) * (ld + 1)], c);
          dst[k][t] = on ? fma(RSQRT2, acc[t][k], dc * uu) * scale : 0.0;
        }
    };
    product(0, R.x);
    product(1, R.y);
  } else {
    auto column = [&](int col0, double (&dst)[NB][E]) {
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int t = 0; t < E; ++t) {
          const int row = 16 * t + r, col = col0 + k;
          const bool on = row < p && col < p;
          const double x = (double)S[(on ? row : 0) + (on ? col : 0) * ld];
          dst[k][t] = on ? (row == col ? x + c : x * RSQRT2) * scale : 0.0;
        }
    };
    column(2 * NB * at.grp, R.x);
    column(2 * NB * at.grp + NB, R.y);
  }
  int rev;
  __syncthreads();   // S and the previous eigenvectors have been read
  double *order = Ut + p * p;   // the columns, on their way to their order
  const SweepCount sw = jacobi_sweeps<NT, G, NB, E, PMAX>(
      R, at, reinterpret_cast<double *>(smem), lamd, pos_idx, p, sweep_rule(a, p), a.warm_read != 0, mx_s, rev,
      [&](int col, int row, double x) {
        if (col < p) order[col * p + row] = x;
      },
      [&](int col, int row) { return col < p ? order[col * p + row] : 0.0; });
  __syncthreads();
  if (at.busy) {
    const ColumnNorms nm = unit_columns<G, NB, E>(R);
    if (at.act) {
      const BlockCols b = block_cols<G, NB>(at, rev);
      auto store = [&](int col0, const double (&src)[NB][E]) {
#pragma unroll
        for (int k = 0; k < NB; ++k)
          if (col0 + k < p)
#pragma unroll
            for (int t = 0; t < E; ++t)
              if (t < E - 1 || tail) {
                const size_t e = (size_t)(col0 + k) * p + 16 * t + r;
                Ut[e] = src[k][t];
                if (a.U) a.U[d.uoff + e] = (T)src[k][t];
              }
      };
      store(b.x, R.x);
      store(b.y, R.y);
      if (r < NB) {
        if (b.x + r < p) lamd[b.x + r] = nm.x / scale - c;
        if (b.y + r < p) lamd[b.y + r] = nm.y / scale - c;
      }
    }
  }
  __syncthreads();
  if (a.lam)
    for (int i = tid; i < p; i += NT) a.lam[d.loff + i] = (T)lamd[i];
  list_positive(lamd, p, pos_idx, npos_s);
  if (tid == 0) count_sweeps(a, d, sw);
  __syncthreads();
  // Pi = sum_{lam_k > 0} lam_k u_k u_k': a wave takes the row strips wave and
  // E - 1 - wave, E + 1 upper-triangle tiles together
  const int npos = *npos_s;
  const PutEntry<T> put(a, d);
  for (int h = 0; h < 2; ++h) {
    const int I = h == 0 ? wave : E - 1 - wave;
    if (h == 0 ? 2 * wave > E - 1 : 2 * wave >= E - 1) break;
    v4 acc[E];
#pragma unroll
    for (int t = 0; t < E; ++t) acc[t] = v4{0, 0, 0, 0};
    for (int k0 = 0; k0 < npos; k0 += 4) {
      const int k = pos_idx[k0 + kk];
      const double *u = Ut + (size_t)k * p;
      const double ai = u[min(16 * I + r, p - 1)] * (k0 + kk < npos ? lamd[k] : 0.0);
#pragma unroll
      for (int t = 0; t < E; ++t)
        if (t >= I) acc[t] = Mma<double>::op(ai, u[min(16 * t + r, p - 1)], acc[t]);
    }
#pragma unroll
    for (int t = 0; t < E; ++t)
      if (t >= I) {
        const int col = 16 * t + r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = 16 * I + Mma<double>::row(lane, e);
          if (row <= col && col < p) put(row, col, acc[t][e]);
        }
      }
  }
}

template <typename T, int E, int PMAX>
__device__ __forceinline__ void eig_large_by_order(const EigArgs<T> &a, const PsdDesc &d, unsigned char *smem,
                                                   double *lamd, short *pos_idx, double *red, SweepShared<T> &mx_s, int *npos_s) {
  if constexpr (16 * E < PMAX) {
    if (d.p > 16 * E) return eig_large_by_order<T, E + 1, PMAX>(a, d, smem, lamd, pos_idx, red, mx_s, npos_s);
  }
  eig_large<T, E, PMAX>(a, d, smem, lamd, pos_idx, red, mx_s, npos_s);
}

template <typename T, int PMAX>
__global__ __launch_bounds__(LARGE_NT) void k_psd_eig_large(const EigArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[LARGE_NT / 64];
  __shared__ __align__(16) double lamd[jacobi_cols<4>(PMAX)];   // eigenvalues; the moving scalars during the sweeps
  __shared__ short pos_idx[PMAX + 16];
  __shared__ SweepShared<T> mx_s;
  __shared__ int npos_s;
  const PsdDesc d = a.descs[blockIdx.x];
  eig_large_by_order<T, 9, PMAX>(a, d, smem_raw, lamd, pos_idx, red, mx_s, &npos_s);
}

// Leading dimension of the DK VJP's LDS buffers: the smallest stride >= p
// that is 4 modulo 8 words, so the 16 columns one matrix-core operand read
// touches (16 lanes, one column each, four consecutive rows per column
// group) fall on distinct banks; a stride that is a multiple of 16 would put
// all 16 on one bank.
__host__ __device__ constexpr int dk_ld(int p) { return p + ((4 - p % 8) + 8) % 8; }

// Weight of entry (i, j) of U' smat(g) U in the input cotangent.
//   rule 0 (DK, eq:lowner): divided differences of max(., 0), f' on ties,
//     f'(0) = 0.
//   rule 1 (eq:psd-cotangent as autograd evaluates it on U max(L, 0) U', then
//     symmetrised by the svec adjoint): f'(l_i) on the diagonal, else
//     f(l_j) / (l_j - l_i) + f(l_i) / (l_i - l_j) with both quotients formed,
//     so a tie gives inf - inf or 0 / 0 and close eigenvalues cancel.
//   rule 2 (Tikhonov): rule 1 at the eigenvalues of S + eps I.
template <typename T> __device__ inline T vjp_weight(int rule, T li, T lj, bool diag, T eps) {
  if (rule == 0) {
    if (li > (T)0 && lj > (T)0) return (T)1;
    if (li <= (T)0 && lj <= (T)0) return (T)0;
    return fmax(li, lj) / (fabs(li) + fabs(lj));
  }
  const T a = li + eps, b = lj + eps;
  if (diag) return a > (T)0 ? (T)1 : (T)0;
  const T fa = fmax(a, (T)0), fb = fmax(b, (T)0);
  return fb / (b - a) + fa / (a - b);
}

// PSD VJP of orders up to 128: out = svec(U (W o (U' smat(g) U)) U'), W from
// vjp_weight.  Buffers: B0 (p x p, stride dk_ld(p)) in LDS, B1 too when both
// fit, else in global scratch (stride p); U read from LDS when a third buffer
// fits, else from global memory.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_psd_vjp(const PsdDesc *__restrict__ descs, const T *__restrict__ Ug,
                                                const T *__restrict__ lam, const T *__restrict__ g,
                                                T *__restrict__ out, T *__restrict__ scratch, int32_t lds_elems,
                                                int32_t rule, T eps) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *lds = reinterpret_cast<T *>(smem_raw);
  __shared__ T lam_s[128];
  const PsdDesc d = descs[blockIdx.x];
  const int p = d.p, pp = p * p, lp = dk_ld(p), ppl = p * lp;
  const int tid = threadIdx.x;
  T *B0 = lds;
  const int l0 = lp;
  const bool b1_lds = 2 * ppl <= lds_elems;
  T *B1 = b1_lds ? lds + ppl : scratch + d.uoff;
  const int l1 = b1_lds ? lp : p;
  const T *U = Ug + d.uoff;
  int lu = p;
  if (3 * ppl <= lds_elems) {
    T *Ul = lds + 2 * ppl;
    for (int e = tid; e < pp; e += NT) {
      const int j = e / p;
      Ul[(e - j * p) + j * lp] = U[e];
    }
    U = Ul;
    lu = lp;
  }
  for (int i = tid; i < p; i += NT) lam_s[i] = lam[d.loff + i];
  const T *gb = g + d.row0;
  const int nrows = p * (p + 1) / 2;
  for (int idx = tid; idx < nrows; idx += NT) {
    const int j = svec_col(idx);
    const int i = idx - j * (j + 1) / 2;
    T val = gb[idx];
    if (i != j) val *= (T)RSQRT2;
    B0[i + j * l0] = val;
    B0[j + i * l0] = val;
  }
  __syncthreads();
  const int nt = (p + 15) / 16;
  const int wave = tid >> 6, lane = tid & 63;
  const int NWv = NT / 64;
  // B1 = B0 U
  for (int t = wave; t < nt * nt; t += NWv) {
    const int I = t / nt, J = t % nt;
    auto fa = [&](int i, int k) -> T { return (i < p && k < p) ? B0[i + k * l0] : (T)0; };
    auto fb = [&](int k, int j) -> T { return (k < p && j < p) ? U[k + j * lu] : (T)0; };
    const typename Mma<T>::v4 acc = tile_mma<T>(I * 16, J * 16, p, fa, fb);
    const int col = J * 16 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = I * 16 + Mma<T>::row(lane, e);
      if (row < p && col < p) B1[row + col * l1] = acc[e];
    }
  }
  __syncthreads();
  // B0 = W o (U' B1): U' smat(g) U and W are symmetric, so only the upper
  // tiles are formed; entry (row, col), row <= col, is written to both
  // places by the lane that owns it (one writer per element).
  const int nup = nt * (nt + 1) / 2;
  for (int t = wave; t < nup; t += NWv) {
    int I, J;
    upper_tile(t, I, J);
    auto fa = [&](int i, int k) -> T { return (i < p && k < p) ? U[k + i * lu] : (T)0; };
    auto fb = [&](int k, int j) -> T { return (k < p && j < p) ? B1[k + j * l1] : (T)0; };
    const typename Mma<T>::v4 acc = tile_mma<T>(I * 16, J * 16, p, fa, fb);
    const int col = J * 16 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = I * 16 + Mma<T>::row(lane, e);
      if (row <= col && col < p) {
        const T val = vjp_weight<T>(rule, lam_s[row], lam_s[col], row == col, eps) * acc[e];
        B0[row + col * l0] = val;
        B0[col + row * l0] = val;
      }
    }
  }
  __syncthreads();
  // B1 = U B0
  for (int t = wave; t < nt * nt; t += NWv) {
    const int I = t / nt, J = t % nt;
    auto fa = [&](int i, int k) -> T { return (i < p && k < p) ? U[i + k * lu] : (T)0; };
    auto fb = [&](int k, int j) -> T { return (k < p && j < p) ? B0[k + j * l0] : (T)0; };
    const typename Mma<T>::v4 acc = tile_mma<T>(I * 16, J * 16, p, fa, fb);
    const int col = J * 16 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = I * 16 + Mma<T>::row(lane, e);
      if (row < p && col < p) B1[row + col * l1] = acc[e];
    }
  }
  __syncthreads();
  // out = svec(B1 U'), upper tiles
  const int ntiles = nt * (nt + 1) / 2;
  T *ob = out + d.row0;
  for (int t = wave; t < ntiles; t += NWv) {
    int I, J;
    upper_tile(t, I, J);
    auto fa = [&](int i, int k) -> T { return (i < p && k < p) ? B1[i + k * l1] : (T)0; };
    auto fb = [&](int k, int j) -> T { return (k < p && j < p) ? U[j + k * lu] : (T)0; };
    const typename Mma<T>::v4 acc = tile_mma<T>(I * 16, J * 16, p, fa, fb);
    const int col = J * 16 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = I * 16 + Mma<T>::row(lane, e);
      if (row <= col && col < p) {
        const int idx = col * (col + 1) / 2 + row;
        ob[idx] = (row == col) ? acc[e] : acc[e] * (T)SQRT2;
      }
    }
  }
}

// The same for orders above 128, where U and B1 do not fit the LDS beside B0:
// a wave takes a strip of 16 result columns, E tiles in registers, so the
// strip's operand is read once, and each lane takes four consecutive k of a
// group of 16 (one 16-byte load where the operand is stored along k).  Bound
// by the matrix cores at 13 waves on four of them and the operands' latency;
// tile by tile, each reading both its operands in single strided entries,
// 16 blocks of orders 129 to 200 in float32 took 612 us, so 238.
template <typename T, int E>
__device__ __forceinline__ void vjp_large(const PsdDesc &d, const T *__restrict__ U, const T *lam_s,
                                          const T *__restrict__ gb, T *__restrict__ ob, T *B1, T *B0, int rule,
                                          T eps, int NT) {
  typedef typename Mma<T>::v4 v4;
  const int p = d.p, l0 = large_ld(p);
  const int tid = threadIdx.x, J = tid >> 6, lane = tid & 63, r = lane & 15, kk = lane >> 4;
  const int nrows = p * (p + 1) / 2;
  for (int idx = tid; idx < nrows; idx += NT) {
    const int j = svec_col(idx);
    const int i = idx - j * (j + 1) / 2;
    T val = gb[idx];
    if (i != j) val *= (T)RSQRT2;
    B0[i + j * l0] = val;
    B0[j + i * l0] = val;
  }
  for (int j = tid; j < p; j += NT)
    for (int i = p; i < l0; ++i) B0[i + j * l0] = (T)0;
  __syncthreads();
  const bool act = J < E;
  const int col = 16 * J + r;   // this lane's column of the strip
  const bool in = act && col < p;
  const int cs = in ? col : 0;
  v4 acc[E];
  // acc[t] = sum_k a(t, k..k+3) b(k..k+3) for the tiles t that `tiles` wants;
  // both are zero from k = p on
  auto strip = [&](auto tiles, auto a4, auto b4) {
#pragma unroll
    for (int t = 0; t < E; ++t) acc[t] = v4{0, 0, 0, 0};
    for (int k0 = 0; k0 < p; k0 += 16) {
      const int k = k0 + 4 * kk;
      T b[4];
      b4(k, b);
#pragma unroll
      for (int w = 0; w < 4; ++w) b[w] = in ? b[w] : (T)0;
#pragma unroll
      for (int t = 0; t < E; ++t)
        if (tiles(t)) {
          T a[4];
          a4(min(16 * t + r, p - 1), k, a);
#pragma unroll
          for (int w = 0; w < 4; ++w) acc[t] = Mma<T>::op(a[w], b[w], acc[t]);
        }
    }
  };
  // four entries along k of column c of a p x p matrix, of its row c, and of B0
  auto along = [&](const T *M, int c, int k, T (&x)[4]) {
    if (k + 4 <= p) {
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = M[k + w + c * p];
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = k + w < p ? M[k + w + c * p] : (T)0;
    }
  };
  auto across = [&](const T *M, int c, int k, T (&x)[4]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const T e = M[c + min(k + w, p - 1) * p];
      x[w] = k + w < p ? e : (T)0;
    }
  };
  auto lds4 = [&](int c, int k, T (&x)[4]) {   // B0 is symmetric; its rows p to l0 - 1 are zero
#pragma unroll
    for (int w = 0; w < 4; ++w) x[w] = 0;
    if (k < p) {
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = B0[k + w + c * l0];
    }
  };
  auto all = [](int) { return true; };
  auto upper = [&](int t) { return t <= J; };
  auto put_b1 = [&]() {
#pragma unroll
    for (int t = 0; t < E; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * t + Mma<T>::row(lane, e);
        if (row < p && in) B1[row + col * p] = acc[t][e];
      }
  };
  if (act) {   // B1 = B0 U
    strip(all, lds4, [&](int k, T (&x)[4]) { along(U, cs, k, x); });
    put_b1();
  }
  __syncthreads();
  if (act) {   // B0 = W o (U' B1), upper tiles; one lane writes an entry to both places
    strip(upper, [&](int i, int k, T (&x)[4]) { along(U, i, k, x); }, [&](int k, T (&x)[4]) { along(B1, cs, k, x); });
#pragma unroll
    for (int t = 0; t < E; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * t + Mma<T>::row(lane, e);
        if (t <= J && row <= col && in) {
          const T val = vjp_weight<T>(rule, lam_s[row], lam_s[col], row == col, eps) * acc[t][e];
          B0[row + col * l0] = val;
          B0[col + row * l0] = val;
        }
      }
  }
  __syncthreads();
  if (act) {   // B1 = U B0
    strip(all, [&](int i, int k, T (&x)[4]) { across(U, i, k, x); }, [&](int k, T (&x)[4]) { lds4(cs, k, x); });
    put_b1();
  }
  __syncthreads();
  if (act) {   // out = svec(B1 U'), upper tiles
    strip(upper, [&](int i, int k, T (&x)[4]) { across(B1, i, k, x); }, [&](int k, T (&x)[4]) { across(U, cs, k, x); });
#pragma unroll
    for (int t = 0; t < E; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 16 * t + Mma<T>::row(lane, e);
        if (t <= J && row <= col && in)
          ob[col * (col + 1) / 2 + row] = row == col ? acc[t][e] : acc[t][e] * (T)SQRT2;
      }
  }
}

template <typename T, int E, int EMAX, typename... A>
__device__ __forceinline__ void vjp_large_by_order(const PsdDesc &d, A... args) {
  if constexpr (E < EMAX) {
    if (d.p > 16 * E) return vjp_large_by_order<T, E + 1, EMAX>(d, args...);
  }
  vjp_large<T, E>(d, args...);
}

template <typename T, int EMAX>
__global__ __launch_bounds__(64 * EMAX) void k_psd_vjp_large(const PsdDesc *__restrict__ descs,
                                                             const T *__restrict__ Ug, const T *__restrict__ lam,
                                                             const T *__restrict__ g, T *__restrict__ out,
                                                             T *__restrict__ scratch, int32_t rule, T eps) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ T lam_s[MAXP];
  const PsdDesc d = descs[blockIdx.x];
  for (int i = threadIdx.x; i < d.p; i += 64 * EMAX) lam_s[i] = lam[d.loff + i];
  vjp_large_by_order<T, 9, EMAX>(d, Ug + d.uoff, lam_s, g + d.row0, out + d.row0, scratch + d.uoff,
                                 reinterpret_cast<T *>(smem_raw), rule, eps, 64 * EMAX);
}

// Elements of the exchange buffer for a launch whose largest order is p.
template <int G, int NB, int E, int EMAX, int PMAX> constexpr int exchange_elems(int p) {
  if constexpr (E < EMAX) {
    if (p > G * E) return exchange_elems<G, NB, E + 1, EMAX, PMAX>(p);
  }
  return Exchange<G, NB, E, PMAX>::elems;
}

// Dynamic LDS of a block of order p in a class.
template <int G, int NB, int PMAX> size_t eig_lds(int32_t p) {
  const size_t block = (size_t)jacobi_cols<NB>(p) * (size_t)eig_ld<G, NB>(p);
  const size_t exch = (size_t)exchange_elems<G, NB, 1, (PMAX + G - 1) / G, PMAX>(p);
  return std::max(block, exch) * sizeof(double);
}

template <typename T, int NT, int G, int NB, int PMAX>
void run_eig(const EigArgs<T> &a, int32_t n, int32_t max_p, hipStream_t st) {
  (void)allow_dyn_lds(reinterpret_cast<const void *>(&k_psd_eig<T, NT, G, NB, PMAX>));
  k_psd_eig<T, NT, G, NB, PMAX><<<n, NT, eig_lds<G, NB, PMAX>(max_p), st>>>(a);
}

template <typename T, int PMAX>
void run_eig_large(const EigArgs<T> &a, int32_t n, int32_t max_p, hipStream_t st) {
  const size_t block = (size_t)max_p * large_ld(max_p) * sizeof(T);
  const size_t exch = (size_t)exchange_elems<16, 4, 9, (PMAX + 15) / 16, PMAX>(max_p) * sizeof(double);
  (void)allow_dyn_lds(reinterpret_cast<const void *>(&k_psd_eig_large<T, PMAX>));
  k_psd_eig_large<T, PMAX><<<n, LARGE_NT, std::max(block, exch), st>>>(a);
}

}  // namespace

// Blocks arrive sorted by order class (see the plan): callers pass one class
// per call with its largest order.  Lanes and column blocks per class: two
// columns per block while that fills at most one wave per SIMD (a sweep is
// then its ~p dependent steps, each as short as its rows are spread); four
// above order 64, where the exchange of blocks between the groups costs as
// much as the rotations (order 100: 55 us per sweep against 64 us with two).
// The largest class's configuration is named by kEigThreads[3]; it has no
// other, and runs seven waves (above).
template <typename T>
void launch_psd_step(const PsdDesc *d, int32_t n, const PsdLaunchCfg &cfg, const T *rho_hat, const T *vv,
                     const T *sh, const T *y, T *s_new, T *y_new, T *U, T *lam, double *rscratch,
                     bool warm, cosmo_stats *stats, hipStream_t st) {
  if (n <= 0) return;
  const int mp = cfg.max_p;
  const int cls = mp <= 32 ? 0 : mp <= 64 ? 1 : mp <= 128 ? 2 : 3;
  const bool alt = cfg.threads != 0 && cfg.threads == kEigThreadsAlt[cls] && cfg.threads != kEigThreads[cls];
  const EigArgs<T> a{d, cfg.max_sweeps, cfg.tol, y_new != nullptr ? 0 : 1, rho_hat, vv, sh, y, s_new, y_new, U, lam,
                     stats, cfg.refine, rscratch, warm && rscratch ? 1 : 0, cfg.keep_warm && rscratch ? 1 : 0};
  static_assert(kEigThreads[0] == 64 && kEigThreads[1] == 256 && kEigThreads[2] == 512 && kEigThreads[3] == 1024,
                "class defaults");
  static_assert(kEigThreadsAlt[0] == 128 && kEigThreadsAlt[1] == 512 && kEigThreadsAlt[2] == 1024, "class alternatives");
  if (cls == 0) {
    if (alt) run_eig<T, 128, 16, 2, 32>(a, n, mp, st); else run_eig<T, 64, 8, 2, 32>(a, n, mp, st);
  } else if (cls == 1) {
    if (alt) run_eig<T, 512, 16, 2, 64>(a, n, mp, st); else run_eig<T, 256, 16, 2, 64>(a, n, mp, st);
  } else if (cls == 2) {
    if (alt) run_eig<T, 1024, 16, 2, 128>(a, n, mp, st); else run_eig<T, 512, 16, 4, 128>(a, n, mp, st);
  } else {
    run_eig_large<T, std::is_same<T, float>::value ? COSMO_MAX_PSD_ORDER_F32 : COSMO_MAX_PSD_ORDER_F64>(a, n, mp, st);
  }
}

// Classes 0 to 2 of a projection without a plan, descriptors in class order;
// begin, maxp: of the three classes.  One launch for all where more than one
// has blocks and all of them together do not fill the device.
template <typename T>
void launch_psd_proj(const PsdDesc *d, const int32_t *begin, const int32_t *maxp, const PsdLaunchCfg &cfg, const T *in,
                     T *out, T *U, T *lam, double *rscratch, int32_t ncu, hipStream_t st) {
  const int32_t n = begin[3] - begin[0];
  const int classes = (begin[1] > begin[0]) + (begin[2] > begin[1]) + (begin[3] > begin[2]);
  if (classes > 1 && n <= ncu) {
    const EigArgs<T> a{d + begin[0], cfg.max_sweeps, cfg.tol, 1, nullptr, in, nullptr, nullptr, out, nullptr, U, lam,
                       nullptr, cfg.refine, rscratch, 0, 0};
    size_t lds = 0;
    if (begin[1] > begin[0]) lds = std::max(lds, eig_lds<8, 2, 32>(maxp[0]));
    if (begin[2] > begin[1]) lds = std::max(lds, eig_lds<16, 2, 64>(maxp[1]));
    if (begin[3] > begin[2]) lds = std::max(lds, eig_lds<16, 4, 128>(maxp[2]));
    (void)allow_dyn_lds(reinterpret_cast<const void *>(&k_psd_eig_mixed<T>));
    k_psd_eig_mixed<T><<<n, 512, lds, st>>>(a);
    return;
  }
  for (int c = 0; c < 3; ++c) {
    PsdLaunchCfg one = cfg;
    one.max_p = maxp[c];
    launch_psd_step<T>(d + begin[c], begin[c + 1] - begin[c], one, nullptr, in, nullptr, nullptr, out, nullptr, U, lam,
                       rscratch, false, nullptr, st);
  }
}

// 16 waves by default: a block of order ~100 has 49 output tiles per
// product, so the longest wave runs 4 of them instead of 7 with 8 waves; the
// autotuner may pick 8 waves (two workgroups per compute unit where LDS
// allows).  Every tile is formed by one wave with the same instructions
// whichever wave it is, so both shapes give bitwise the same result.
template <typename T, int NT>
bool run_vjp(const PsdDesc *d, int32_t n, int32_t max_p, const T *U, const T *lam, const T *g, T *out, T *scratch,
             hipStream_t st, int32_t rule, double eps) {
  const size_t dyn_bytes = allow_dyn_lds(reinterpret_cast<const void *>(&k_psd_vjp<T, NT>));
  // LDS holds B0, then B1, then U while they fit; B0 alone always does (order
  // 128 in float64: 135,168 bytes)
  const size_t ppl = (size_t)max_p * dk_ld(max_p);   // p dk_ld(p) does not decrease with p
  const size_t budget = dyn_bytes / sizeof(T);
  if (max_p > 128 || ppl > budget) return false;
  const size_t elems = std::min<size_t>(3, budget / ppl) * ppl;
  k_psd_vjp<T, NT><<<n, NT, elems * sizeof(T), st>>>(d, U, lam, g, out, scratch, (int32_t)elems, rule, (T)eps);
  return true;
}

template <typename T>
bool run_vjp_large(const PsdDesc *d, int32_t n, int32_t max_p, const T *U, const T *lam, const T *g, T *out, T *scratch,
                   hipStream_t st, int32_t rule, double eps) {
  constexpr int PMAX = std::is_same<T, float>::value ? COSMO_MAX_PSD_ORDER_F32 : COSMO_MAX_PSD_ORDER_F64;
  constexpr int EMAX = (PMAX + 15) / 16;
  const size_t dyn_bytes = allow_dyn_lds(reinterpret_cast<const void *>(&k_psd_vjp_large<T, EMAX>));
  const size_t need = (size_t)max_p * large_ld(max_p) * sizeof(T);
  if (max_p > PMAX || need > dyn_bytes) return false;
  k_psd_vjp_large<T, EMAX><<<n, 64 * EMAX, need, st>>>(d, U, lam, g, out, scratch, rule, (T)eps);
  return true;
}

template <typename T>
bool launch_psd_vjp(const PsdDesc *d, int32_t n, int32_t max_p, const T *U, const T *lam, const T *g, T *out,
                    T *scratch, hipStream_t st, int32_t rule, double eps, int32_t threads) {
  if (n <= 0) return true;
  static_assert(kVjpThreads == 1024 && kVjpThreadsAlt == 512, "VJP shapes");
  if (max_p > 128) return run_vjp_large<T>(d, n, max_p, U, lam, g, out, scratch, st, rule, eps);
  if (threads == kVjpThreadsAlt) return run_vjp<T, 512>(d, n, max_p, U, lam, g, out, scratch, st, rule, eps);
  return run_vjp<T, 1024>(d, n, max_p, U, lam, g, out, scratch, st, rule, eps);
}

template void launch_psd_step<float>(const PsdDesc *, int32_t, const PsdLaunchCfg &, const float *, const float *,
                                     const float *, const float *, float *, float *, float *, float *, double *,
                                     bool, cosmo_stats *, hipStream_t);
template void launch_psd_step<double>(const PsdDesc *, int32_t, const PsdLaunchCfg &, const double *,
                                      const double *, const double *, const double *, double *, double *, double *,
                                      double *, double *, bool, cosmo_stats *, hipStream_t);
template void launch_psd_proj<float>(const PsdDesc *, const int32_t *, const int32_t *, const PsdLaunchCfg &,
                                     const float *, float *, float *, float *, double *, int32_t, hipStream_t);
template void launch_psd_proj<double>(const PsdDesc *, const int32_t *, const int32_t *, const PsdLaunchCfg &,
                                      const double *, double *, double *, double *, double *, int32_t, hipStream_t);
template bool launch_psd_vjp<float>(const PsdDesc *, int32_t, int32_t, const float *, const float *, const float *,
                                    float *, float *, hipStream_t, int32_t, double, int32_t);
template bool launch_psd_vjp<double>(const PsdDesc *, int32_t, int32_t, const double *, const double *,
                                     const double *, double *, double *, hipStream_t, int32_t, double, int32_t);
}  // namespace cosmo
