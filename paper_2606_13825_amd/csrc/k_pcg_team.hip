// The per-instance CG with a team of workgroups per instance (form 0 of plans
// with fewer instances than compute units).  Same iteration and stopping rule
// as k_pcg (see k_pcg.hip); an instance's rows and columns are cut into
// `slices` parts, one per workgroup of a full team, and the workgroups meet at
// two team barriers per iteration: after the row half of the operator, which
// also gives p'Mp = sum rho_hat (A p)^2 + p'(P p + sigma p), and with the sums
// of r'z and r'r.  (With p'Mp formed from the columns of M p, behind a third
// barrier, the covariance-steering solves below took 10 % longer.)
//
// Teams.  A team's workgroups run on one XCD: each reads its XCD's number
// (the XCC_ID hardware register) and takes a ticket there, so what a team
// exchanges stays in that XCD's L2, which its compute units share -- no L2
// write-back or invalidation, which make a device-wide exchange several times
// as expensive (measured, one barrier with 16 KB exchanged: 3.2 us here; 6.5
// us with agent-scope release and acquire, which a team spread over XCDs
// needs).  A store is in L2 when its wave's vmcnt reaches 0, which every wave
// waits for before a team barrier; what other workgroups wrote is read with
// agent-scope loads, which pass the compute unit's own cache by.
//
// A team starts with as many members as have arrived: it closes when it is
// full, or when a member has waited FORM_TICKS for more; later arrivals leave
// (a member does slices rank, rank + size, ..).  So the launch needs no
// co-residency: whatever else runs on the device, the workgroups that are
// running form teams and finish.  The teams of a launch take instances from
// one queue, largest first, until it is empty.  Sums are formed per slice and
// added in slice order: the result does not depend on the teams' sizes.
// Waits inside a closed team end because all its members are running; each is
// bounded in time all the same.  A member whose wait runs out, and with it its
// team, gives its instance up and leaves; the last workgroup of the launch
// then marks the instances given up, and those that no team took, as
// non-finite and not converged.
//
// p (in the residual pass: x) is kept whole in every workgroup's LDS: the row
// half gathers from there, and p = z + beta p needs no barrier of its own.
// The column half first copies the rows that its columns use, where they
// fit (a coalesced copy with all loads in flight; gathers of single entries
// past the compute unit's cache took 10 us a pass on a slice of 300 columns of
// 50 entries).
//
// A workgroup keeps its slice of A in LDS through a solve's iterations, and
// its slice of A' where that still fits: an instance's A and A' do not fit the
// die's L2 together with its vectors, and read from behind it they took 8 to
// 11 us a half (covariance steering with 290,000 entries, a program with
// 500,000); from LDS a half takes 3 to 4.  Slices of A' that do not fit are
// read with 16-bit indices and eight lanes per row of 50 to 256 entries (16
// lanes left most of their loads without an entry: 11 us, now 7).
//
// What bounds it: latency.  Per iteration about 5 us are the two team
// barriers with their sums and 2 to 3 the copies of p and t; the rest is the
// operator, by the LDS's rate and, for what is not kept, by dependent loads of
// the few rows a lane group has.  Measured per iteration, one workgroup per
// instance or the device-wide form against teams of 32: 4 Huber instances of
// 2000 x 500 in float64 137 -> 19 us; 16 covariance-steering instances 97 ->
// 20 us; one program with 500,000 nonzeros 83 -> 18 us.
#include <algorithm>
#include <type_traits>

#include "pcg_ops.h"

namespace cosmo {
namespace {

constexpr uint64_t FORM_TICKS = 5000;           // 50 us of the 100 MHz real-time counter

__device__ inline uint32_t ld_agent(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_agent(uint32_t *p, uint32_t x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// An array other workgroups of the team write.
template <typename T> struct Shared {
  const T *p;
  __device__ T operator[](int64_t i) const {
    return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};
// The LDS copy of the instance's slice of a column vector.
template <typename T> struct Local {
  const T *p;
  int32_t n0;
  __device__ T operator[](int32_t c) const { return p[c - n0]; }
};

extern __shared__ double dyn_lds[];

// Sum of a row's products by L lanes, four entries per lane in flight.  The
// order of the additions, and so the result, depends on L and the row alone.
template <int L, typename AT, typename V, typename G> __device__ inline AT strided_sum(int len, V val, G gather) {
  AT a = 0;
  for (int k = threadIdx.x % L; k < len; k += 4 * L) {
    AT e[4], g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ku = min(k + u * L, len - 1);   // past the end: the last entry again, not counted
      e[u] = (AT)val(ku);
      g[u] = (AT)gather(ku);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) a = k + u * L < len ? fma(e[u], g[u], a) : a;
  }
  return sub_sum(a, L);
}

// Eight waves: the kernel's state does not fit the 128 registers of sixteen
// (with 1024 threads 16 covariance-steering instances took 8.5 ms per training
// step instead of 6.9, one program with 500,000 nonzeros 3.8 instead of 3.2).
// In the 256 of eight it fits without dense blocks (185 to 201) and with
// narrow ones; the instantiations for the widest blocks of a stored type spill
// 18 to 73, those that run 2000 x 500 blocks stored in float32 27.
constexpr int NTH = 512;

// Where the length classes of a slice end in its list, from its list ranges
// (class 0, class 1, class 2: short, long rows).
__device__ inline void class_ends(const int64_t *cut, int32_t (&end)[4]) {
  auto uni = [](int64_t x) { return __builtin_amdgcn_readfirstlane((int32_t)x); };
  end[0] = uni(cut[1] - cut[0]);
  end[1] = end[0] + uni(cut[3] - cut[2]);
  end[2] = end[1] + uni(cut[5] - cut[4]);
  end[3] = end[2] + uni(cut[6] - cut[5]);
}
__device__ inline int64_t list_at(const int64_t *cut, const int32_t (&end)[4], int q) {
  return q < end[0] ? cut[0] + q : q < end[1] ? cut[2] + (q - end[0]) : cut[4] + (q - end[1]);
}

// A slice's rows (or columns) in LDS: per listed row its id and where its
// entries begin, for rows rho_hat, then values and 16-bit indices.  Offsets
// into the dynamic LDS, the same in every thread (scalar registers).
template <typename T> struct Kept {
  int32_t o_first = 0, o_rho = 0, o_val = 0, o_idx = 0, o_row = 0;
  int32_t end[4] = {0, 0, 0, 0};   // where each length class ends
  bool on = false;
  __device__ void place(int64_t at, const int64_t *cut, int32_t entries, bool with_rho) {
    on = true;
    class_ends(cut, end);
    auto uni = [](int64_t x) { return __builtin_amdgcn_readfirstlane((int32_t)x); };
    o_row = uni(at);
    o_first = o_row + 4 * end[3];
    o_rho = o_row + ((end[3] + 1) * 8 + 15) / 16 * 16;
    o_val = o_rho + (with_rho ? (end[3] * (int32_t)sizeof(T) + 15) / 16 * 16 : 0);
    o_idx = o_val + (uni(entries) * (int32_t)sizeof(T) + 15) / 16 * 16;
  }
  template <typename X> static __device__ X *lds(int32_t off) {
    return reinterpret_cast<X *>(reinterpret_cast<char *>(dyn_lds) + off);
  }
  __device__ int32_t *row() const { return lds<int32_t>(o_row); }
  __device__ int32_t *first() const { return lds<int32_t>(o_first); }
  __device__ T *rho() const { return lds<T>(o_rho); }
  // 16 lanes per row; id(row) is what is kept as the row's id; base: the index
  // kept as 0.  Ends with a barrier.
  template <bool RHO, typename CT, typename Id>
  __device__ void fill(const int64_t *cut, int32_t entries, const int32_t *rows, const RowSpan *span,
                       const int32_t *begin, const CT *col, const T *v, const T *rho_hat, int64_t base, Id id) {
    const int lane = threadIdx.x % 16;
    T *val = lds<T>(o_val);
    uint16_t *idx = lds<uint16_t>(o_idx);
    for (int q0 = threadIdx.x / 16; q0 < end[3]; q0 += 4 * (NTH / 16)) {   // four rows in flight per 16 lanes
      int32_t r[4], o[4];
      RowSpan sp[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = min(q0 + u * (NTH / 16), end[3] - 1);   // past the end: the last row again, not stored
        const int64_t li = list_at(cut, end, q);
        r[u] = rows[li];
        o[u] = begin[li];
        sp[u] = span[li];
      }
      T e[4], rh[4];
      CT c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool on = lane < sp[u].k1 - sp[u].kb;
        e[u] = on ? v[sp[u].kb + lane] : (T)0;
        c[u] = on ? col[sp[u].kb + lane] : (CT)0;
        rh[u] = RHO ? rho_hat[r[u]] : (T)0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + u * (NTH / 16), len = (int)(sp[u].k1 - sp[u].kb);
        if (q >= end[3]) continue;
        if (lane < len) {
          val[o[u] + lane] = e[u];
          idx[o[u] + lane] = (uint16_t)(c[u] - base);
        }
        for (int k = lane + 16; k < len; k += 16) {
          val[o[u] + k] = v[sp[u].kb + k];
          idx[o[u] + k] = (uint16_t)(col[sp[u].kb + k] - base);
        }
        if (lane == 0) {
          row()[q] = id(r[u]);
          first()[q] = o[u];
          if (RHO) rho()[q] = rh[u];
        }
      }
    }
    if (threadIdx.x == 0) first()[end[3]] = entries;
    __syncthreads();
  }
  // Row q of the list, L lanes: its sum, on every lane.  x: the vector by kept
  // index.
  template <int L, typename AT, typename X> __device__ AT row_sum(int q, const X *x) const {
    const T *val = lds<T>(o_val);
    const uint16_t *idx = lds<uint16_t>(o_idx);
    const int o = first()[q];
    return strided_sum<L, AT>(first()[q + 1] - o, [&](int k) { return val[o + k]; }, [&](int k) { return x[idx[o + k]]; });
  }
};

// Length classes of a slice's rows, by rows [q0, q1) of its list and the lanes
// that one of them takes; f<L>(q) runs on those lanes.
template <typename F> __device__ inline void strided_rows(const int32_t (&end)[4], F f) {
  auto pass = [&](auto lanes, int q0, int q1) {
    constexpr int L = decltype(lanes)::value;
    for (int q = q0 + threadIdx.x / L; q < q1; q += NTH / L) f(lanes, q);
  };
  pass(std::integral_constant<int, 64>{}, end[2], end[3]);
  pass(std::integral_constant<int, 16>{}, end[1], end[2]);
  pass(std::integral_constant<int, 4>{}, end[0], end[1]);
  pass(std::integral_constant<int, 1>{}, 0, end[0]);
}

// Control words of one launch, zero before it and left zero by it: a head, a
// record per team, and per queue position whether its instance was given up.
struct TeamHead {
  uint32_t queue, exits;
  uint32_t aborted;   // a team gave up
  uint32_t pad[61];
  uint32_t ticket[TEAM_XCDS * 64];   // one line per XCD
};
struct TeamRec {
  uint32_t joined;   // arrivals; CLOSED once the team has its members
  uint32_t size;     // members, set by whoever closed it
  uint32_t inst;     // queue position of the instance in work
  uint32_t abort;
  uint32_t pad0[60];
  uint32_t count;    // arrivals at barriers
  uint32_t pad1[63];
  uint32_t gen;      // barriers passed
  uint32_t pad2[63];
  double sum[2][3][TEAM_MAX_SLICES];   // slices' partial sums, two sets in turn
};
constexpr uint32_t CLOSED = 0x80000000u;

struct Team {
  TeamRec *rec;
  uint64_t wait_ticks;
  uint32_t rank, size, gen, parity;
  bool aborted;
};

// All members' stores before it are visible to Shared reads after it.
__device__ inline void team_sync(Team &tm, int32_t *flag_s) {
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's stores are in L2
  __syncthreads();
  const uint32_t target = tm.gen + 1;
  if (tm.size > 1) {
    if (threadIdx.x == 0) {
      if (__hip_atomic_fetch_add(&tm.rec->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
          tm.size * target - 1) {
        st_agent(&tm.rec->gen, target);
      } else {
        const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        while (ld_agent(&tm.rec->gen) < target) {
          if (ld_agent(&tm.rec->abort) != 0) break;
          if (__builtin_amdgcn_s_memrealtime() - t0 > tm.wait_ticks) {
            st_agent(&tm.rec->abort, 1u);
            break;
          }
        }
      }
      *flag_s = (int32_t)ld_agent(&tm.rec->abort);
    }
    __syncthreads();
    tm.aborted = tm.aborted || *flag_s != 0;
  }
  tm.gen = target;
}

// Team sums of up to three values whose slice partials this workgroup has
// stored (by thread 0) in the record's current set; same bits in every thread
// of every member.
template <int NV> __device__ inline void team_sums(Team &tm, int slices, double (&out)[NV], double *sum_s,
                                                            int32_t *flag_s) {
  team_sync(tm, flag_s);
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double x = lane < slices ? Shared<double>{tm.rec->sum[tm.parity][k]}[lane] : 0.0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
      if (lane == 0) sum_s[k] = x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) out[k] = sum_s[k];
  tm.parity ^= 1;
}

template <typename T, int DMP, typename TG>
__global__ __launch_bounds__(NTH) void k_pcg_team(View<T> v, TeamView tv, const T *__restrict__ rho_hat,
                                                           const T *__restrict__ dg, const double *__restrict__ rhs,
                                                           T *x, T *r, T *z, T *Mp, T *t, double *t64,
                                                           double *c64, T tol, int32_t max_iter, const T *__restrict__ alpha_k,
                                                           const T *__restrict__ xold, T *__restrict__ xnew,
                                                           const T *__restrict__ gx_in, T *__restrict__ gx_out,
                                                           int32_t mode, cosmo_stats *stats) {
  __shared__ T red[2 * (NTH / 64)];
  __shared__ double redd[2 * (NTH / 64)];
  __shared__ double sum_s[3];
  __shared__ int32_t flag_s;
  __shared__ uint32_t join_s[3];
  __shared__ int64_t cuts[TEAM_MAX_SLICES][20];
  const int tid = threadIdx.x;
  const int V = tv.slices;
  TeamHead *head = static_cast<TeamHead *>(tv.state);
  TeamRec *recs = reinterpret_cast<TeamRec *>(head + 1);
  uint32_t *given_up = reinterpret_cast<uint32_t *>(recs + TEAM_XCDS * tv.teams_per_xcd);

  // ---- join a team --------------------------------------------------------------
  if (tid == 0) {
    const uint32_t xcc = (uint32_t)__builtin_amdgcn_s_getreg(20 | (3 << 11)) % TEAM_XCDS;   // XCC_ID, bits 3:0
    const uint32_t ticket = __hip_atomic_fetch_add(&head->ticket[64 * xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t team = TEAM_NONE, rank = 0, size = 0;
    const uint32_t M = tv.members;
    if (ticket < (uint32_t)tv.teams_per_xcd * M) {
      TeamRec *rec = recs + xcc * tv.teams_per_xcd + ticket / M;
      const uint32_t old = __hip_atomic_fetch_add(&rec->joined, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!(old & CLOSED)) {
        team = xcc * tv.teams_per_xcd + ticket / M;
        rank = old;
        auto close = [&]() {
          const uint32_t was = __hip_atomic_fetch_or(&rec->joined, CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (!(was & CLOSED)) st_agent(&rec->size, was);
        };
        if (rank == M - 1) close();
        const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        while ((size = ld_agent(&rec->size)) == 0)
          if (__builtin_amdgcn_s_memrealtime() - t0 > FORM_TICKS) close();
      }
    }
    join_s[0] = team;
    join_s[1] = rank;
    join_s[2] = size;
  }
  __syncthreads();
  Team tm{recs + (join_s[0] == TEAM_NONE ? 0 : join_s[0]), tv.wait_ticks, join_s[1], join_s[2], 0, 0, false};

  T *pl = reinterpret_cast<T *>(dyn_lds);
  auto all = [](int32_t) { return true; };
  while (join_s[0] != TEAM_NONE) {
    // ---- the next instance of the queue ------------------------------------------
    uint32_t popped = (uint32_t)v.B;   // what this thread took from the queue
    if (tm.rank == 0 && tid == 0) {
      popped = __hip_atomic_fetch_add(&head->queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      st_agent(&tm.rec->inst, popped);
    }
    team_sync(tm, &flag_s);
    if (tid == 0) sum_s[0] = (double)(tm.aborted ? popped : ld_agent(&tm.rec->inst));
    __syncthreads();
    const uint32_t pos = (uint32_t)sum_s[0];
    __syncthreads();   // sum_s is written again below
    if (pos >= (uint32_t)v.B) break;
    if (tm.aborted) {
      if (tid == 0) st_agent(&given_up[pos], 1u);
      break;
    }
    const int b = tv.order[pos];
    const int64_t n0 = v.n_off[b], n1 = v.n_off[b + 1];
    const int n = (int)(n1 - n0);
    // the waves' partials of the dense product, then the sums of a slice's dense columns
    double *dl = dyn_lds + ((size_t)n * sizeof(T) + 7) / 8;
    const int64_t BV = (int64_t)v.B * V, bV = (int64_t)b * V;
    const Local<T> pv{pl, (int32_t)n0};
    char *tl = reinterpret_cast<char *>(dyn_lds) + tv.cap_off;   // the copied rows of t, then a kept slice

    // where this workgroup's slices begin and end: list ranges of the rows
    // (0-6: three classes, the last one's short and long rows) and of the
    // columns (7-13), the rows the columns use (14, 15), the columns (16, 17),
    // the dense ones among them (18, 19)
    for (int e = tid; e < 20 * V; e += NTH) {
      const int s = e / 20, k = e % 20;
      if (s % (int)tm.size != (int)tm.rank) continue;
      const int64_t *sl = (k < 7 ? tv.sliceA : tv.sliceAt) + bV + s, *mid = (k < 7 ? tv.midA : tv.midAt) + bV + s;
      const int q = k < 7 ? k : k - 7;
      cuts[s][k] = k >= 18 ? (DMP > 0 ? tv.dense_cut[bV + s + k - 18] : 0) : k >= 16 ? tv.colcut[bV + s + k - 16]
                   : k >= 14 ? tv.used[2 * (bV + s) + k - 14]
                   : q == 5 ? *mid : q == 6 ? sl[2 * (BV + 1) + 1] : sl[(q / 2) * (BV + 1) + (q & 1)];
    }
    __syncthreads();

    // A slice's entries are read again in every iteration: a workgroup with one
    // slice keeps them in LDS where they fit, the rows first, behind the copied
    // rows of t.  Set up before the first iteration of a round (a residual
    // pass in float64 uses the same LDS).  A smaller team adds the rows of
    // slices that would fit in the same order, from memory.
    Kept<T> keptA, keptAt;
    auto t_bytes = [&](int s) { return (cuts[s][15] * (int64_t)sizeof(T) + 15) / 16 * 16; };
    auto fits = [&](int s, int64_t &at, int64_t &na) {   // bit 0: the rows, bit 1: the columns
      const int64_t *cut = cuts[s];
      na = team_kept_bytes(cut[1] - cut[0] + cut[3] - cut[2] + cut[6] - cut[4], tv.entries[2 * (bV + s)], sizeof(T), true);
      const int64_t nat = team_kept_bytes(cut[8] - cut[7] + cut[10] - cut[9] + cut[13] - cut[11],
                                          tv.entries[2 * (bV + s) + 1], sizeof(T), false);
      at = t_bytes(s) <= tv.cap ? t_bytes(s) : 0;
      if (at + na > tv.cap || n > 65536) return 0;
      return t_bytes(s) > tv.cap || at + na + nat > tv.cap ? 1 : 3;
    };
    auto keep_slice = [&]() {
      if ((int)tm.size != V || keptA.on) return;
      const int s = tm.rank;
      int64_t at, na;
      const int kept = fits(s, at, na);
      if (kept == 0) return;
      const int32_t ea = tv.entries[2 * (bV + s)], eat = tv.entries[2 * (bV + s) + 1];
      keptA.place(tv.cap_off + at, cuts[s], ea, true);
      keptA.template fill<true>(cuts[s], ea, v.rowsA, v.spanA, tv.keptA, v.A_col, v.A_val, rho_hat, n0,
                                [&](int32_t r) { return DMP > 0 && v.drow && v.drow[r] >= 0 ? ~r : r; });
      if (kept == 1) return;
      keptAt.place(tv.cap_off + at + na, cuts[s] + 7, eat, false);
      keptAt.template fill<false>(cuts[s] + 7, eat, v.rowsAt, v.spanAt, tv.keptAt, tv.At_loc, v.At_val, rho_hat, 0,
                                  [](int32_t j) { return j; });
    };
    // a fitting slice's rows from memory: emit(id, sum) on a row's first lane
    auto strided_from_memory = [&](auto zero, const int64_t *cut, const int32_t *rows, const RowSpan *span,
                                   const auto *col, const T *val, auto vin, auto emit) {
      using AT = decltype(zero);
      int32_t end[4];
      class_ends(cut, end);
      strided_rows(end, [&](auto lanes, int q) {
        constexpr int L = decltype(lanes)::value;
        const int64_t li = list_at(cut, end, q);
        const RowSpan sp = span[li];
        const AT acc = strided_sum<L, AT>((int)(sp.k1 - sp.kb), [&](int k) { return val[sp.kb + k]; },
                                          [&](int k) { return vin[col[sp.kb + k]]; });
        if (threadIdx.x % L == 0) emit(rows[li], acc);
      });
    };

    // this workgroup's columns of slice s
    auto own = [&](int s, auto f) {
      for (int64_t j = cuts[s][16] + tid; j < cuts[s][17]; j += NTH) f(j);
    };
    auto sum_set = [&](int k, int s, double val) {
      if (tid == 0) tm.rec->sum[tm.parity][k][s] = val;
    };
    // LDS copy of a vector the team's members wrote; f(old LDS value, new entry)
    auto fill = [&](const T *src, auto f) {
      const Shared<T> sv{src + n0};
      for (int j = tid; j < n; j += 8 * NTH) {   // past the end: the last entry again, not stored
        T e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = sv[min(j + u * NTH, n - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (j + u * NTH < n) pl[j + u * NTH] = f(pl[j + u * NTH], e[u]);
      }
      __syncthreads();
    };
    // All length classes of one slice's rows.  A team has few rows per lane
    // group, so the time is the dependent loads of the rows one after another:
    // few lanes per row, all of a row's pieces in flight at once.
    auto class_rows_of = [&](auto zero, const int32_t *rows, const RowSpan *span, const int64_t *cut,
                             const auto *col, const T *val, auto vin, auto emit) {
      using AT = decltype(zero);
      constexpr int U = 16 / sizeof(AT);
      row_pass<1, AT>(rows, span, cut[0], cut[1], tid, NTH, col, val, vin, all, emit);
      row_pass<4, AT, U>(rows, span, cut[2], cut[3], tid / 4, NTH / 4, col, val, vin, all, emit);
      row_pass<8, AT, U>(rows, span, cut[4], cut[5], tid / 8, NTH / 8, col, val, vin, all, emit);
      row_pass<64, AT>(rows, span, cut[5], cut[6], tid / 64, NTH / 64, col, val, vin, all, emit);
    };
    // The dense blocks' column products of slice s's columns, summed over the
    // slices in order, into dl (by place among the slice's dense columns, of
    // which dl has room for the most a slice has): half a wave per column.
    auto dense_columns = [&](int s) {
      const int32_t *list = tv.dense_list + cuts[s][18];
      const int cnt = (int)(cuts[s][19] - cuts[s][18]);
      const int lane = tid % 32;
      for (int base = 0; base < cnt; base += 4 * (NTH / 32)) {
        int32_t e[4];
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = base + u * (NTH / 32) + tid / 32;
          e[u] = k < cnt ? list[k] : -1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          x[u] = e[u] >= 0 && lane < V ? Shared<double>{tv.ecp + (int64_t)lane * tv.ec_stride}[e[u]] : 0.0;
#pragma unroll
        for (int off = 16; off > 0; off >>= 1)
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] += __shfl_xor(x[u], off, 64);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (e[u] >= 0 && lane == 0) dl[base + u * (NTH / 32) + tid / 32] = x[u];
      }
      __syncthreads();
    };
    // Row half: tt = rho_hat o (A p) on this workgroup's slices, sums in AT;
    // rows of dense blocks are completed there and give the slice's G'w.
    // term((A p)_i, tt_i) is called once per row, done(s) after each slice.
    auto rows_half = [&](auto zero, auto *tt, auto term, auto done) {
      using AT = decltype(zero);
      constexpr bool ITER = !std::is_same<decltype(term), NoTerm>::value;   // an iteration, not the residual
      for (int s = tm.rank; s < V; s += tm.size) {
        auto emit = [&](int32_t i, AT acc) {
          if (v.drow && v.drow[i] >= 0) {
            tt[i] = acc;
          } else {
            const AT w = (AT)rho_hat[i] * acc;
            tt[i] = w;
            term(acc, w);
          }
        };
        int64_t at, na;
        if (ITER && keptA.on) {
          strided_rows(keptA.end, [&](auto lanes, int q) {
            constexpr int L = decltype(lanes)::value;
            const AT acc = keptA.template row_sum<L, AT>(q, pl);
            if (tid % L == 0) {
              const int32_t i = keptA.row()[q];
              if (DMP > 0 && i < 0) {
                tt[~i] = acc;
              } else {
                const AT w = (AT)keptA.rho()[q] * acc;
                tt[i] = w;
                term(acc, w);
              }
            }
          });
        } else if (ITER && (int)tm.size != V && fits(s, at, na) != 0) {
          strided_from_memory((AT)0, cuts[s], v.rowsA, v.spanA, v.A_col, v.A_val, pv, emit);
        } else {
          class_rows_of((AT)0, v.rowsA, v.spanA, cuts[s], v.A_col, v.A_val, pv, emit);
        }
        if constexpr (DMP > 0) {
          __syncthreads();   // the CSR part of the slice's dense rows
          for (int k = v.dense_inst[b]; k < v.dense_inst[b + 1]; ++k) {
            const DenseDesc &d = v.dense[k];
            const int rb = (int)((int64_t)d.rows * s / V), re = (int)((int64_t)d.rows * (s + 1) / V);
            const T *vd = pl + (d.col0 - n0);
            dense_block_fused<NTH, DMP, AT, TG>(d, rb, re, rho_hat, [&](int c) { return vd[c]; }, tt,
                                                reinterpret_cast<AT *>(dl), tv.ecp + (int64_t)s * tv.ec_stride, term);
          }
        }
        done(s);
      }
    };
    // (P p + sigma p)_j, added to acc
    auto col_diag = [&](auto acc, int64_t j) {
      using AT = decltype(acc);
      if (v.P_rowptr)
        for (int64_t k = v.P_rowptr[j]; k < v.P_rowptr[j + 1]; ++k) acc += (AT)v.P_val[k] * (AT)pv[v.P_col[k]];
      return acc + (AT)v.sigma * (AT)pv[j];
    };
    // that and the dense blocks' part of (A' t)_j, added to the column half's
    // sum where the column's owner reads it (all loads of a column
    // independent, none behind the sum)
    auto col_rest = [&](auto acc, int64_t j) {
      using AT = decltype(acc);
      if constexpr (DMP > 0) {
        const int32_t q = tv.dense_slot[j];
        if (q >= 0) acc += (AT)dl[q];
      }
      return col_diag(acc, j);
    };
    // Column half: emit(j, (CSR part of A' tt)_j) on this workgroup's slices.
    auto cols_half = [&](bool iter, auto zero, auto *tt, auto emit) {
      using AT = decltype(zero);
      const Shared<AT> tsh{tt};
      for (int s = tm.rank; s < V; s += tm.size) {
        const int64_t i0 = cuts[s][14];
        const int cnt = (int)cuts[s][15];
        if (cnt * (int64_t)sizeof(AT) <= tv.cap) {
          AT *tc = reinterpret_cast<AT *>(tl);
          if (sizeof(AT) != sizeof(T)) {   // wider than the place left for it
            __syncthreads();
            keptA.on = keptAt.on = false;
          }
          auto copy = [&](auto entry) {
            for (int i = tid; i < cnt; i += 4 * NTH) {
              AT e[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) e[u] = entry(min(i + u * NTH, cnt - 1));
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (i + u * NTH < cnt) tc[i + u * NTH] = e[u];
            }
          };
          if (i0 >= 0) {
            const Shared<AT> src{tt + i0};
            copy([&](int k) { return src[k]; });
          } else {
            const int32_t *list = tv.uses + (-1 - i0);
            copy([&](int k) { return tsh[list[k]]; });
          }
          __syncthreads();
          int64_t at, na;
          if (iter && keptAt.on)
            strided_rows(keptAt.end, [&](auto lanes, int q) {
              constexpr int L = decltype(lanes)::value;
              const AT acc = keptAt.template row_sum<L, AT>(q, tc);
              if (tid % L == 0) emit(keptAt.row()[q], acc);
            });
          else if (iter && (int)tm.size != V && (fits(s, at, na) & 2) != 0)
            strided_from_memory((AT)0, cuts[s] + 7, v.rowsAt, v.spanAt, tv.At_loc, v.At_val, Local<AT>{tc, 0}, emit);
          else
            class_rows_of((AT)0, v.rowsAt, v.spanAt, cuts[s] + 7, tv.At_loc, v.At_val, Local<AT>{tc, 0}, emit);
          __syncthreads();   // the next slice's copy may overwrite it
        } else {
          class_rows_of((AT)0, v.rowsAt, v.spanAt, cuts[s] + 7, v.At_col, v.At_val, tsh, emit);
        }
      }
      __syncthreads();   // the columns' results are read by other threads of this workgroup
    };

    for (int s = tm.rank; s < V; s += tm.size) {
      double bb = 0, dd = 0;
      own(s, [&](int64_t j) { bb += rhs[j] * rhs[j]; });
      wg_sum2<NTH>(bb, dd, redd);
      sum_set(0, s, bb);
    }
    double tot[3];
    {
      double one[1];
      team_sums<1>(tm, V, one, sum_s, &flag_s);
      tot[0] = one[0];
    }
    const double thr = (double)tol * (double)tol * tot[0];
    bool fail = !isfinite(tot[0]);
    int it = 0, passes = 0;
    double rrt = 0, rrt_prev = 0;
    for (int restart = 0; !tm.aborted; ++restart) {
      // true residual with float64 accumulation; z = r / diag M, p = z
      fill(x, [](T, T e) { return e; });
      rows_half(0.0, t64, NoTerm{}, [](int) {});
      team_sync(tm, &flag_s);
      cols_half(false, 0.0, t64, [&](int32_t j, double acc) { c64[j] = acc; });
      ++passes;
      for (int s = tm.rank; s < V; s += tm.size) {
        if constexpr (DMP > 0) dense_columns(s);
        T rz = 0, rr = 0;
        double rt = 0, dd = 0;
        own(s, [&](int64_t j) {
          const T rj = (T)(rhs[j] - col_rest(c64[j], j));
          r[j] = rj;
          const T zj = rj / dg[j];
          z[j] = zj;
          rz += rj * zj;
          rr += rj * rj;
          rt += (double)rj * (double)rj;
        });
        wg_sum2<NTH>(rz, rr, red);
        wg_sum2<NTH>(rt, dd, redd);
        sum_set(0, s, (double)rz);
        sum_set(1, s, (double)rr);
        sum_set(2, s, rt);
      }
      team_sums<3>(tm, V, tot, sum_s, &flag_s);
      T rz = (T)tot[0], rr = (T)tot[1];
      rrt = tot[2];
      fail = fail || !isfinite(rrt);
      const bool stalled = restart > 0 && rrt > STALL2 * rrt_prev;
      if (fail || rrt <= thr || it >= max_iter || restart > NRESTART || stalled || tm.aborted) break;
      rrt_prev = rrt;
      const T target = (T)(restart == 0 ? thr : fmax(thr, ROUND_DROP2 * (double)rr));
      fill(z, [](T, T e) { return e; });
      keep_slice();
      while (rr > target && it < max_iter) {
        // p'Mp = sum rho_hat (A p)^2 + p'(P p + sigma p): known with the row
        // half, so its sum needs no barrier of its own
        T pMp = 0;
        rows_half((T)0, t, [&](T ap, T w) { pMp += ap * w; },
                  [&](int s) {
                    T dummy = 0;
                    own(s, [&](int64_t j) { pMp += pl[j - n0] * col_diag((T)0, j); });
                    wg_sum2<NTH>(pMp, dummy, red);
                    sum_set(0, s, (double)pMp);
                    pMp = 0;
                  });
        double one[1];
        team_sums<1>(tm, V, one, sum_s, &flag_s);
        if (tm.aborted) break;
        pMp = (T)one[0];
        if (!(pMp > (T)0)) {   // breakdown: restart from the true residual (or fail if non-finite)
          fail = !isfinite(pMp);
          break;
        }
        const T a = rz / pMp;
        // this thread's first column: what its update reads is on its way
        // while the column half runs
        const int64_t jf = cuts[tm.rank][16] + tid;
        const bool has = jf < cuts[tm.rank][17];
        const T xf = has ? x[jf] : (T)0, rf = has ? r[jf] : (T)0, df = has ? dg[jf] : (T)1;
        cols_half(true, (T)0, t, [&](int32_t j, T acc) { Mp[j] = acc; });
        for (int s = tm.rank; s < V; s += tm.size) {
          if constexpr (DMP > 0) dense_columns(s);
          T rzn = 0, rrn = 0;
          own(s, [&](int64_t j) {
            const bool pre = j == jf;
            x[j] = (pre ? xf : x[j]) + a * pl[j - n0];
            const T rj = (pre ? rf : r[j]) - a * col_rest(Mp[j], j);
            const T zj = rj / (pre ? df : dg[j]);
            r[j] = rj;
            z[j] = zj;
            rzn += rj * zj;
            rrn += rj * rj;
          });
          wg_sum2<NTH>(rzn, rrn, red);
          sum_set(0, s, (double)rzn);
          sum_set(1, s, (double)rrn);
        }
        double two[2];
        team_sums<2>(tm, V, two, sum_s, &flag_s);
        if (tm.aborted) break;
        const T rz_new = (T)two[0];
        rr = (T)two[1];
        const T beta = rz_new / rz;
        rz = rz_new;
        fill(z, [beta](T p, T e) { return e + beta * p; });
        ++it;
        if (!isfinite(rr)) {
          fail = true;
          break;
        }
      }
      if (fail) break;
    }
    // A team that gives up: whichever of its members misses another, the one
    // that took the instance or a member that worked on it says so here or above.
    if (tm.aborted) {
      if (tid == 0) st_agent(&given_up[pos], 1u);
      break;
    }
    // ---- epilogue on this workgroup's columns --------------------------------------
    const T al = alpha_k ? alpha_k[b] : (T)1;
    for (int s = tm.rank; s < V; s += tm.size)
      own(s, [&](int64_t j) {
        if (fail) x[j] = (T)NAN;   // a non-finite system marks its solution, never a finite warm start
        if (mode == 0) {
          if (xnew) xnew[j] = al * x[j] + ((T)1 - al) * xold[j];
        } else {
          gx_out[j] = ((T)1 - al) * gx_in[j] + v.sigma * x[j];
        }
      });
    if (stats && tm.rank == 0 && tid == 0) {
      atomicMax(&stats[b].cg_iters_max, it);
      atomicAdd(&stats[b].cg_iters_total, it);
      atomicAdd(&stats[b].cg_passes_total, passes);
      if (!(rrt <= thr)) atomicAdd(&stats[b].cg_not_converged, 1);
    }
  }

  // ---- the last workgroup out: instances given up; control words left zero ----------
  if (tm.aborted) {   // what this workgroup stored is in memory before it counts as gone
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __syncthreads();
    if (tid == 0) {
      st_agent(&head->aborted, 1u);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    }
  }
  __syncthreads();
  if (tid == 0)
    flag_s = __hip_atomic_fetch_add(&head->exits, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (flag_s) {
    if (ld_agent(&head->aborted) != 0) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const uint32_t taken = ld_agent(&head->queue);
      for (uint32_t q = 0; q < (uint32_t)v.B; ++q) {
        if (q < taken && ld_agent(&given_up[q]) == 0) continue;
        const int b = tv.order[q];
        T *out = mode == 0 ? xnew : gx_out;
        for (int64_t j = v.n_off[b] + tid; j < v.n_off[b + 1]; j += NTH) {
          x[j] = (T)NAN;
          if (out) out[j] = (T)NAN;
        }
        if (stats && tid == 0) atomicAdd(&stats[b].cg_not_converged, 1);
      }
      __syncthreads();   // the words have been read
      for (int q = tid; q < v.B; q += NTH) st_agent(&given_up[q], 0);
    }
    for (int i = tid; i < TEAM_XCDS * tv.teams_per_xcd; i += NTH) {
      TeamRec &rec = recs[i];
      st_agent(&rec.joined, 0);
      st_agent(&rec.size, 0);
      st_agent(&rec.abort, 0);
      st_agent(&rec.count, 0);
      st_agent(&rec.gen, 0);
    }
    for (int i = tid; i < TEAM_XCDS; i += NTH) st_agent(&head->ticket[64 * i], 0);
    if (tid == 0) {
      st_agent(&head->queue, 0);
      st_agent(&head->exits, 0);
      st_agent(&head->aborted, 0);
    }
  }
}

// Zeroes the control words (once per call of an unroll; a solve leaves them zero).
__global__ __launch_bounds__(256) void k_team_reset(uint32_t *words, int64_t n) {
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) words[i] = 0;
}

}  // namespace

size_t team_state_bytes(int32_t teams_per_xcd, int32_t B) {
  return sizeof(TeamHead) + (size_t)TEAM_XCDS * teams_per_xcd * sizeof(TeamRec) + ((size_t)B + 1) / 2 * 8;
}

void launch_team_reset(const TeamView &tv, int32_t B, hipStream_t st) {
  const int64_t n = (int64_t)team_state_bytes(tv.teams_per_xcd, B) / 4;
  k_team_reset<<<(int)std::min<int64_t>((n + 255) / 256, 64), 256, 0, st>>>(static_cast<uint32_t *>(tv.state), n);
}

// Dynamic LDS of a workgroup: the longest instance's vector, and one region
// for the waves' partials of the dense product (float64 in the residual pass)
// and for the sums of a slice's dense columns.
size_t team_lds_bytes(size_t esz, int64_t max_n, int32_t dense_maxcols, int32_t dense_slots) {
  const int64_t dense = std::max<int64_t>((int64_t)(NTH / 64) * dense_maxcols, dense_slots);
  return (size_t)(max_n * (int64_t)esz + 7) / 8 * 8 + (size_t)dense * 8;
}

template <typename T>
void launch_pcg_team(const View<T> &v, const TeamView &tv, const T *rho_hat, const T *dg, const double *rhs, T *x, T *r,
                     T *z, T *Mp, T *t, double *t64, double *c64, double tol, int32_t max_iter, const T *alpha_k,
                     const T *xold, T *xnew, const T *gx_in, T *gx_out, int32_t mode, cosmo_stats *stats,
                     hipStream_t st) {
  TeamView tvl = tv;
  tvl.cap_off = (int64_t)(team_lds_bytes(sizeof(T), tv.max_n, v.n_dense > 0 ? v.dense_maxcols : 0, tv.dense_slots) + 15) / 16 * 16;
  auto go = [&](auto kern) {
    (void)allow_dyn_lds(reinterpret_cast<const void *>(kern));
    kern<<<tv.grid, NTH, tvl.cap_off + tv.cap, st>>>(v, tvl, rho_hat, dg, rhs, x, r, z, Mp, t, t64, c64, (T)tol,
                                                         max_iter, alpha_k, xold, xnew, gx_in, gx_out, mode, stats);
  };
  if (v.n_dense <= 0) {
    go(&k_pcg_team<T, 0, T>);
    return;
  }
  auto pick = [&](auto tg) {
    using TG = decltype(tg);
    constexpr int VE = 16 / sizeof(TG), MAXPC = COSMO_DENSE_MAX_COLS / (64 * VE);
    const int pieces = (v.dense_maxcols + 64 * VE - 1) / (64 * VE);
    if (pieces <= MAXPC / 4) go(&k_pcg_team<T, MAXPC / 4, TG>);
    else if (pieces <= MAXPC / 2) go(&k_pcg_team<T, MAXPC / 2, TG>);
    else go(&k_pcg_team<T, MAXPC, TG>);
  };
  if (sizeof(T) == 8 && v.dense_g32) pick(float{});
  else pick(T{});
}

#define INST(T)                                                                                                        \
  template void launch_pcg_team<T>(const View<T> &, const TeamView &, const T *, const T *, const double *, T *, T *, \
                                   T *, T *, T *, double *, double *, double, int32_t, const T *, const T *, T *,     \
                                   const T *, T *, int32_t, cosmo_stats *, hipStream_t);
INST(float)
INST(double)

}  // namespace cosmo
