// Persistent propagation on the site-operator form (parity.h): one launch runs
// every step, exponential and Lanczos iteration of a call, on one workgroup
// or on a team of workgroups that share one XCD.
//
// Block b of a team owns 2^tl consecutive rows; thread t the rows t + r T of
// them.  u_k of the block's rows is in LDS: a term that flips only low row bits
// is an LDS read, a DPP lane move or another register of the same thread.  Every
// thread keeps, in registers and for the whole launch, the LDS address and the
// value of each term on its rows and its rows' diagonal: no matrix is read, and
// a term costs its read and its multiply-adds.  (Decoding a table of terms in
// every iteration, from LDS or by v_readlane, cost 100 to 250 cycles a term.  Where
// the terms are too many for the registers, plan_site says which shapes, they
// spill.)
// The recurrence is the pipelined one of persistent.hip,
//     u_k = (z_{k-1} - alpha_{k-1} u_{k-1}) / nu_{k-1} - (nu_{k-1} / nu_{k-2}) u_{k-2},
// z_k = H_w u_k, alpha_k = <u_k, z_k> / nu_k^2, nu_k = ||u_k||.
//
// What bounds it is the chain of one iteration, not bandwidth.  A team
// exchanges once per iteration, through the L2 its workgroups share: every block
// publishes its part of z_k and, after that, its partial sums, each with a tag;
// the others poll the tags and gather the z_k that terms flipping high bits
// need.  u_{k-1} and u_{k-2} of those rows are running copies that each thread
// forms itself with the owner's fused multiply-adds.  Stores are ordinary (they
// reach the XCD's L2), loads of other blocks' data carry the device-scope
// policy, which passes the CU's own cache; the tags grow over all launches, so
// nothing is reset.  An exchange with its gathers takes 1.0 us (8 blocks) to
// 1.1 us (32) this way, 2.1 to 2.7 us with device-scope stores.
//
// The launch is cooperative with eight times the team's blocks, so that every
// XCD holds a whole team; the blocks publish the XCD they run on, the first
// XCD with enough blocks does the work and the others leave.  If none has
// enough, the first blocks of the grid form the team and exchange with
// device-scope stores.  Every wait is bounded by a wall-clock limit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <type_traits>

#include "parity.h"
#include "sweep_common.hpp"
#include "tridiag.hpp"

namespace cfet {

namespace {

constexpr int kCpolDevice = 16;  // cache-policy operand: device scope

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           0x00020000);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// element i of a vector of n elements, past the CU's cache
__device__ __forceinline__ double2 shared_load(const double2* base, uint32_t i, uint32_t n) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc(base, n * 16u), (int)(i * 16u), 0,
                                                        kCpolDevice);
  return make_double2(__hiloint2double((int)v[1], (int)v[0]),
                      __hiloint2double((int)v[3], (int)v[2]));
}

template <int CS>
__device__ __forceinline__ void shared_store(double2* base, uint32_t i, uint32_t n, double2 x) {
  u32x4 v;
  v[0] = (unsigned)__double2loint(x.x);
  v[1] = (unsigned)__double2hiint(x.x);
  v[2] = (unsigned)__double2loint(x.y);
  v[3] = (unsigned)__double2hiint(x.y);
  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc(base, n * 16u), (int)(i * 16u), 0, CS);
}

// A value and its tag: 16 bytes, stored and loaded whole.
struct Rec {
  double v;
  unsigned long long tag;
};

template <int CS>
__device__ __forceinline__ void rec_store(Rec* base, int i, double x, unsigned long long tag) {
  u32x4 v;
  v[0] = (unsigned)__double2loint(x);
  v[1] = (unsigned)__double2hiint(x);
  v[2] = (unsigned)tag;
  v[3] = (unsigned)(tag >> 32);
  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc(base, kSiteRecs * 16u), i * 16, 0, CS);
}

// Waits until record l of `base` carries `tag` for every active lane (lane's
// record: l); false after `limit` ticks.  v: the lane's value.
__device__ __forceinline__ bool rec_wait(const Rec* base, bool active, int l,
                                         unsigned long long tag, long long limit, double& v) {
  const long long t0 = wall_clock64();
  for (int spin = 0;; ++spin) {
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc(base, kSiteRecs * 16u),
                                                          (active ? l : 0) * 16, 0, kCpolDevice);
    const unsigned long long got = (unsigned long long)q[2] | ((unsigned long long)q[3] << 32);
    v = active ? __hiloint2double((int)q[1], (int)q[0]) : 0.0;
    asm volatile("" ::: "memory");  // every round loads; later loads stay behind
    if (__ballot(active && got != tag) == 0ull) return true;
    if ((spin & 15) == 15 && wall_clock64() - t0 > limit) return false;
  }
}

// Block barrier for data in LDS: waits for this wavefront's LDS operations, not
// for its stores to memory.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The same after all of the wavefront's memory operations are done.
__device__ __forceinline__ void full_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Sums of a and b over the 64 lanes in a fixed order: lane 31 gets a's, lane 63
// b's.  The two halves of the wavefront take one sum each after the first step.
__device__ __forceinline__ double wave_sum2(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  double v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  v = w_step<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
  v = w_step<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
  v = w_step<0x141, 0xf>(v);  // row_half_mirror
  v = w_step<0x140, 0xf>(v);  // row_mirror
  return w_step<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
}

// The block's two sums from the W wavefronts' (at most 8), in a fixed order;
// every lane gets them.
template <int W>
__device__ __forceinline__ void block_sums(const double (*red)[8], int lane, double& a,
                                           double& b) {
  static_assert(W <= 8, "one row of eight per sum");
  double v = (lane & 7) < W ? red[(lane >> 3) & 1][lane & 7] : 0.0;
  if (W > 1) v = w_step<0xB1, 0xf>(v);
  if (W > 2) v = w_step<0x4E, 0xf>(v);
  if (W > 4) v = w_step<0x141, 0xf>(v);
  a = lane_read(v, 0);
  b = lane_read(v, 8);
}

// x of the lane whose index differs by the flips that CTRL stands for
template <int CTRL>
__device__ __forceinline__ double2 lane_move(double2 x) {
  auto mv = [](int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false); };
  return make_double2(__hiloint2double(mv(__double2hiint(x.x)), mv(__double2loint(x.x))),
                      __hiloint2double(mv(__double2hiint(x.y)), mv(__double2loint(x.y))));
}

// How the terms are divided (SitePlan): kOneSet, all off-diagonal terms of one
// operator term (a driven sum, or H0's); kTwoSets, a driven operator term (set
// 0) and H0 (set 1), summed apart and weighted at the end; kWeighted, several
// driven terms, all in set 0 and weighted at the start of each exponential.
enum SiteMode { kOneSet = 0, kTwoSets = 1, kWeighted = 2 };

constexpr int log2_of(int t) { return t <= 1 ? 0 : 1 + log2_of(t / 2); }

// A set's slots, in the order of its terms in the table: moves (set 0: flips 1,
// 2 and 8; set 1: flip 3), LDS terms, flips of the register index alone (mask
// 1 .. R - 1), in set 1 a term that flips it with thread bits, and terms that
// leave the block.  Absent terms hold value 0.
template <int T, int R, int MODE, int NF>
struct Slots {
  static constexpr bool kTwo = MODE == kTwoSets;
  static constexpr int mv(int set) { return set == 0 ? 3 : kTwo ? 1 : 0; }
  static constexpr int lds(int set) {
    return set == 0 ? log2_of(T) - 3 : kTwo ? log2_of(T) - 2 : 0;
  }
  static constexpr int reg(int set) { return set == 0 || kTwo ? R - 1 : 0; }
  static constexpr int mix(int set) { return set == 1 && kTwo && R > 1 ? 1 : 0; }
  static constexpr int far(int set) { return set == 0 || kTwo ? NF : 0; }
  static constexpr int count(int set) {
    return mv(set) + lds(set) + reg(set) + mix(set) + far(set);
  }
};

// The value of one term on a row: the parity picked, the parts not yet
// weighted (kWeighted: two, of different operator terms).
template <bool RV, bool TWO_PARTS>
struct TermValue {
  double a, ai, b, bi;
  __device__ __forceinline__ void set(const PElem& e, uint32_t row) {
    const bool p = __popc(row & e.pmask) & 1;
    a = p ? e.v1 : e.v0;
    ai = p ? e.w1 : e.w0;
    b = p ? e.b1 : e.b0;
    bi = p ? e.d1 : e.d0;
  }
  __device__ __forceinline__ dv2 get(double w, double w2) const {
    if (!TWO_PARTS) return dv2{a, RV ? 0.0 : ai};
    return dv2{fma(w2, b, w * a), RV ? 0.0 : fma(w2, bi, w * ai)};
  }
};

struct SiteShared {
  double cheb[kChebMaxTerms];
  double red[2][8];
  double s1[kMaxM], s2[kMaxM];  // the phases' sums
  double2 coef[kMaxM];
  int hist[16];
  int rank, bad;
  unsigned long long launch;
};

// Segment timer (block of rank 0, thread 0): products, reductions, small
// exponentials, recombinations.
struct SiteTimer {
  long long last = 0, acc[4] = {0, 0, 0, 0};
  bool on = false;
  __device__ void start(bool enable) {
    on = enable;
    if (on) last = wall_clock64();
  }
  __device__ void lap(int seg) {
    if (!on) return;
    const long long t = wall_clock64();
    acc[seg] += t - last;
    last = t;
  }
};

// The same fused multiply-adds wherever u_k of a row is formed, so that every
// block holds the same bits.
__device__ __forceinline__ double2 form_u(double2 z, double2 u1, double2 u2, double c1, double c2,
                                          double c3) {
  return make_double2(fma(c1, z.x, fma(-c2, u1.x, -c3 * u2.x)),
                      fma(c1, z.y, fma(-c2, u1.y, -c3 * u2.y)));
}

// A wait of this launch has timed out: latch a device error, in the statistics
// and in their pinned copy, which the next call on the context looks at.
__device__ __forceinline__ void report_fault(const SiteArgs& A) {
  __hip_atomic_store(&A.p.stats->status, (int)CFET_EDEVICE, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  if (A.p.stats_out)
    __hip_atomic_store(&A.p.stats_out->status, (int)CFET_EDEVICE, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// The statistics to their pinned copy (one thread of a launch).  The host
// clears the copy's status; here it is only ever set, so that a fault another
// block reports at the same time stays.
__device__ __forceinline__ void publish_stats(const SiteArgs& A) {
  DevStats* const st = A.p.stats;
  DevStats* const out = A.p.stats_out;
  if (!out) return;
  out->exponentials = st->exponentials;
  out->matvecs = st->matvecs;
  out->min_m_eff = st->min_m_eff;
  out->breakdowns = st->breakdowns;
  out->last_norm2 = st->last_norm2;
  for (int q = 0; q < 4; ++q) out->seg[q] = st->seg[q];
  const int status =
      __hip_atomic_load(&st->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (status != CFET_OK)
    __hip_atomic_store(&out->status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The work of one block.  NF: terms of a set that leave the block, at most (0:
// one block); CS: cache policy of the stores that other blocks read.
template <int T, int R, int MODE, int NF, bool RV, int CS>
__device__ __forceinline__ void site_run(const SiteArgs& A, int rank, double2* xt,
                                         SiteShared& sh) {
  using Sl = Slots<T, R, MODE, NF>;
  constexpr int W = T / 64;
  constexpr bool TEAM = NF > 0;
  constexpr bool WTD = MODE == kWeighted;
  constexpr int NS = MODE == kTwoSets ? 2 : 1;
  const int t = threadIdx.x;
  const int wv = t >> 6, lane = t & 63;
  const uint32_t n = (uint32_t)A.p.n;
  const uint32_t row0 = ((uint32_t)rank << A.tl) + (uint32_t)t;
  const bool act = (uint32_t)t < n;  // fewer rows than threads: one block, R = 1
  const int NB = A.blocks;
  const int nt1 = A.p.nterms + 1;
  double2* const psi = A.p.psi;
  uint32_t qb = (uint32_t)(uintptr_t)(lds_cptr)xt + ((uint32_t)t << 4);
  asm volatile("" : "+v"(qb));

  // ---- the terms on this thread's rows
  using Val = TermValue<RV, WTD>;
  constexpr int NV0 = Sl::mv(0) + Sl::lds(0), NV1 = NS > 1 ? Sl::mv(1) + Sl::lds(1) : 1;
  Val tv[NS][NV0 > NV1 ? NV0 : NV1];          // moves and LDS terms
  uint32_t ta[NS][NV0 > NV1 ? NV0 : NV1];     // LDS addresses
  constexpr int NRG = R > 1 ? R - 1 : 1;
  Val rv[NS][NRG][R];                         // register flips, per row
  constexpr int NG = TEAM ? NF : 1;
  Val xv[R];                                  // the mixed term
  uint32_t xa = qb;
  Val fv[NS][NG][R];                          // terms that leave the block
  uint32_t fo[NS][NG];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const PElem* e = A.e + (s == 0 ? 0 : Sl::count(0));
#pragma unroll
    for (int i = 0; i < Sl::mv(s) + Sl::lds(s); ++i) {
      tv[s][i].set(e[i], row0);
      ta[s][i] = qb ^ (e[i].off << 4);
    }
    e += Sl::mv(s) + Sl::lds(s);
    if constexpr (R > 1) {
#pragma unroll
      for (int m = 0; m < R - 1; ++m)
#pragma unroll
        for (int r = 0; r < R; ++r) rv[s][m][r].set(e[m], row0 + (uint32_t)(r * T));
      e += R - 1;
      if (Sl::mix(s)) {
#pragma unroll
        for (int r = 0; r < R; ++r) xv[r].set(e[0], row0 + (uint32_t)(r * T));
        xa = qb ^ ((e[0].off & (uint32_t)(T - 1)) << 4);
        e += 1;
      }
    }
    if constexpr (TEAM) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        fo[s][f] = e[f].off;
#pragma unroll
        for (int r = 0; r < R; ++r) fv[s][f][r].set(e[f], row0 + (uint32_t)(r * T));
      }
    }
  }
  double dg[R];
  double2 u1[R], u2[R], zp[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    dg[r] = (A.diag && act) ? A.diag[row0 + (uint32_t)(r * T)] : 0.0;
    u1[r] = act ? psi[row0 + (uint32_t)(r * T)] : make_double2(0.0, 0.0);
    u2[r] = zp[r] = make_double2(0.0, 0.0);
  }
  // rows of the terms that leave the block: running copies of u_{k-1} (g1) and
  // u_{k-2} (g2), and the gathered z_{k-1} (gz)
  double2 g1[NS][NG][R], g2[NS][NG][R], gz[NS][NG][R];
  auto gather = [&](const double2* base, double2 (*g)[NG][R]) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int f = 0; f < NG; ++f)
#pragma unroll
        for (int r = 0; r < R; ++r)
          g[s][f][r] = shared_load(base, (row0 + (uint32_t)(r * T)) ^ fo[s][f], n);
  };
  // Tags grow by one per exchange.  The sums use two sets of records in turn: a
  // block may post its next sums while another still reads the last ones, but
  // not the ones after (those need every block's next sums, posted after the
  // last ones were read).  z_k uses two buffers in the same way.  The tag of psi
  // is posted once per exponential, with exchanges of sums between.
  unsigned long long tag_s = sh.launch << 32, tag_u = tag_s;
  auto rec_s = [&](unsigned long long tag) {
    return static_cast<Rec*>(A.rec) + (tag & 1) * kSiteRecs;
  };
  Rec* const rec_u = static_cast<Rec*>(A.rec) + 2 * kSiteRecs;
  unsigned long long expo = 0, mv = 0;
  int minm = 1 << 30, brk = 0, status = CFET_OK;
  SiteTimer tm;
  tm.start(A.p.timing != 0 && rank == 0 && t == 0);
  bool ok = true;
  for (int64_t sq = 0; ok && sq < A.p.nsteps; ++sq) {
    const int64_t step = A.p.rev ? A.p.nsteps - 1 - sq : sq;
    for (int iq = 0; ok && iq < A.p.s; ++iq) {
      const int i = A.p.rev ? iq : A.p.s - 1 - iq;
      const int64_t eidx = step * A.p.s + (A.p.s - 1 - i);
      const double* const wts = (A.inline_w ? A.w : A.p.wts) + ((size_t)step * A.p.s + i) * nt1;
      // the sets' weights and the diagonal's
      const double ws0 = WTD ? 1.0 : wts[A.set_term[0]];
      const double ws1 = NS > 1 ? wts[A.set_term[1]] : 0.0;
      const double wd = A.diag ? wts[A.diag_term] : 0.0;
      // values as the products use them (kWeighted: weighted now)
      auto part = [&](const Val& v, int slot) -> dv2 {
        if (!WTD) return v.get(1.0, 1.0);
        return v.get(wts[A.e[slot].term], wts[A.e[slot].term2]);
      };
      dv2 w_t[NS][NV0 > NV1 ? NV0 : NV1], w_r[NS][NRG][R], w_x[R], w_f[NS][NG][R];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        int slot = s == 0 ? 0 : Sl::count(0);
#pragma unroll
        for (int q = 0; q < Sl::mv(s) + Sl::lds(s); ++q) w_t[s][q] = part(tv[s][q], slot++);
        if constexpr (R > 1) {
#pragma unroll
          for (int q = 0; q < R - 1; ++q, ++slot)
#pragma unroll
            for (int r = 0; r < R; ++r) w_r[s][q][r] = part(rv[s][q][r], slot);
          if (Sl::mix(s)) {
#pragma unroll
            for (int r = 0; r < R; ++r) w_x[r] = part(xv[r], slot);
            ++slot;
          }
        }
        if constexpr (TEAM) {
#pragma unroll
          for (int q = 0; q < NF; ++q, ++slot)
#pragma unroll
            for (int r = 0; r < R; ++r) w_f[s][q][r] = part(fv[s][q][r], slot);
        }
      }
      const int m = A.p.m;
      int meff = m;
      // where u_1 is kept; the later ones follow
      auto first = [&]() -> double2* {
        return A.p.basis + (A.p.basis_each ? ((size_t)eidx * m + 1) * n : 0);
      };
      double2* uk = first() + row0;
      bool zero = false;
      double scale = 0.0, alpha_prev = 0.0, inv_prev = 0.0;
      double S1 = 0.0, S2 = 0.0;
      LzScalars* const XT =
          (A.p.export_T && A.p.export_each) ? A.p.export_T + eidx : A.p.export_T;
      double2* const XY = (A.p.export_Y && A.p.export_each)
                              ? A.p.export_Y + (size_t)eidx * (size_t)m * (size_t)n
                              : A.p.export_Y;
      if (A.p.basis_each && act) {
#pragma unroll
        for (int r = 0; r < R; ++r) (uk - n)[r * T] = u1[r];
      }
      if (A.p.save && act) {
#pragma unroll
        for (int r = 0; r < R; ++r) A.p.save[eidx * n + row0 + (uint32_t)(r * T)] = u1[r];
      }
      if (TEAM) {
        // u_0 = psi of the other blocks, once all have written it
        if (sq + iq > 0 && !A.p.no_combine) {
          double v;
          if (!rec_wait(rec_u, lane < NB, lane, tag_u, A.p.spin_limit, v)) sh.bad = 1;
        }
        gather(psi, g1);
      }
      for (int k = 0; k <= m; ++k) {
        double c1 = 0.0, c2 = 0.0, c3 = 0.0, nu = 0.0;
        bool stop = false;
        // early-stop rule and records of phase k - 1 (off the path to u_k)
        auto record = [&]() {
          if (k == 1) {
            zero = stop = (nu == 0.0);
          } else {
            scale = fmax(scale, fabs(alpha_prev) + nu);
            stop = (nu <= kBreakdownRel * scale);
            if (stop) meff = k - 1;
          }
          if (t == 0) {
            sh.s1[k - 1] = S1;
            sh.s2[k - 1] = S2;
          }
          alpha_prev = c2 * nu;
          inv_prev = c1;
        };
        if (k >= 1) {
          // ---- sums of phase k - 1
          if (TEAM) {
            double v;
            const int b = lane & 31;
            // lanes 0..31 the first sum of every block, lanes 32..63 the second
            if (!rec_wait(rec_s(tag_s), b < NB, (lane & 32) + b, tag_s, A.p.spin_limit, v))
              sh.bad = 1;
            if (k < m) gather(A.p.zbuf + (size_t)((k - 1) & 1) * n, gz);
            v = w_step<0xB1, 0xf>(v);
            v = w_step<0x4E, 0xf>(v);
            v = w_step<0x141, 0xf>(v);
            v = w_step<0x140, 0xf>(v);
            v = w_step<0x142, 0xa>(v);
            S1 = lane_read(v, 31);
            S2 = lane_read(v, 63);
          } else {
            block_sums<W>(sh.red, lane, S1, S2);
          }
          // (c1 * c1 would overflow for norms below 7e-155)
          c1 = rsqrt(S2);
          nu = S2 > 0.0 ? S2 * c1 : S2;
          c2 = S1 * c1 * c1 * c1;
          c3 = nu * inv_prev;
          if (k == m) {
            record();
            break;
          }
          tm.lap(1);
        }
        // ---- u_k on the own rows
        double2 uc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          uc[r] = k >= 1 ? form_u(zp[r], u1[r], u2[r], c1, c2, c3) : u1[r];
          xt[t + r * T] = uc[r];
        }
        lds_barrier();
        if (TEAM && sh.bad) {
          ok = false;
          break;
        }
        // ---- z_k = H_w u_k
        double2 acc[NS][R];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            double2 a = make_double2(0.0, 0.0);
            if (s == 0) {
              acc_fma<RV>(a, w_t[s][0], lane_move<0xB1>(uc[r]));   // quad_perm [1,0,3,2]
              acc_fma<RV>(a, w_t[s][1], lane_move<0x4E>(uc[r]));   // quad_perm [2,3,0,1]
              acc_fma<RV>(a, w_t[s][2], lane_move<0x128>(uc[r]));  // row_ror:8
            } else {
              acc_fma<RV>(a, w_t[s][0], lane_move<0x1B>(uc[r]));   // quad_perm [3,2,1,0]
            }
            acc[s][r] = a;
          }
          if constexpr (R > 1) {
#pragma unroll
            for (int q = 1; q < R; ++q)
#pragma unroll
              for (int r = 0; r < R; ++r) acc_fma<RV>(acc[s][r], w_r[s][q - 1][r], uc[r ^ q]);
            if (Sl::mix(s))
#pragma unroll
              for (int r = 0; r < R; ++r)
                acc_fma<RV>(acc[s][r], w_x[r], lds_at(xa + (r ^ 1) * T * 16));
          }
          // (with two rows, few loads at a time: more would spill registers)
          constexpr int Q = R == 1 ? 8 : MODE == kOneSet ? 3 : 2;
#pragma unroll
          for (int q0 = 0; q0 < Sl::lds(s); q0 += Q) {
            double2 x[Q][R];
#pragma unroll
            for (int q = 0; q < Q && q0 + q < Sl::lds(s); ++q)
#pragma unroll
              for (int r = 0; r < R; ++r)
                x[q][r] = lds_at(ta[s][Sl::mv(s) + q0 + q] + r * T * 16);
#pragma unroll
            for (int q = 0; q < Q && q0 + q < Sl::lds(s); ++q)
#pragma unroll
              for (int r = 0; r < R; ++r)
                acc_fma<RV>(acc[s][r], w_t[s][Sl::mv(s) + q0 + q], x[q][r]);
            if (R > 1) __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (k >= 1) {
          record();
          if (stop) break;
          if (act) {
#pragma unroll
            for (int r = 0; r < R; ++r) uk[r * T] = uc[r];
            uk += n;
          }
        }
        if constexpr (TEAM) {
#pragma unroll
          for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
#pragma unroll
              for (int r = 0; r < R; ++r) {
                double2 x = g1[s][f][r];
                if (k >= 1) {
                  x = form_u(gz[s][f][r], g1[s][f][r], g2[s][f][r], c1, c2, c3);
                  g2[s][f][r] = g1[s][f][r];
                  g1[s][f][r] = x;
                } else {
                  g2[s][f][r] = make_double2(0.0, 0.0);
                }
                acc_fma<RV>(acc[s][r], w_f[s][f][r], x);
              }
            }
        }
        double s_uz = 0.0, s_uu = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double d = wd * dg[r];
          double2 z = make_double2(fma(ws0, acc[0][r].x, d * uc[r].x),
                                   fma(ws0, acc[0][r].y, d * uc[r].y));
          if (NS > 1) {
            z.x = fma(ws1, acc[NS - 1][r].x, z.x);
            z.y = fma(ws1, acc[NS - 1][r].y, z.y);
          }
          if (XY && act) {
            // the driven term's part alone
            double2 y = A.set_term[0] == 1 ? acc[0][r] : make_double2(0.0, 0.0);
            if (A.diag_term == 1) {
              y.x = fma(dg[r], uc[r].x, y.x);
              y.y = fma(dg[r], uc[r].y, y.y);
            }
            XY[(size_t)k * (size_t)n + row0 + (uint32_t)(r * T)] = y;
          }
          if (TEAM && k + 1 < m)
            shared_store<CS>(A.p.zbuf + (size_t)(k & 1) * n, row0 + (uint32_t)(r * T), n, z);
          s_uz = fma(uc[r].x, z.x, fma(uc[r].y, z.y, s_uz));
          s_uu = fma(uc[r].x, uc[r].x, fma(uc[r].y, uc[r].y, s_uu));
          u2[r] = k >= 1 ? u1[r] : make_double2(0.0, 0.0);
          u1[r] = uc[r];
          zp[r] = z;
        }
        tm.lap(0);
        const double s2 = wave_sum2(s_uz, s_uu);
        if ((lane & 31) == 31) sh.red[lane >> 5][wv] = s2;
        if (TEAM) full_barrier();  // z_k is where the others read it
        else lds_barrier();
        if (TEAM) {
          ++tag_s;
          if (t < 64) {
            block_sums<W>(sh.red, lane, S1, S2);
            if (lane < 2) rec_store<CS>(rec_s(tag_s), lane * 32 + rank, lane == 0 ? S1 : S2, tag_s);
          }
        }
      }
      if (!ok) break;
      if (zero) {
        if (rank == 0 && t == 0) {
          expo += 1;
          brk += 1;
          minm = 0;
          if (XT) {
            XT->beta0 = 0.0;
            XT->m_eff = 0;
          }
        }
        lds_barrier();
        if (TEAM) {
          ++tag_u;
          if (t == 0) rec_store<CS>(rec_u, rank, 0.0, tag_u);
        }
        continue;
      }
      lds_barrier();
      // ---- projection and small exponential (wavefront 0; the same in every
      // block).  The path to u_k takes rsqrt(S2); the projection's entries are
      // formed here, all at once, with square roots and divisions (without them
      // the norm drifts twice as fast).  Errors against converged exponentials, mean of
      // 120 runs on 2^4 to 2^14 rows: 1.29e-15; 1.31e-15 with square roots and
      // divisions all along (persistent.hip).
      if (t < 64) {
        const double s2 = lane < meff ? sh.s2[lane] : 1.0;
        const double a = lane < meff ? sh.s1[lane] / s2 : 0.0;
        const double nrm = sqrt(s2);
        const double inv = 1.0 / nrm;
        const double nu0 = lane_read(nrm, 0);
        const double b = lane < meff - 1 ? sqrt(sh.s2[lane + 1]) : 0.0;
        if (XT && rank == 0) {
          if (lane < meff) {
            XT->alpha[lane] = a;
            XT->inv_nrm[lane] = inv;
          }
          if (lane < meff - 1) XT->beta[lane] = b;
          if (lane == 0) {
            XT->beta0 = nu0;
            XT->m_eff = meff;
          }
        }
        tm.lap(1);
        if (!A.p.no_combine) {
          double2 c = make_double2(0.0, 0.0);
          int rc;
          const bool bad = !(isfinite(a) && isfinite(b) && isfinite(nu0));
          if (__ballot(bad) != 0ull) rc = CFET_ENONFINITE;
          else rc = tridiag_exp_e1(a, b, meff, A.p.dt, sh.cheb, c);
          if (lane < meff) {
            const double scl = nu0 * inv;
            sh.coef[lane] = make_double2(c.x * scl, c.y * scl);
          }
          if (lane == 0 && rank == 0) {
            expo += 1;
            mv += (unsigned long long)meff;
            if (meff < minm) minm = meff;
            if (meff < m) brk += 1;
            if (rc != CFET_OK && status == CFET_OK) status = rc;
          }
        }
      }
      if (A.p.no_combine) continue;
      lds_barrier();
      tm.lap(2);
      // ---- recombination on the own rows
      if (act) {
        constexpr int Q = R >= 4 ? 4 : 8 / R;  // vectors whose loads are in flight together
        double2 sum[R];
#pragma unroll
        for (int r = 0; r < R; ++r) sum[r] = make_double2(0.0, 0.0);
        const double2* const uf = first();
        for (int k = 0; k < meff; k += Q) {
          double2 v[Q][R];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int kq = k + q < meff ? k + q : meff - 1;
            const double2* const b = kq == 0 ? psi : uf + (size_t)(kq - 1) * (size_t)n;
#pragma unroll
            for (int r = 0; r < R; ++r) v[q][r] = b[row0 + (uint32_t)(r * T)];
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            if (k + q >= meff) break;
            const double2 cf = sh.coef[k + q];
#pragma unroll
            for (int r = 0; r < R; ++r) {
              sum[r].x += cf.x * v[q][r].x - cf.y * v[q][r].y;
              sum[r].y += cf.x * v[q][r].y + cf.y * v[q][r].x;
            }
          }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          shared_store<CS>(psi, row0 + (uint32_t)(r * T), n, sum[r]);
          u1[r] = sum[r];
        }
      }
      if (TEAM) {
        full_barrier();  // psi is where the others read it
        ++tag_u;
        if (t == 0) rec_store<CS>(rec_u, rank, 0.0, tag_u);
      } else {
        lds_barrier();
      }
      tm.lap(3);
    }
  }
  lds_barrier();
  if (TEAM && sh.bad) ok = false;
  // ||psi||^2 after the last exponential, for the statistics
  if (ok && A.p.nsteps > 0) {
    double s1 = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) s1 = fma(u1[r].x, u1[r].x, fma(u1[r].y, u1[r].y, s1));
    const double s2 = wave_sum2(s1, s1);
    if ((lane & 31) == 31) sh.red[lane >> 5][wv] = s2;
    lds_barrier();
    double s0;
    block_sums<W>(sh.red, lane, s0, s1);
    if (TEAM) {
      ++tag_s;
      if (t < 2) rec_store<CS>(rec_s(tag_s), t * 32 + rank, s1, tag_s);
      if (rank == 0 && t < 64) {
        double v;
        ok = rec_wait(rec_s(tag_s), lane < NB, lane, tag_s, A.p.spin_limit, v);
        s1 = lane_read(w_sum63(v), 63);
      }
    }
    if (ok && rank == 0 && t == 0) A.p.stats->last_norm2 = s1;
  }
  if (rank == 0 && t == 0) {
    DevStats* const st = A.p.stats;
    if (expo) {
      st->exponentials += expo;
      st->matvecs += mv;
      if (minm < st->min_m_eff) st->min_m_eff = minm;
      st->breakdowns += brk;
      if (status != CFET_OK && st->status == CFET_OK) st->status = status;
    }
    if (tm.on)
      for (int q = 0; q < 4; ++q) st->seg[q] += tm.acc[q];
    publish_stats(A);
  }
  if (!ok && t == 0) report_fault(A);
}

template <int T, int R, int MODE, bool RV>
__global__ __launch_bounds__(T) void k_site_one(SiteArgs A) {
  extern __shared__ double2 xt[];
  SiteShared& sh = *reinterpret_cast<SiteShared*>(xt + T * R);
  if (threadIdx.x == 0) {
    sh.bad = 0;
    sh.launch = 0;
  }
  __syncthreads();
  site_run<T, R, MODE, 0, RV, 0>(A, 0, xt, sh);
}

template <int T, int R, int MODE, int NF, bool RV>
__global__ __launch_bounds__(T) void k_site_team(SiteArgs A) {
  extern __shared__ double2 xt[];
  SiteShared& sh = *reinterpret_cast<SiteShared*>(xt + T * R);
  const int t = threadIdx.x;
  const int G = gridDim.x;
  // the XCDs the blocks run on (tagged with the launch number, the same in
  // all of its blocks: the counter grows by the grid's size per launch)
  if (t == 0) {
    sh.bad = 0;
    sh.rank = 0;
    sh.launch = __hip_atomic_fetch_add(A.count, 1ull, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT) / (unsigned)G + 1ull;
  }
  if (t < 16) sh.hist[t] = 0;
  __syncthreads();
  const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;  // HW_REG_XCC_ID
  if (t == 0)
    __hip_atomic_store(A.ids + blockIdx.x, (sh.launch << 4) | xcc, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  for (int b = t; b < G; b += T) {
    const long long t0 = wall_clock64();
    unsigned long long v;
    for (int spin = 0;; ++spin) {
      v = __hip_atomic_load(A.ids + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((v >> 4) == sh.launch + A.skew) break;
      if ((spin & 15) == 15 && wall_clock64() - t0 > A.p.spin_limit) {
        sh.bad = 1;
        break;
      }
    }
    atomicAdd(&sh.hist[v & 15], 1);
    if ((unsigned)(v & 15) == xcc && b < (int)blockIdx.x) atomicAdd(&sh.rank, 1);
  }
  __syncthreads();
  if (sh.bad) {
    if (t == 0) report_fault(A);
    return;
  }
  int team = -1;
  for (int x = 15; x >= 0 && !A.spread; --x)
    if (sh.hist[x] >= A.blocks) team = x;
  if (team >= 0) {
    if ((int)xcc == team && sh.rank < A.blocks) 
      site_run<T, R, MODE, NF, RV, 0>(A, sh.rank, xt, sh);
  } else if ((int)blockIdx.x < A.blocks) {
    site_run<T, R, MODE, NF, RV, kCpolDevice>(A, blockIdx.x, xt, sh);
  }
}

// The launch shapes.  The host fills the table of terms by the slots of the
// shape it takes, so both come from here.
struct Shape {
  const void* fn = nullptr;
  int mv[2], lds[2], reg[2], mix[2], far[2];
};

template <int T, int R, int MODE, int NF>
Shape shape_of(bool real) {
  using Sl = Slots<T, R, MODE, NF>;
  Shape S;
  if constexpr (NF == 0)
    S.fn = real ? (const void*)&k_site_one<T, R, MODE, true>
                : (const void*)&k_site_one<T, R, MODE, false>;
  else
    S.fn = real ? (const void*)&k_site_team<T, R, MODE, NF, true>
                : (const void*)&k_site_team<T, R, MODE, NF, false>;
  for (int s = 0; s < 2; ++s) {
    S.mv[s] = Sl::mv(s);
    S.lds[s] = Sl::lds(s);
    S.reg[s] = Sl::reg(s);
    S.mix[s] = Sl::mix(s);
    S.far[s] = Sl::far(s);
  }
  return S;
}

template <int T, int R, int NF>
Shape shape_mode(int mode, bool real) {
  return mode == kOneSet    ? shape_of<T, R, kOneSet, NF>(real)
         : mode == kTwoSets ? shape_of<T, R, kTwoSets, NF>(real)
                            : shape_of<T, R, kWeighted, NF>(real);
}

// (no kernel: fn null)
Shape site_shape(const SitePlan& P, bool real) {
  if (P.blocks == 1) {
    if (P.R == 2) return shape_mode<512, 2, 0>(P.mode, real);
    switch (P.T) {
      case 64: return shape_mode<64, 1, 0>(P.mode, real);
      case 128: return shape_mode<128, 1, 0>(P.mode, real);
      case 256: return shape_mode<256, 1, 0>(P.mode, real);
      default: return shape_mode<512, 1, 0>(P.mode, real);
    }
  }
  if (P.T == 512) return P.mode == kOneSet ? shape_of<512, 1, kOneSet, 5>(real) : Shape{};
  switch (std::max(P.nfar[0], P.nfar[1])) {
    case 0: case 1: case 2:
    case 3: return shape_mode<256, 1, 3>(P.mode, real);
    case 4: return shape_mode<256, 1, 4>(P.mode, real);
    case 5: return shape_mode<256, 1, 5>(P.mode, real);
    default: return Shape{};
  }
}

size_t site_lds(const SitePlan& P) {
  return size_t(P.T) * size_t(P.R) * sizeof(double2) + sizeof(SiteShared);
}

}  // namespace

bool plan_site(const ParityForm& F, int max_row, SitePlan* P) try {
  const int nb = F.nb;
  if (nb < 1) return false;
  SitePlan S;
  // the sets: with one driven term, its terms and H0's apart (set 0 the larger
  // part of most models: single flips); with several, all in one
  std::vector<ParityTerm> sets[2];
  if (F.nterms > 1) {
    S.mode = kWeighted;
    sets[0] = merge_terms(F.terms);
  } else {
    for (const ParityTerm& t : F.terms) sets[t.term == 1 ? 0 : 1].push_back(t);
    S.set_term[0] = 1;
    S.set_term[1] = 0;
    if (sets[0].empty()) {
      sets[0].swap(sets[1]);
      std::swap(S.set_term[0], S.set_term[1]);
    }
    S.mode = sets[1].empty() ? kOneSet : kTwoSets;
  }
  // The shape: as few wavefronts per SIMD and rows per thread as keep the terms
  // in registers.  Measured per iteration (MI355X, driven Ising chain; in
  // parentheses the CSR kernels of persistent.hip): 2^9 rows, one workgroup,
  // 1.2 us (2.6); 2^10, one workgroup with two rows per thread 1.4 (3.0), a team of
  // four 2.0; 2^11, a team of eight 2.1 (4.3), one workgroup with four rows 8.0,
  // as it spills; 2^13, 32 blocks of 256 threads 2.1 (4.3), 16 of 512 2.4; 2^14,
  // 32 of 512 2.8 (4.6), 32 of 256 with two rows 3.1 (the teams before the
  // number of terms that leave the block was fixed at compile time: 2.0 at 2^13
  // and 2.5 at 2^14 since, without a branch per term).  Two sets or several
  // driven terms need registers for twice the terms: at 2^14 rows they spill
  // and take 15 us (6.0).  Larger teams than 32 do not fit one XCD.  One
  // workgroup is kept up to 2^10 rows also where a team is faster (two sets: 3.4
  // against 2.4), so that calls on several streams run side by side.  There two sets
  // spill (69 registers, 119 with complex values, as do 32 of the complex teams of
  // 512), and short rows are left to the CSR kernel: rows of 11 entries 276 and 290 us
  // (three steps), of 13 284 and 290, of 14 308 and 291, of 20 (a driven Heisenberg
  // chain) 5.6 and 3.2 us an iteration.
  const bool simple = S.mode == kOneSet;
  S.R = 1;
  if (nb == 10 && S.mode == kTwoSets && max_row <= 13) return false;
  if (nb <= 10) {
    S.blocks = 1;
    S.T = nb <= 6 ? 64 : nb <= 9 ? 1 << nb : 512;
    S.R = nb == 10 ? 2 : 1;
  } else if (nb <= 13) {
    S.T = 256;
    S.blocks = 1 << (nb - 8);
  } else if (nb == 14 && simple) {
    S.T = 512;
    S.blocks = 32;
  } else {
    return false;
  }
  for (S.tl = nb; (1 << (nb - S.tl)) < S.blocks;) S.tl -= 1;
  for (int s = 0; s < 2; ++s)
    for (const ParityTerm& t : sets[s]) S.nfar[s] += (t.off >> S.tl) != 0;
  const Shape K = site_shape(S, F.real);
  if (!K.fn) return false;
  int base = 0;
  for (int s = 0; s < 2; ++s) {
    const int first_lds = base + K.mv[s], first_reg = first_lds + K.lds[s];
    const int mix = first_reg + K.reg[s], first_far = mix + K.mix[s];
    int lds = 0, far = 0;
    std::vector<char> used(size_t(first_far + K.far[s]), 0);
    for (const ParityTerm& t : sets[s]) {
      const uint32_t thread = t.off & uint32_t(S.T - 1);
      const uint32_t reg = (t.off & ((1u << S.tl) - 1u)) / uint32_t(S.T);
      const bool by_reg = (t.pmask & ((1u << S.tl) - 1u)) / uint32_t(S.T);
      int slot = -1;
      if (t.off >> S.tl) {
        if (far < K.far[s]) slot = first_far + far++;
      } else if (reg != 0 && thread == 0) {
        slot = first_reg + int(reg) - 1;
      } else if (reg != 0) {
        if (K.mix[s] && reg == 1) slot = mix;
      } else if (!by_reg) {  // (these slots hold one value for a thread's rows)
        const int move = s == 0 ? (t.off == 1 ? 0 : t.off == 2 ? 1 : t.off == 8 ? 2 : -1)
                                : (t.off == 3 ? 0 : -1);
        if (move >= 0 && !used[size_t(base + move)]) slot = base + move;
        else if (lds < K.lds[s]) slot = first_lds + lds++;
      }
      if (slot < 0 || slot >= kSiteSlots || used[size_t(slot)]) return false;
      used[size_t(slot)] = 1;
      S.e[slot] = make_elem(t);
      S.e[slot].off = t.off;
    }
    base = first_far + K.far[s];
  }
  *P = S;
  return true;
} catch (const std::bad_alloc&) {
  return false;
}

hipError_t site_prepare(const SitePlan& P, bool real, int num_cus, bool* fits) {
  if (P.blocks == 1) {  // at most 512 threads and 64 KiB
    *fits = true;
    return hipSuccess;
  }
  const void* fn = site_shape(P, real).fn;
  const size_t lds = site_lds(P);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, P.T, lds);
  if (e != hipSuccess) return e;
  *fits = per * num_cus >= 8 * P.blocks;
  return hipSuccess;
}

hipError_t site_upload(const ParityForm& F, DevSite* S) try {
  const size_t ids = 3 * kSiteRecs * sizeof(Rec);
  const size_t table = ids + 264 * sizeof(unsigned long long);  // 256 blocks, the counter
  const size_t diag = table + sizeof(S->plan.e);
  std::vector<unsigned char> h(diag + F.diag.size() * sizeof(double), 0);
  std::memcpy(h.data() + table, S->plan.e, sizeof(S->plan.e));
  if (!F.diag.empty())
    std::memcpy(h.data() + diag, F.diag.data(), F.diag.size() * sizeof(double));
  hipError_t e = hipMalloc(&S->rec, h.size());
  if (e != hipSuccess) return e;
  char* const d = static_cast<char*>(S->rec);
  S->ids = reinterpret_cast<unsigned long long*>(d + ids);
  S->count = S->ids + 256;
  S->e = reinterpret_cast<PElem*>(d + table);
  S->diag = F.diag.empty() ? nullptr : reinterpret_cast<double*>(d + diag);
  S->real = F.real;
  S->diag_term = F.diag_term;
  return hipMemcpy(d, h.data(), h.size(), hipMemcpyHostToDevice);
} catch (const std::bad_alloc&) {
  return hipErrorOutOfMemory;
}

hipError_t launch_site(const DevSite& S, const PersistArgs& args, hipStream_t st, int nwts) {
  SiteArgs A{};
  A.p = args;
  if (nwts > 0) {
    A.inline_w = 1;
    std::copy(args.wts, args.wts + nwts, A.w);
    A.p.wts = nullptr;
  }
  A.e = S.e;
  for (int s = 0; s < 2; ++s) A.set_term[s] = S.plan.set_term[s];
  A.diag = S.diag;
  A.diag_term = S.diag_term;
  A.tl = S.plan.tl;
  A.blocks = S.plan.blocks;
  A.rec = S.rec;
  A.ids = S.ids;
  A.count = S.count;
  A.skew = S.skew;
  A.spread = S.spread;
  const void* fn = site_shape(S.plan, S.real).fn;
  void* kargs[] = {&A};
  if (S.plan.blocks == 1)
    return hipLaunchKernel(fn, dim3(1), dim3(S.plan.T), kargs, site_lds(S.plan), st);
  return hipLaunchCooperativeKernel(fn, dim3(8 * S.plan.blocks), dim3(S.plan.T), kargs,
                                    (unsigned)site_lds(S.plan), st);
}

}  // namespace cfet
