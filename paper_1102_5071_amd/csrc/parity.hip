// Two-sweep kernels on the site-operator form (parity.h).
//
// One application y = H_w x is two launches.  The first sweep walks tiles of
// the bit-permuted order and writes the part of y from the terms that flip
// high row bits; the second walks tiles of consecutive rows and adds the
// rest and the diagonal.  A workgroup holds the tile's x in LDS; thread t owns
// the tile indices t + r T (r < R) and keeps their x and their sums in
// registers, so one pass over the terms serves R rows: every block weights the
// table of terms into LDS, and the operator is read from memory only as that
// table and its diagonal, 8 bytes per row.
//
// In the Lanczos recurrence the three-term update is folded into the first
// sweep's loads (the pipelined form of the persistent kernels):
//     u_k = (z_{k-1} - alpha_{k-1} u_{k-1}) / nu_{k-1} - (nu_{k-1} / nu_{k-2}) u_{k-2}
// with z_k = H_w u_k, alpha_k = <u_k, z_k> / nu_k^2, nu_k = ||u_k||, so an
// iteration is two launches and one reduction: the first sweep reads three
// vectors and writes two (u_k and its part of z_k), the second reads u_k, that
// part and the diagonal and writes z_k.  8.5 vectors of traffic against 9.5
// for SpMV and update apart, and what the second sweep gathers beyond its tile
// on top: at 2^24 rows the counters show 9.4 for the Heisenberg chain, 2.52 GB
// in 472 us (239 for the first sweep, 231 for the second).  z_k is stored where
// u_{k+1} will be.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "parity.h"
#include "sweep_common.hpp"
#include "tridiag.hpp"

namespace cfet {

namespace {

// what a launch computes
enum SweepOp { kApply = 0, kLanczos = 1, kCheb = 2 };

// Sums of a and b over the block, in wavefront order; every thread gets them.
template <int T>
__device__ __forceinline__ void block_sum2(double& a, double& b, double* red) {
  constexpr int W = T / 64;
  a = w_sum63(a);
  b = w_sum63(b);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) {
    red[threadIdx.x >> 6] = a;
    red[W + (threadIdx.x >> 6)] = b;
  }
  __syncthreads();
  double ta = 0.0, tb = 0.0;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    ta += red[i];
    tb += red[W + i];
  }
  a = ta;
  b = tb;
}

// This thread's share of the np records, added in a fixed order; the loads of
// a chunk are in flight together.
template <int T>
__device__ __forceinline__ void thread_records(const double2* __restrict__ p, int np, double& a,
                                               double& b) {
  constexpr int PER = T >= 512 ? 2 : T >= 256 ? 4 : 8;
  a = b = 0.0;
  for (int c = 0; c < np; c += PER * T) {
    double2 v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = c + (int)threadIdx.x + j * T;
      v[j] = p[i < np ? i : np - 1];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (c + (int)threadIdx.x + j * T < np) {
        a += v[j].x;
        b += v[j].y;
      }
  }
}

// Start of phase k >= 1 (k = m: the end of the recurrence): the sums of phase
// k - 1, its alpha and norm, the early-stop rule.  False when the recurrence
// has stopped; else the coefficients of u_k.  Block 0 writes the scalars.
template <int T>
__device__ bool phase_start(int k, const double2* part, int np, LzScalars* S, double* scale,
                            double* red, double& c1, double& c2, double& c3) {
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (S->brk[k - 1]) {
    if (first && k < kMaxM) S->brk[k] = 1;
    return false;
  }
  const double sc_prev = (k >= 2) ? scale[k - 2] : 0.0;
  const double al_prev = (k >= 2) ? S->alpha[k - 2] : 0.0;
  const double inv_prev = (k >= 2) ? S->inv_nrm[k - 2] : 0.0;
  double s1, s2;
  thread_records<T>(part, np, s1, s2);
  block_sum2<T>(s1, s2, red);
  const double nu = sqrt(s2);
  bool stop;
  double sc = 0.0;
  if (k == 1) {
    stop = (nu == 0.0);  // psi = 0 stays 0
  } else {
    sc = fmax(sc_prev, fabs(al_prev) + nu);
    stop = (nu <= kBreakdownRel * sc);
  }
  const double inv = 1.0 / nu;
  const double alpha = s1 * inv * inv;
  if (first) {
    if (k == 1) S->beta0 = nu;
    else S->beta[k - 2] = nu;
    scale[k - 1] = sc;
    if (k < kMaxM) S->brk[k] = stop ? 1 : 0;
    if (stop) {
      S->m_eff = k - 1;
    } else {
      S->alpha[k - 1] = alpha;
      S->inv_nrm[k - 1] = inv;
    }
  }
  if (stop) return false;
  c1 = inv;
  c2 = alpha * inv;
  c3 = (k >= 2) ? nu * inv_prev : 0.0;
  return true;
}

// blocks to tiles: XCD b % 8 takes a contiguous eighth, so that the tiles its
// blocks work on at one time share cache lines and gathered neighbours
struct Tiles {
  int first, end, stride;
};
__device__ __forceinline__ Tiles my_tiles(int ntiles) {
  constexpr int kXcds = 8;
  const int nb = gridDim.x;
  if (nb % kXcds != 0 || ntiles % kXcds != 0) return {(int)blockIdx.x, ntiles, nb};
  const int per = ntiles / kXcds;
  const int beg = (blockIdx.x % kXcds) * per;
  return {beg + (int)(blockIdx.x / kXcds), beg + per, nb / kXcds};
}

// the value of term e at a row of parity p, real and imaginary part
template <bool RV, class E>
__device__ __forceinline__ dv2 value_of(const E& e, uint32_t p) {
  dv2 v;
  v.x = p ? e.v1 : e.v0;
  v.y = RV ? 0.0 : (p ? e.w1 : e.w0);
  return v;
}

// Element of a vector at a wavefront-uniform row plus the thread's own byte
// offset (32 bits: nb <= kParityMaxBits): one scalar base per access and one
// vector register for all of them.
template <class V>
__device__ __forceinline__ V* at(V* base, uint32_t row, uint32_t tb) {
  using B = std::conditional_t<std::is_const<V>::value, const char, char>;
  return reinterpret_cast<V*>(reinterpret_cast<B*>(base + row) + tb);
}

template <bool NTL>
__device__ __forceinline__ double2 ld(const double2* p) {
  if (NTL) {
    const dv2 v = __builtin_nontemporal_load(reinterpret_cast<const dv2*>(p));
    return make_double2(v.x, v.y);
  }
  return *p;
}

template <bool NTL>
__device__ __forceinline__ void st(double2* p, double2 v) {
  if (NTL) __builtin_nontemporal_store(dv2{v.x, v.y}, reinterpret_cast<dv2*>(p));
  else *p = v;
}

// Terms of a sweep, weighted, in LDS.  The groups, in order: n[0] terms of one
// value whose flips move the thread index only; n[1] the same with a value that
// depends on the row (one parity for all R rows of a thread); n[2] terms that
// move or depend on the register index as well; n[3] terms that move the
// register index alone (their x is in this thread's registers); n[4] terms
// gathered from memory (second sweep).
struct WElem {
  uint32_t off, pmask, rpar;
  uint32_t has;  // bit p: the operator stores an entry on rows of parity p
  double v0, v1;
  double w0, w1;
};

// terms whose tile reads are in flight together, for R rows per thread
constexpr int batch_of(int R) { return R <= 2 ? 4 : R == 4 ? 2 : 1; }

// (Real values are held to 128 registers, two blocks a CU.  With eight rows per
// thread, tiles of 2^12, that spills 20 in the first sweep of the recurrence and 18
// in the second, 26 in the Chebyshev and 38 in the apply sweep.)
template <int TB, int T, bool RV, bool HI, int OP, bool NTL>
__global__ __launch_bounds__(T, RV ? 4 : 2) void k_sweep(SweepArgs A) {
  constexpr int R = (1 << TB) / T;
  constexpr int CH = R < 4 ? R : 4;  // rows whose tile reads are in flight together
  constexpr int U = batch_of(R);     // and terms
  extern __shared__ double2 xt[];
  WElem* we = reinterpret_cast<WElem*>(xt + (1 << TB));
  double* red = reinterpret_cast<double*>(we + kSweepTerms);
  // by wavefront: its part of the tile holds an infinity or a NaN
  typedef __attribute__((address_space(3))) uint8_t* lds_bytes;
  const lds_bytes odd_x = (lds_bytes)(uint8_t*)(red + 2 * (T / 64));
  auto any_odd = [&]() {
    unsigned long long v = *(__attribute__((address_space(3))) const unsigned long long*)odd_x;
    if (T < 512) v &= (1ull << (T / 8)) - 1ull;
    return __builtin_amdgcn_readfirstlane((uint32_t)v | (uint32_t)(v >> 32)) != 0u;
  };
  const int t = threadIdx.x;
  const int n0 = A.n[0], n1 = n0 + A.n[1], n2 = n1 + A.n[2], n3 = n2 + A.n[3],
            n4 = HI ? n3 : n3 + A.n[4];
  // row bits of a tile index q < 2^TB
  auto row_of = [&](uint32_t q) -> uint32_t {
    return HI ? (q & ((1u << A.low) - 1u)) | ((q >> A.low) << A.high) : q;
  };
  const uint32_t rt = row_of((uint32_t)t);
  const uint32_t tb = rt << 4;
  uint32_t rr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) rr[r] = row_of((uint32_t)(r * T));
  // LDS byte address of this thread's first element; the tile starts at a
  // multiple of its size, so XORs stay inside it.  Opaque to the compiler so
  // that it keeps one XOR per term.
  uint32_t qb = (uint32_t)(uintptr_t)(lds_cptr)xt + ((uint32_t)t << 4);
  asm volatile("" : "+v"(qb));
  // first sweep: tiles that hold whole 128-byte lines go to the blocks in plain
  // order (neighbouring lines are open at the same time); half lines need the
  // other half's tile on the same XCD
  const Tiles Q = (HI && A.low >= 3) ? Tiles{(int)blockIdx.x, 1 << (A.nb - TB), (int)gridDim.x}
                                     : my_tiles(1 << (A.nb - TB));
  const bool form = HI && OP == kLanczos && A.k > 0;  // x = u_k is formed here
  const bool last = OP == kLanczos && A.k + 1 == A.m;  // only the sums are wanted
  double c1 = 0.0, c2 = 0.0, c3 = 0.0;
  double dot = 0.0, nrm = 0.0;
  PElem e{};
  if (t < n4) e = A.e[t];
  bool fresh = true;
  // with few rows per thread the reduction of the last phase overlaps the
  // first tile's loads; with eight the registers do not allow it, and a block
  // has several tiles
  constexpr bool kOverlap = R <= 4;
  if (form && !kOverlap &&
      !phase_start<T>(A.k, A.part_in, 2 * A.nblk, A.S, A.scale, red, c1, c2, c3))
    return;
  // the end of the sweep on the row that urow and off (at) stand for
  auto finish = [&](uint32_t urow, uint32_t off, double2 x, double2 a) {
    if (OP != kCheb) {
      st<NTL>(at(A.y, urow, off), a);
      return;
    }
    double wr = A.ct.scale * (a.x - A.ct.sigma * x.x);
    double wi = A.ct.scale * (a.y - A.ct.sigma * x.y);
    double2 pp = make_double2(0.0, 0.0);
    if (!A.ct.first) pp = ld<NTL>(at(A.ct.prev, urow, off));
    wr -= pp.x;
    wi -= pp.y;
    st<false>(at(A.ct.prev, urow, off), make_double2(wr, wi));
    if (A.ct.acc) {
      // t_{k-2} = prev, t_{k-1} = x and t_k = w are all here: psi is read and
      // written at every third term only (7.2 vectors of traffic a term
      // instead of 8.5; one step on 2^22 rows 8.9 -> 8.0 ms)
      double2 q = ld<NTL>(at(A.ct.psi, urow, off));
      q.x += A.ct.cp.x * pp.x - A.ct.cp.y * pp.y;
      q.y += A.ct.cp.x * pp.y + A.ct.cp.y * pp.x;
      q.x += A.ct.cx.x * x.x - A.ct.cx.y * x.y;
      q.y += A.ct.cx.x * x.y + A.ct.cx.y * x.x;
      q.x += A.ct.ck.x * wr - A.ct.ck.y * wi;
      q.y += A.ct.ck.x * wi + A.ct.ck.y * wr;
      st<NTL>(at(A.ct.psi, urow, off), q);
    }
  };
  bool redo = false;  // a tile holds an infinity or a NaN
  for (int tile = Q.first; tile < Q.end; tile += Q.stride) {
    const uint32_t tr = (uint32_t)tile << (HI ? A.low : TB);
    const uint32_t row0 = tr | rt;
    // every load of the tile is issued before anything waits
    double2 xo[R], acc[R];
    double dg[R];
    if (form) {
      double2 b[R];
#pragma unroll
      for (int r = 0; r < R; ++r) xo[r] = ld<NTL>(at(A.u, tr | rr[r], tb));
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = ld<NTL>(at(A.x, tr | rr[r], tb));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        b[r] = make_double2(0.0, 0.0);
        if (A.k >= 2) b[r] = ld<NTL>(at(A.u2, tr | rr[r], tb));
      }
      if (kOverlap && fresh &&
          !phase_start<T>(A.k, A.part_in, 2 * A.nblk, A.S, A.scale, red, c1, c2, c3))
        return;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        xo[r].x = fma(c1, xo[r].x, fma(-c2, acc[r].x, -c3 * b[r].x));
        xo[r].y = fma(c1, xo[r].y, fma(-c2, acc[r].y, -c3 * b[r].y));
        st<false>(at(A.u, tr | rr[r], tb), xo[r]);
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) xo[r] = ld<false>(at(A.x, tr | rr[r], tb));
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      acc[r] = make_double2(0.0, 0.0);
      dg[r] = 0.0;
      if (!HI) {
        if (!last) acc[r] = ld<NTL>(at(A.y, tr | rr[r], tb));
        if (A.diag) dg[r] = __builtin_nontemporal_load(at(A.diag, tr | rr[r], tb >> 1));
      }
    }
    if (!HI) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double d = A.wdiag * dg[r];
        acc[r].x = fma(d, xo[r].x, acc[r].x);
        acc[r].y = fma(d, xo[r].y, acc[r].y);
      }
    }
    if (fresh) {
      fresh = false;
      if (OP == kLanczos && !form) {
        if (HI) {
          if (blockIdx.x == 0 && t == 0) A.S->brk[0] = 0;
        } else if (A.S->brk[A.k]) {
          return;
        }
      }
      if (t < n4) {
        double w = A.tw.w[0], w2 = A.tw.w[0];
#pragma unroll
        for (int k = 1; k <= kMaxTerms; ++k) {
          w = e.term == k ? A.tw.w[k] : w;
          w2 = e.term2 == k ? A.tw.w[k] : w2;
        }
        const uint32_t has0 = OP != kLanczos && (e.v0 != 0.0 || e.w0 != 0.0 || e.b0 != 0.0 || e.d0 != 0.0);
        const uint32_t has1 = OP != kLanczos && (e.v1 != 0.0 || e.w1 != 0.0 || e.b1 != 0.0 || e.d1 != 0.0);
        we[t] = {e.off, e.pmask, e.rpar, has0 | has1 << 1,
                 fma(w2, e.b0, w * e.v0), fma(w2, e.b1, w * e.v1),
                 fma(w2, e.d0, w * e.w0), fma(w2, e.d1, w * e.w1)};
      }
    } else {
      __syncthreads();  // the previous tile's readers are done
    }
#pragma unroll
    for (int r = 0; r < R; ++r) xt[t + r * T] = xo[r];
    if (OP != kLanczos) {
      // wavefronts that hold an infinity or a NaN (in the recurrence one makes
      // every norm, and so the whole state, not finite)
      double z = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) z = fma(xo[r].x, 0.0, fma(xo[r].y, 0.0, z));
      const bool odd = __ballot(z != 0.0) != 0ull;
      if ((t & 63) == 0) odd_x[t >> 6] = odd;
    }
    __syncthreads();
    if (!HI) {
      for (int i = n3; i < n4; ++i) {
        const WElem e = we[i];
        const uint32_t eo = __builtin_amdgcn_readfirstlane(e.off);
        const uint32_t ep = __builtin_amdgcn_readfirstlane(e.rpar);
        const uint32_t p = (uint32_t)__popc(row0 & e.pmask) & 1u;
        const dv2 va = value_of<RV>(e, p), vb = value_of<RV>(e, p ^ 1u);
#pragma unroll
        for (int q = 0; q < R; q += CH) {
          double2 xv[CH];
#pragma unroll
          for (int j = 0; j < CH; ++j) {
            const dv2 v = ((ep >> (q + j)) & 1u) ? vb : va;
            xv[j] = make_double2(0.0, 0.0);
            if (v.x != 0.0 || (!RV && v.y != 0.0))
              xv[j] = *at(A.x, (tr | rr[q + j]) ^ (eo & ~(uint32_t)(T - 1)),
                          tb ^ ((eo & (uint32_t)(T - 1)) << 4));
          }
#pragma unroll
          for (int j = 0; j < CH; ++j)
            acc_fma<RV>(acc[q + j], ((ep >> (q + j)) & 1u) ? vb : va, xv[j]);
        }
      }
    }
    // U terms at a time (the groups are padded with terms of value 0), their
    // tile reads in flight together
    for (int i = 0; i < n0; i += U) {
      uint32_t a[U];
      dv2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const WElem& e = we[i + u];
        a[u] = qb ^ (e.off << 4);
        v[u] = dv2{e.v0, RV ? 0.0 : e.w0};
      }
#pragma unroll
      for (int q = 0; q < R; q += CH) {
        double2 xv[U][CH];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < CH; ++j) xv[u][j] = lds_at(a[u] + (q + j) * T * 16);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < CH; ++j) acc_fma<RV>(acc[q + j], v[u], xv[u][j]);
      }
    }
    for (int i = n0; i < n1; i += U) {
      uint32_t a[U];
      dv2 v[U];
      bool any = U > 1;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const WElem& e = we[i + u];
        a[u] = qb ^ (e.off << 4);
        v[u] = value_of<RV>(e, (uint32_t)__popc(row0 & e.pmask) & 1u);
        if (U == 1) any = __ballot(v[u].x != 0.0 || (!RV && v[u].y != 0.0)) != 0ull;
      }
      if (!any) continue;
#pragma unroll
      for (int q = 0; q < R; q += CH) {
        double2 xv[U][CH];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < CH; ++j) xv[u][j] = lds_at(a[u] + (q + j) * T * 16);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < CH; ++j) acc_fma<RV>(acc[q + j], v[u], xv[u][j]);
      }
    }
    for (int i = n1; i < n2; ++i) {
      const WElem& e = we[i];
      const uint32_t a = qb ^ (e.off << 4);
      const uint32_t p = (uint32_t)__popc(row0 & e.pmask) & 1u;
      const dv2 va = value_of<RV>(e, p), vb = value_of<RV>(e, p ^ 1u);
      const uint32_t ep = __builtin_amdgcn_readfirstlane(e.rpar);
#pragma unroll
      for (int q = 0; q < R; q += CH) {
        double2 xv[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) xv[j] = lds_at(a ^ (uint32_t)((q + j) * T * 16));
#pragma unroll
        for (int j = 0; j < CH; ++j)
          acc_fma<RV>(acc[q + j], ((ep >> (q + j)) & 1u) ? vb : va, xv[j]);
      }
    }
    for (int i = n2; i < n3; ++i) {
      const WElem& e = we[i];
      const uint32_t p = (uint32_t)__popc(row0 & e.pmask) & 1u;
      const dv2 va = value_of<RV>(e, p), vb = value_of<RV>(e, p ^ 1u);
      const uint32_t ep = __builtin_amdgcn_readfirstlane(e.rpar);
#define CFET_FLIP(M)                                                              \
  case M:                                                                         \
    _Pragma("unroll") for (int r = 0; r < R; ++r)                                 \
        acc_fma<RV>(acc[r], ((ep >> r) & 1u) ? vb : va, xo[(r ^ M) & (R - 1)]);   \
    break;
      switch (__builtin_amdgcn_readfirstlane(e.off) / T) {
        CFET_FLIP(1)
        CFET_FLIP(2)
        CFET_FLIP(3)
        CFET_FLIP(4)
        CFET_FLIP(5)
        CFET_FLIP(6)
        CFET_FLIP(7)
      }
#undef CFET_FLIP
    }
    if (OP != kLanczos && __builtin_expect(any_odd(), 0)) {
      redo = true;
      continue;
    }
    if (OP == kLanczos) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!HI || last) dot = fma(xo[r].x, acc[r].x, fma(xo[r].y, acc[r].y, dot));
        if (HI) nrm = fma(xo[r].x, xo[r].x, fma(xo[r].y, xo[r].y, nrm));
      }
      if (last) continue;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) finish(tr | rr[r], tb, xo[r], acc[r]);
  }
  if (OP != kLanczos && __builtin_expect(redo, 0)) {
    // The loops above multiply by the zeros of entries that the operator does
    // not store, which an infinity or a NaN in the tile must not meet: such
    // tiles again, a row at a time, over the stored entries only.  (Looking for
    // them costs a Chebyshev run up to 1 %: 2^22 rows 3144 -> 3157 us, 2^19 619 -> 626.)
    for (int tile = Q.first; tile < Q.end; tile += Q.stride) {
      const uint32_t tr = (uint32_t)tile << (HI ? A.low : TB);
      __syncthreads();
      double z = 0.0;
#pragma unroll 1
      for (int r = 0; r < R; ++r) {
        const double2 x = A.x[tr | row_of((uint32_t)(t + r * T))];
        z = fma(x.x, 0.0, fma(x.y, 0.0, z));
        xt[t + r * T] = x;
      }
      const bool mine = __ballot(z != 0.0) != 0ull;
      if ((t & 63) == 0) odd_x[t >> 6] = mine;
      __syncthreads();
      if (!any_odd()) continue;
#pragma unroll 1
      for (int r = 0; r < R; ++r) {
        const uint32_t q = (uint32_t)(t + r * T);
        const uint32_t row = tr | row_of(q);
        double2 a = make_double2(0.0, 0.0);
        if (!HI) {
          a = A.y[row];
          const double d = A.diag ? A.diag[row] : 0.0;
          if (d != 0.0) acc_fma<true>(a, dv2{A.wdiag * d, 0.0}, xt[q]);
        }
#pragma unroll 1
        for (int i = 0; i < n4; ++i) {
          const WElem& e = we[i];
          const uint32_t p = (uint32_t)__popc(row & e.pmask) & 1u;
          if (!((e.has >> p) & 1u)) continue;
          const double2 x = HI || i < n3 ? xt[q ^ e.off] : A.x[row ^ e.off];
          acc_fma<RV>(a, value_of<RV>(e, p), x);
        }
        finish(row, 0u, xt[q], a);
      }
    }
  }
  if (OP == kLanczos) {
    block_sum2<T>(dot, nrm, red);
    if (t == 0) A.part_out[(HI ? 0 : A.nblk) + blockIdx.x] = make_double2(dot, nrm);
  }
}

// End of the recurrence: the last alpha and norm, then the small exponential
// and the recombination coefficients.
__global__ __launch_bounds__(64) void k_parity_small(const double2* part, int np, LzScalars* S,
                                                     double* scale, int m, double dt,
                                                     DevStats* stats) {
  __shared__ double lds[kChebMaxTerms];
  __shared__ double red[4];
  const int lane = threadIdx.x;
  double c1, c2, c3;
  const bool done = !phase_start<64>(m, part, np, S, scale, red, c1, c2, c3);
  __threadfence_block();
  __syncthreads();
  const volatile LzScalars* V = S;  // written by lane 0 above
  const int meff = done ? V->m_eff : m;
  double a = (lane < meff) ? V->alpha[lane] : 0.0;
  double b = (lane < meff - 1) ? V->beta[lane] : 0.0;
  const double beta0 = V->beta0;
  int status = CFET_OK;
  double2 c = make_double2(0.0, 0.0);
  if (meff > 0) {
    const bool bad = !(isfinite(a) && isfinite(b) && isfinite(beta0));
    if (__ballot(bad) != 0ull) status = CFET_ENONFINITE;
    else status = tridiag_exp_e1(a, b, meff, dt, lds, c);
  }
  if (lane < meff) {
    const double sc = beta0 * V->inv_nrm[lane];
    S->coef[2 * lane] = c.x * sc;
    S->coef[2 * lane + 1] = c.y * sc;
  }
  if (lane == 0) {
    S->m_eff = meff;
    stats->exponentials += 1;
    stats->matvecs += (unsigned long long)meff;
    if (meff < stats->min_m_eff) stats->min_m_eff = meff;
    if (done) stats->breakdowns += 1;
    if (status != CFET_OK && stats->status == CFET_OK) stats->status = status;
    stats->last_norm2 = beta0 * beta0;
  }
}

constexpr int threads_of(int tb) { return tb >= 10 ? 512 : 256; }

size_t lds_of(int tb) {
  return (size_t(16) << tb) + kSweepTerms * sizeof(WElem) +
         2 * (threads_of(tb) / 64) * sizeof(double) + 8;
}

template <int TB, bool RV, bool HI, int OP, bool NTL>
void go(const SweepArgs& A, hipStream_t st) {
  hipLaunchKernelGGL((k_sweep<TB, threads_of(TB), RV, HI, OP, NTL>), dim3(A.nblk),
                     dim3(threads_of(TB)), lds_of(TB), st, A);
}

// Non-temporal accesses of the vectors that stream through, where a vector
// does not fit the memory-side cache (256 MB); below that they evict what the
// next launch reads (2^20 rows: 39.6 us per iteration with them, 35.8 without;
// 2^22: equal).  Such vectors take the largest tile.
constexpr int kStreamBits = 24;

template <bool RV, bool HI, int OP>
hipError_t go_tb(const SweepArgs& A, hipStream_t st) {
  if (A.nb >= kStreamBits && A.tb != 12) return hipErrorInvalidValue;
  switch (A.tb) {
    case 9: go<9, RV, HI, OP, false>(A, st); break;
    case 10: go<10, RV, HI, OP, false>(A, st); break;
    case 11: go<11, RV, HI, OP, false>(A, st); break;
    case 12:
      if (A.nb >= kStreamBits) go<12, RV, HI, OP, true>(A, st);
      else go<12, RV, HI, OP, false>(A, st);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int OP>
hipError_t go_any(const SweepArgs& A, bool real, bool hi, hipStream_t st) {
  if (real) return hi ? go_tb<true, true, OP>(A, st) : go_tb<true, false, OP>(A, st);
  return hi ? go_tb<false, true, OP>(A, st) : go_tb<false, false, OP>(A, st);
}

SweepArgs sweep_args(const DevParity& P, const TermWeights& tw, int sweep) {
  SweepArgs A{};
  A.e = P.e + sweep * kSweepTerms;
  for (int g = 0; g < 5; ++g) A.n[g] = P.n[sweep][g];
  A.nb = P.plan.nb;
  A.tb = sweep == 0 ? P.plan.tbh : P.plan.tbl;
  A.low = P.plan.low;
  A.high = P.plan.high;
  A.nblk = P.nblk;
  A.diag = P.diag;
  A.wdiag = P.diag_term >= 0 ? tw.w[P.diag_term] : 0.0;
  A.tw = tw;
  return A;
}

template <class K>
hipError_t allow(K kernel, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <bool RV, bool HI, bool NTL>
hipError_t allow_ops() {
  constexpr int TB = 12, T = threads_of(TB);
  const size_t b = lds_of(TB);
  hipError_t e = allow(k_sweep<TB, T, RV, HI, kApply, NTL>, b);
  if (e == hipSuccess) e = allow(k_sweep<TB, T, RV, HI, kLanczos, NTL>, b);
  if constexpr (!HI)
    if (e == hipSuccess) e = allow(k_sweep<TB, T, RV, HI, kCheb, NTL>, b);
  return e;
}

template <bool RV>
hipError_t allow_values() {
  hipError_t e = allow_ops<RV, true, true>();
  if (e == hipSuccess) e = allow_ops<RV, false, true>();
  if (e == hipSuccess) e = allow_ops<RV, true, false>();
  if (e == hipSuccess) e = allow_ops<RV, false, false>();
  return e;
}

}  // namespace

int parity_grid(const ParityPlan& P, int num_cus) {
  // two workgroups per CU share it, one loading while the other computes
  return std::min(1 << (P.nb - std::max(P.tbh, P.tbl)), 2 * std::max(num_cus, 1));
}

size_t parity_part_bytes(int nblk) {
  return size_t(4) * size_t(nblk) * sizeof(double2) + kMaxM * sizeof(double);
}

// Allows the kernels on the largest tile their LDS (above 64 KiB).
hipError_t parity_prepare() {
  const hipError_t e = allow_values<true>();
  return e == hipSuccess ? allow_values<false>() : e;
}

void parity_tables(const ParityPlan& P, PElem* out, int n[2][5]) {
  for (int sweep = 0; sweep < 2; ++sweep) {
    const bool hi = sweep == 0;
    PElem* const e_out = out + sweep * kSweepTerms;
    const int tb = hi ? P.tbh : P.tbl;
    const int T = threads_of(tb), R = (1 << tb) / T;
    auto row_of = [&](uint32_t q) {
      return hi ? (q & ((1u << P.low) - 1u)) | ((q >> P.low) << P.high) : q;
    };
    auto local = [&](uint32_t off) {  // flips on the tile index
      return hi ? (off & ((1u << P.low) - 1u)) | ((off >> P.high) << P.low) : off;
    };
    auto element = [&](const ParityTerm& t, bool gather, int* group) {
      PElem e = make_elem(t);
      e.off = gather ? t.off : local(t.off);
      for (int r = 0; r < R; ++r)
        e.rpar |= uint32_t(__builtin_popcount(row_of(uint32_t(r * T)) & t.pmask) & 1) << r;
      const bool thread_flip = (e.off & uint32_t(T - 1)) != 0;
      const bool reg_flip = (e.off & ~uint32_t(T - 1)) != 0;
      *group = gather ? 4 : !thread_flip ? 3 : (reg_flip || e.rpar) ? 2 : e.pmask ? 1 : 0;
      return e;
    };
    int k = 0;
    for (int g = 0; g < 5; ++g) {
      n[sweep][g] = 0;
      auto take = [&](const std::vector<ParityTerm>& list, bool gather) {
        for (const ParityTerm& t : list) {
          int group = 0;
          const PElem e = element(t, gather, &group);
          if (group != g) continue;
          e_out[k++] = e;
          n[sweep][g] += 1;
        }
      };
      take(hi ? P.hi : P.lo, false);
      if (!hi) take(P.far, true);
      if (g < 2)
        for (; n[sweep][g] % batch_of(R); n[sweep][g] += 1) e_out[k++] = PElem{};
    }
  }
}

hipError_t launch_parity_apply(const DevParity& P, const TermWeights& tw, const double2* x,
                               double2* y, const ChebTerm& ct, hipStream_t st) {
  SweepArgs A = sweep_args(P, tw, 0);
  A.x = x;
  A.y = y;
  hipError_t e = go_any<kApply>(A, P.real, true, st);
  if (e != hipSuccess) return e;
  A = sweep_args(P, tw, 1);
  A.x = x;
  A.y = y;
  A.ct = ct;
  if (!ct.psi) return go_any<kApply>(A, P.real, false, st);
  return P.real ? go_tb<true, false, kCheb>(A, st) : go_tb<false, false, kCheb>(A, st);
}

hipError_t launch_parity_lanczos(const DevParity& P, const TermWeights& tw, double dt, int m,
                                 double2* const* W, LzScalars* S, DevStats* stats,
                                 EventPool* events, hipStream_t st) {
  SweepArgs H = sweep_args(P, tw, 0), L = sweep_args(P, tw, 1);
  H.S = L.S = S;
  H.scale = L.scale = reinterpret_cast<double*>(P.part + size_t(4) * size_t(P.nblk));
  H.m = L.m = m;
  const size_t set = size_t(2) * size_t(P.nblk);
  for (int k = 0; k < m; ++k) {
    double2* const z = (k + 1 < m) ? W[k + 1] : nullptr;
    H.k = L.k = k;
    H.x = k > 0 ? W[k - 1] : W[0];
    H.u = W[k];
    H.u2 = k >= 2 ? W[k - 2] : nullptr;
    H.y = z;
    H.part_in = P.part + size_t((k + 1) & 1) * set;
    H.part_out = P.part + size_t(k & 1) * set;
    L.x = W[k];
    L.y = z;
    L.part_out = H.part_out;
    EventPool* ev = (events && events->used < events->cap) ? events : nullptr;
    if (ev) (void)hipEventRecord(ev->begin[ev->used], st);
    hipError_t e = go_any<kLanczos>(H, P.real, true, st);
    if (e == hipSuccess) e = go_any<kLanczos>(L, P.real, false, st);
    if (e != hipSuccess) return e;
    if (ev) {
      (void)hipEventRecord(ev->end[ev->used], st);
      ev->used += 1;
    }
  }
  hipLaunchKernelGGL(k_parity_small, dim3(1), dim3(64), 0, st,
                     P.part + size_t((m - 1) & 1) * set, 2 * P.nblk, S, H.scale, m, dt, stats);
  return hipGetLastError();
}

}  // namespace cfet
