// Site-operator form of a merged operator and the two-sweep kernels on it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "cfet_internal.h"
#include "host_common.h"

namespace cfet {

// One off-diagonal term of an operator on 2^nb rows: row r couples to column
// r XOR off with a value that depends on one parity of the row's bits only,
//     v(r) = parity(r & pmask) ? v1 : v0
// (0 where the operator stores nothing).  Every Pauli string and the sums of
// strings with the same flips have this form: sigma^x (pmask = 0), sigma^y
// (pmask = off, v1 = -v0 imaginary), a flip-flop s+s- + s-s+ of two sites
// (pmask = off, v0 = 0).
struct ParityTerm {
  uint32_t off, pmask;
  int term;  // 0: H0, 1 + k: H_k
  double v0[2], v1[2];
  // a second operator term's part with the same flips (-1: none), on the same
  // mask; see merge_terms
  int term2 = -1;
  double b0[2] = {0.0, 0.0}, b1[2] = {0.0, 0.0};
};

struct ParityForm {
  int nb = 0;                      // rows = 2^nb
  int nterms = 0;                  // driven terms
  std::vector<ParityTerm> terms;   // off-diagonal part
  int diag_term = -1;              // term that holds the diagonal (-1: none)
  std::vector<double> diag;        // real diagonal, one value per row
  bool real = true;                // every value is real
};

// The form of the merged operator, or false: the rows are not a power of two,
// an entry's values follow no parity, the diagonal is complex or lies in more
// than one term, or there are more than kParityMaxTerms off-diagonal terms.
// Exact: every stored value is compared with what the form says, bit for bit.
constexpr int kParityMaxTerms = 56;
constexpr int kSweepTerms = 64;  // with the padding of the sweeps' groups
bool find_parity_form(const std::vector<HostCSR>& mats, int nterms, int64_t n, unsigned nth,
                      ParityForm* F);

// Terms of different operator terms with the same flips as one, where one of
// the two has a single value or both the same mask (sigma^x and sigma^y of a
// site): the kernels read x once for both.
std::vector<ParityTerm> merge_terms(const std::vector<ParityTerm>& terms);

// The plan of the two sweeps.  The second sweep walks tiles of 2^tbl
// consecutive rows and applies every term whose flips stay inside the tile.
// The first walks tiles of a permuted order whose index bits are the `low`
// lowest row bits (contiguous segments of a vector), then the row bits from
// `high` up, then those between; it applies the terms that flip high bits.  A
// term that fits neither is gathered from memory in the second sweep.
struct ParityPlan {
  int nb = 0;
  int tbh = 0, tbl = 0;            // tile bits of the first and of the second sweep
  int low = 0, high = 0;           // tbh = low + nb - high
  std::vector<ParityTerm> hi, lo, far;
};
constexpr int kParityMinBits = 16;
constexpr int kParityMaxBits = 27;  // byte offsets inside a vector fit 32 bits
bool plan_parity(const ParityForm& F, ParityPlan* P);

// One term as a kernel reads it (device memory).
struct PElem {
  uint32_t off;    // XOR on the tile index (gathered terms: on the row)
  uint32_t pmask;  // parity mask on the row
  uint32_t rpar;   // bit r: parity of the mask over the row bits of register r
  int32_t term;    // 0: H0, 1 + k: H_k
  double v0, v1;   // real parts
  double w0, w1;   // imaginary parts
  int32_t term2;   // second part (ParityTerm), 0 with zero values where there is none
  int32_t pad;
  double b0, b1;
  double d0, d1;
};
// (off and rpar are the caller's)
inline PElem make_elem(const ParityTerm& t) {
  PElem e{};
  e.pmask = t.pmask;
  e.term = t.term;
  e.v0 = t.v0[0];
  e.v1 = t.v1[0];
  e.w0 = t.v0[1];
  e.w1 = t.v1[1];
  if (t.term2 >= 0) {
    e.term2 = t.term2;
    e.b0 = t.b0[0];
    e.b1 = t.b1[0];
    e.d0 = t.b0[1];
    e.d1 = t.b1[1];
  }
  return e;
}

struct SweepArgs {
  const PElem* e;           // the sweep's terms, in five groups (parity.hip) of n[0] .. n[4]
  int n[5];
  int nb, tb, low, high;
  int k, m;                 // Lanczos phase and Krylov size (recurrence only)
  int nblk;
  const double2* x;         // the vector multiplied (recurrence: u_{k-1} in the first sweep)
  double2* u;               // recurrence, first sweep: z_{k-1} in, u_k out
  const double2* u2;        // u_{k-2}
  double2* y;               // result: the first sweep writes its part, the second adds to it
  const double* diag;
  LzScalars* S;
  double* scale;            // scale[k]: max over t < k of |alpha_t| + beta_t
  const double2* part_in;   // the last phase's records: first sweep [0, nblk), second [nblk, 2 nblk)
  double2* part_out;
  double wdiag;
  TermWeights tw;
  ChebTerm ct;
};

// Device side of a context's site-operator form.
struct DevParity {
  bool ok = false;
  ParityPlan plan;
  bool real = true;
  int diag_term = -1;
  double* diag = nullptr;   // device
  PElem* e = nullptr;       // device: first sweep's terms, second sweep's
  int n[2][5] = {};         // their group sizes
  double2* part = nullptr;  // device: 2 sets x 2 sweeps x nblk records, then kMaxM
                            // doubles (SweepArgs::scale)
  int nblk = 0;
  int64_t bytes = 0;        // operator bytes one application reads
};

int parity_grid(const ParityPlan& P, int num_cus);
size_t parity_part_bytes(int nblk);
hipError_t parity_prepare();
// The terms of the two sweeps in the kernels' order and groups (host; sweep 0,
// 1 at e + sweep * kSweepTerms).
void parity_tables(const ParityPlan& P, PElem* e, int n[2][5]);
// y = H_w x (x and y distinct); with ct.psi set, the Chebyshev term instead
// of the store of y (y is then scratch).
hipError_t launch_parity_apply(const DevParity& P, const TermWeights& tw, const double2* x,
                               double2* y, const ChebTerm& ct, hipStream_t st);
// The Lanczos recurrence from W[0] with the small exponential (basis W[1..],
// unnormalised, scalars S): the contract of launch_lanczos.
hipError_t launch_parity_lanczos(const DevParity& P, const TermWeights& tw, double dt, int m,
                                 double2* const* W, LzScalars* S, DevStats* stats,
                                 EventPool* events, hipStream_t st);

// ---- persistent propagation on the same form (site.hip)
//
// One workgroup up to 2^10 rows; above, a team of workgroups on one XCD, each
// with 2^tl consecutive rows (T threads times R rows).
constexpr int kSiteRecs = 64;   // records of one exchange: two per block of a team
constexpr int kSiteSlots = 64;  // terms of a plan, at most
struct SitePlan {
  int blocks = 0, T = 0, R = 0, tl = 0;
  int mode = 0;              // SiteMode (site.hip)
  int set_term[2] = {0, 0};  // operator term of each set
  int nfar[2] = {0, 0};      // terms that leave the block, per set
  PElem e[kSiteSlots] = {};  // by slot
};
// max_row: stored entries of the longest row
bool plan_site(const ParityForm& F, int max_row, SitePlan* P);

struct DevSite {
  bool ok = false;
  SitePlan plan;
  bool real = true;
  int diag_term = -1;
  void* rec = nullptr;                // device, the start of the allocation that holds all:
                                      // 3 * kSiteRecs records
  unsigned long long* ids = nullptr;  // XCD of each block of a launch, then the launch counter
  PElem* e = nullptr;
  double* diag = nullptr;             // (null: no diagonal)
  unsigned long long* count = nullptr;
  // tests: skew 1 makes a team wait for a launch that does not come (until the
  // wait's limit), spread 1 forms it from the first blocks of the grid
  int skew = 0, spread = 0;
};

constexpr int kSiteInlineW = 32;  // weights a launch takes in its arguments, at most
struct SiteArgs {
  PersistArgs p;
  int inline_w;            // weights in w (0: in p.wts)
  double w[kSiteInlineW];
  const PElem* e;
  int set_term[2];
  const double* diag;
  int diag_term;
  int tl, blocks;
  void* rec;
  unsigned long long* ids;
  unsigned long long* count;
  int skew, spread;        // (DevSite)
};

// Sets up the plan's kernel; *fits: a launch's blocks are co-resident.
hipError_t site_prepare(const SitePlan& P, bool real, int num_cus, bool* fits);
// The device side of S->plan: one allocation (S->rec), one copy.
hipError_t site_upload(const ParityForm& F, DevSite* S);
// A whole call (see PersistArgs; basis, psi, wts and the exports are used).
// host_wts: p.wts is a host table of nwts <= kSiteInlineW weights
hipError_t launch_site(const DevSite& S, const PersistArgs& args, hipStream_t st, int nwts = 0);

}  // namespace cfet
