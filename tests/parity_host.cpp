// Recognition of the site-operator form when memory runs out: every allocation
// in turn fails, on whichever thread makes it.  Prints the allocations of an
// undisturbed run and how many of the disturbed ones still found the form.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "parity.h"

static std::atomic<long> count{0}, fail_at{-1};

void* operator new(std::size_t n) {
  if (count.fetch_add(1) == fail_at.load()) throw std::bad_alloc();
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

static cfet::HostCSR chain(int L, bool bonds) {
  cfet::HostCSR h{};
  const int64_t n = int64_t(1) << L;
  h.rp_buf.push_back(0);
  for (int64_t r = 0; r < n; ++r) {
    auto put = [&](int64_t c, double v) {
      h.col_buf.push_back(int32_t(c));
      h.val_buf.push_back(v);
      h.val_buf.push_back(0.0);
    };
    if (bonds) put(r, double(r % 7));
    for (int i = 0; i < L; ++i) {
      if (!bonds) put(r ^ (int64_t(1) << i), 1.0);
      else if (i + 1 < L && (((r >> i) ^ (r >> (i + 1))) & 1)) put(r ^ (int64_t(3) << i), 2.0);
    }
    h.rp_buf.push_back(int64_t(h.col_buf.size()));
  }
  h.n = n;
  h.nnz = int64_t(h.col_buf.size());
  return h;
}

int main() {
  std::vector<cfet::HostCSR> mats;
  mats.push_back(chain(16, true));
  mats.push_back(chain(16, false));
  for (auto& h : mats) {
    h.rp = h.rp_buf.data();
    h.col = h.col_buf.data();
    h.val = h.val_buf.data();
  }
  auto run = [&](long fail) {
    count = 0;
    fail_at = fail;
    bool ok = false;
    try {  // as the caller has it
      cfet::ParityForm form;
      cfet::ParityPlan plan;
      ok = cfet::find_parity_form(mats, 1, mats[0].n, 8, &form) && cfet::plan_parity(form, &plan) &&
           form.terms.size() == 31 && form.diag_term == 0;
    } catch (const std::bad_alloc&) {
    }
    fail_at = -1;
    return ok;
  };
  const bool plain = run(-1);
  const long total = count;
  int found = 0;
  for (long k = 0; k < total; ++k) found += run(k);
  std::printf("%d %ld %d\n", plain ? 1 : 0, total, found);
  return 0;
}
