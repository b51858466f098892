// Recognition of the site-operator form (parity.h) and the plan of its sweeps.
#include "parity.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>
#include <thread>

namespace cfet {

namespace {

uint64_t bits_of(double v) {
  uint64_t u;
  std::memcpy(&u, &v, sizeof(u));
  return u;
}

struct Value {
  uint64_t re = 0, im = 0;  // bit patterns; 0, 0 also where nothing is stored
  bool operator==(const Value& o) const { return re == o.re && im == o.im; }
};

// Per (term, offset): the distinct values its rows hold and how many rows do.
struct Cand {
  uint32_t off;
  int term;
  int nval;
  Value val[2];
  int64_t count;
};

// Candidates in order of first appearance with an open-addressing index.
struct Table {
  static constexpr uint32_t kSize = 1024;
  std::vector<Cand> c;
  int16_t slot[kSize];
  bool full = false;
  Table() {
    std::fill(slot, slot + kSize, int16_t(-1));
    c.reserve(kParityMaxTerms + 1);  // threads fill it, which may not throw
  }
  static uint32_t hash(uint32_t off, int term) {
    return ((off * 0x9E3779B1u) ^ (uint32_t(term) * 0x85EBCA6Bu)) >> 22;
  }
  int find(uint32_t off, int term) const {
    for (uint32_t h = hash(off, term);; h = (h + 1) % kSize) {
      const int i = slot[h];
      if (i < 0) return -1;
      if (c[i].off == off && c[i].term == term) return i;
    }
  }
  int get(uint32_t off, int term) {
    for (uint32_t h = hash(off, term);; h = (h + 1) % kSize) {
      const int i = slot[h];
      if (i >= 0) {
        if (c[i].off == off && c[i].term == term) return i;
        continue;
      }
      if (c.size() > size_t(kParityMaxTerms)) {
        full = true;
        return -1;
      }
      slot[h] = int16_t(c.size());
      c.push_back({off, term, 0, {}, 0});
      return int(c.size()) - 1;
    }
  }
  // false: a third distinct value
  static bool add_value(Cand& k, const Value& v) {
    for (int i = 0; i < k.nval; ++i)
      if (k.val[i] == v) return true;
    if (k.nval == 2) return false;
    k.val[k.nval++] = v;
    return true;
  }
};

// body(t, first, last) for nth parts of [0, count); body does not throw.  A part
// whose thread cannot be started runs here.
template <class Body>
void on_threads(int64_t count, unsigned nth, Body body) {
  if (nth <= 1) {
    body(0u, int64_t(0), count);
    return;
  }
  std::vector<std::thread> pool;
  pool.reserve(nth);
  for (unsigned t = 0; t < nth; ++t) {
    auto part = [&, t]() { body(t, count * t / nth, count * (t + 1) / nth); };
    try {
      pool.emplace_back(part);
    } catch (...) {
      part();
    }
  }
  for (auto& th : pool) th.join();
}

inline uint32_t parity32(uint32_t v) { return uint32_t(__builtin_popcount(v)) & 1u; }

}  // namespace

bool find_parity_form(const std::vector<HostCSR>& mats, int nterms, int64_t n, unsigned nth,
                      ParityForm* F) try {
  int nb = 0;
  while ((int64_t(1) << nb) < n) ++nb;
  if ((int64_t(1) << nb) != n || nb > kParityMaxBits) return false;
  F->nb = nb;
  F->nterms = nterms;
  // a first look at a few rows turns most other operators away at once
  for (int64_t r = 0; r < n; r += std::max<int64_t>(1, n / 8)) {
    int64_t len = 0;
    for (int k = 0; k <= nterms; ++k) len += mats[k].rp[r + 1] - mats[k].rp[r];
    if (len > kParityMaxTerms + nterms + 1) return false;
  }
  nth = std::max(1u, nth);
  std::vector<Table> tab(nth);
  std::atomic<bool> good{true};
  std::vector<int32_t> diag_terms(nth, 0);
  on_threads(n, nth, [&](unsigned t, int64_t r0, int64_t r1) {
    Table& T = tab[t];
    int32_t dt = 0;
    for (int64_t r = r0; r < r1; ++r) {
      if ((r & 4095) == 0 && !good.load(std::memory_order_relaxed)) return;
      for (int k = 0; k <= nterms; ++k) {
        const HostCSR& h = mats[k];
        for (int64_t q = h.rp[r]; q < h.rp[r + 1]; ++q) {
          const uint32_t off = uint32_t(int64_t(h.col[q]) ^ r);
          const double re = h.val[2 * q], im = h.val[2 * q + 1];
          if (off == 0) {
            dt |= 1 << k;
            if (im != 0.0) {
              good.store(false);
              return;
            }
            continue;
          }
          const int i = T.get(off, k);
          if (i < 0 || !Table::add_value(T.c[i], Value{bits_of(re), bits_of(im)})) {
            good.store(false);
            return;
          }
          T.c[i].count += 1;
        }
      }
    }
    diag_terms[t] = dt;
  });
  if (!good.load()) return false;
  int32_t dt = 0;
  for (int32_t d : diag_terms) dt |= d;
  if (dt & (dt - 1)) return false;
  for (int k = 0; k <= nterms; ++k)
    if (dt == (1 << k)) F->diag_term = k;
  Table all;
  for (const Table& T : tab)
    for (const Cand& k : T.c) {
      const int i = all.get(k.off, k.term);
      if (i < 0) return false;
      for (int v = 0; v < k.nval; ++v)
        if (!Table::add_value(all.c[i], k.val[v])) return false;
      all.c[i].count += k.count;
    }
  if (all.c.size() > size_t(kParityMaxTerms)) return false;
  std::sort(all.c.begin(), all.c.end(), [](const Cand& a, const Cand& b) {
    return a.off != b.off ? a.off < b.off : a.term < b.term;
  });
  auto value_at = [&](const Cand& k, int64_t r) {
    const HostCSR& h = mats[k.term];
    for (int64_t q = h.rp[r]; q < h.rp[r + 1]; ++q)
      if (uint32_t(int64_t(h.col[q]) ^ r) == k.off)
        return Value{bits_of(h.val[2 * q]), bits_of(h.val[2 * q + 1])};
    return Value{};
  };
  auto put = [](const Value& v, double* out) {
    std::memcpy(&out[0], &v.re, 8);
    std::memcpy(&out[1], &v.im, 8);
  };
  bool two_valued = false;
  for (const Cand& k : all.c) {
    ParityTerm p{k.off, 0u, k.term, {0.0, 0.0}, {0.0, 0.0}};
    if (k.nval == 1 && k.count == n) {
      put(k.val[0], p.v0);
      put(k.val[0], p.v1);
    } else {
      // rows without an entry hold 0, the second value
      const Value zero{};
      Value a = k.val[0], b = k.nval == 2 ? k.val[1] : zero;
      if (k.count != n && k.nval == 2) {
        if (a == zero) a = b;  // stored zeros
        else if (!(b == zero)) return false;
        b = zero;
      }
      const Value at0 = value_at(k, 0);
      if (!(at0 == a) && !(at0 == b)) return false;
      for (int i = 0; i < nb; ++i) {
        const Value vi = value_at(k, int64_t(1) << i);
        if (!(vi == a) && !(vi == b)) return false;
        if (!(vi == at0)) p.pmask |= 1u << i;
      }
      put(at0, p.v0);
      put(at0 == a ? b : a, p.v1);
      if (p.pmask == 0) return false;
      two_valued = true;
    }
    if (p.v0[1] != 0.0 || p.v1[1] != 0.0) F->real = false;
    F->terms.push_back(p);
  }
  if (two_valued) {
    // every stored value against the form, and every value the form says that
    // is not stored (counted: the rows whose value is not 0 must be there)
    std::vector<std::vector<int64_t>> seen(nth, std::vector<int64_t>(all.c.size(), 0));
    Table idx;
    for (size_t i = 0; i < all.c.size(); ++i) idx.get(all.c[i].off, all.c[i].term);
    on_threads(n, nth, [&](unsigned t, int64_t r0, int64_t r1) {
      for (int64_t r = r0; r < r1; ++r) {
        if ((r & 4095) == 0 && !good.load(std::memory_order_relaxed)) return;
        for (int k = 0; k <= nterms; ++k) {
          const HostCSR& h = mats[k];
          for (int64_t q = h.rp[r]; q < h.rp[r + 1]; ++q) {
            const uint32_t off = uint32_t(int64_t(h.col[q]) ^ r);
            if (off == 0) continue;
            const int i = idx.find(off, k);
            const ParityTerm& p = F->terms[i];
            const double* v = parity32(uint32_t(r) & p.pmask) ? p.v1 : p.v0;
            if (v[0] != h.val[2 * q] || v[1] != h.val[2 * q + 1]) {
              good.store(false);
              return;
            }
            if (v[0] != 0.0 || v[1] != 0.0) seen[t][i] += 1;
          }
        }
      }
    });
    if (!good.load()) return false;
    for (size_t i = 0; i < all.c.size(); ++i) {
      const ParityTerm& p = F->terms[i];
      const bool n0 = p.v0[0] != 0.0 || p.v0[1] != 0.0, n1 = p.v1[0] != 0.0 || p.v1[1] != 0.0;
      int64_t want = 0, have = 0;
      if (p.pmask == 0) want = n0 ? n : 0;
      else want = (n0 ? n / 2 : 0) + (n1 ? n / 2 : 0);
      for (unsigned t = 0; t < nth; ++t) have += seen[t][i];
      if (want != have) return false;
    }
  }
  if (F->diag_term >= 0) {
    F->diag.assign(size_t(n), 0.0);
    const HostCSR& h = mats[F->diag_term];
    on_threads(n, nth, [&](unsigned, int64_t r0, int64_t r1) {
      for (int64_t r = r0; r < r1; ++r)
        for (int64_t q = h.rp[r]; q < h.rp[r + 1]; ++q)
          if (int64_t(h.col[q]) == r) F->diag[size_t(r)] = h.val[2 * q];
    });
  }
  return true;
} catch (const std::bad_alloc&) {
  return false;  // the caller falls back to its general layouts
}

namespace {

// Tiles of the two sweeps and the low row bits of the first, by size.  Large
// vectors want long contiguous segments in the first sweep (the chain of 24:
// 606, 466 and 456 us per iteration with 64, 128 and 256-byte segments) at
// the price of a few more gathered terms in the second; vectors that the
// memory-side cache holds want the fewest gathered terms; small ones want a
// tile for every CU (2^18 rows: 17.0 us with 2^10-row tiles, 23.1 with 2^11).
// The two sizes between, by measurement (Ising chain, one step): 2^21 rows 5.23 ms
// with the second sweep on 2^12-row tiles, 5.39 on 2^11; 2^22 rows, whose working
// set is at the edge of that cache, 10.4 ms with 128-byte segments, 12.0 with
// 64-byte ones and 12.4 with those and 2^12-row tiles in the second sweep.
void tiles_of(int nb, int* tbh, int* tbl, int* low) {
  if (nb >= 23) {
    *tbh = *tbl = 12;
    *low = nb >= 25 ? 3 : 4;
  } else {
    *tbh = nb >= 19 ? 11 : nb >= 17 ? 10 : 9;
    *tbl = nb == 21 ? 12 : *tbh;
    *low = nb == 22 ? 3 : 2;
  }
}

}  // namespace

std::vector<ParityTerm> merge_terms(const std::vector<ParityTerm>& terms) {
  std::vector<ParityTerm> out;
  for (const ParityTerm& t : terms) {
    bool done = false;
    for (ParityTerm& o : out) {
      if (o.off != t.off || o.term == t.term || o.term2 >= 0) continue;
      if (o.pmask != t.pmask && o.pmask != 0 && t.pmask != 0) continue;
      if (o.pmask == 0) o.pmask = t.pmask;
      o.term2 = t.term;
      for (int c = 0; c < 2; ++c) {
        o.b0[c] = t.v0[c];
        o.b1[c] = t.v1[c];
      }
      done = true;
      break;
    }
    if (!done) out.push_back(t);
  }
  return out;
}

bool plan_parity(const ParityForm& F, ParityPlan* P) try {
  const int nb = F.nb;
  if (nb < kParityMinBits) return false;
  int tbh, tbl, low;
  tiles_of(nb, &tbh, &tbl, &low);
  // first high bit: the topmost bit of the second sweep's tile as well where
  // there is room, so that a bond across the two needs no gather
  const int s = std::max(nb + low - tbh, tbl - 1);
  low = tbh - (nb - s);
  P->nb = nb;
  P->tbh = tbh;
  P->tbl = tbl;
  P->low = low;
  P->high = s;
  const uint32_t himask = (~0u << s) | ((1u << low) - 1u);
  const std::vector<ParityTerm> terms = merge_terms(F.terms);
  for (const ParityTerm& t : terms) {
    if ((t.off >> tbl) == 0) P->lo.push_back(t);
    else if ((t.off & ~himask) == 0) P->hi.push_back(t);
    else P->far.push_back(t);
  }
  // gathered terms cost a read of the vector from beyond the tile each: more
  // than a quarter of the terms and the other layouts serve better
  return 4 * P->far.size() <= terms.size() + 3;
} catch (const std::bad_alloc&) {
  return false;
}

}  // namespace cfet
