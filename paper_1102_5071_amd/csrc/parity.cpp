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

struct Value {
  uint64_t re = 0, im = 0;  // bit patterns; 0, 0 also where nothing is stored
  bool operator==(const Value& o) const { return re == o.re && im == o.im; }
  void get(double* out) const { std::memcpy(out, this, sizeof(*this)); }
};
Value value_of(const double* v) {
  Value x;
  std::memcpy(&x, v, sizeof(x));
  return x;
}

// One (operator term, offset): its two values, the mask that picks one, and how
// many rows store an entry of it that is not 0.
struct Cand {
  uint32_t off, pmask;
  int term;
  Value v[2];
  int64_t count;
  uint8_t nonzero[2];  // v[p] is not 0
};

// Candidates with an open-addressing index.
struct Table {
  static constexpr uint32_t kSize = 1024;
  static constexpr int kPlaces = 64;
  std::vector<Cand> c;
  int16_t slot[kSize];
  // the candidate of the last row's entry at this place of this term: the next
  // row's is often the same
  int16_t guess[kMaxTerms + 1][kPlaces] = {};
  Table() {
    std::fill(slot, slot + kSize, int16_t(-1));
    c.reserve(kParityMaxTerms + 1);
  }
  static uint32_t hash(uint32_t off, int term) {
    return ((off * 0x9E3779B1u) ^ (uint32_t(term) * 0x85EBCA6Bu)) >> 22;
  }
  int find(uint32_t off, int term) const {
    for (uint32_t h = hash(off, term);; h = (h + 1) % kSize) {
      const int i = slot[h];
      if (i < 0 || (c[i].off == off && c[i].term == term)) return i;
    }
  }
  // false: there are too many
  bool add(uint32_t off, int term) {
    uint32_t h = hash(off, term);
    for (; slot[h] >= 0; h = (h + 1) % kSize)
      if (c[slot[h]].off == off && c[slot[h]].term == term) return true;
    if (c.size() >= size_t(kParityMaxTerms)) return false;
    slot[h] = int16_t(c.size());
    c.push_back({off, 0u, term, {}, 0, {}});
    return true;
  }
  // find, of the entry at this place of a row (g: guess[term], p: c, not empty)
  int at(int16_t* g, const Cand* p, uint32_t off, int term, int64_t place) const {
    int i = g[place & (kPlaces - 1)];
    if (p[i].off == off && p[i].term == term) return i;
    i = find(off, term);
    if (i >= 0) g[place & (kPlaces - 1)] = int16_t(i);
    return i;
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

inline uint32_t parity32(uint32_t v) { return uint32_t(__builtin_parity(v)); }

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
  // A value that depends on one parity of the row's bits is told by row 0 and by
  // the rows of a single bit: those give every term, its two values and its mask.
  Table all;
  for (int i = -1; i < nb; ++i) {
    const int64_t r = i < 0 ? 0 : int64_t(1) << i;
    for (int k = 0; k <= nterms; ++k)
      for (int64_t q = mats[k].rp[r]; q < mats[k].rp[r + 1]; ++q) {
        const uint32_t off = uint32_t(int64_t(mats[k].col[q]) ^ r);
        if (off != 0 && !all.add(off, k)) return false;
      }
  }
  auto value_at = [&](const Cand& k, int64_t r) {
    const HostCSR& h = mats[k.term];
    Value v;
    for (int64_t q = h.rp[r]; q < h.rp[r + 1]; ++q)
      if (uint32_t(int64_t(h.col[q]) ^ r) == k.off) v = value_of(h.val + 2 * q);
    return v;
  };
  for (Cand& k : all.c) {
    const Value a = value_at(k, 0);
    Value b = a;
    for (int i = 0; i < nb; ++i) {
      const Value vi = value_at(k, int64_t(1) << i);
      if (vi == a) continue;
      if (!(b == a) && !(vi == b)) return false;  // a third value
      b = vi;
      k.pmask |= 1u << i;
    }
    if (k.pmask == 0 && a == Value{}) return false;  // stored zeros
    k.v[0] = a;
    k.v[1] = b;
    for (int p = 0; p < 2; ++p) {
      double v[2];
      k.v[p].get(v);
      k.nonzero[p] = v[0] != 0.0 || v[1] != 0.0;
    }
  }
  // every stored value against the form, and every value the form says that is
  // not stored (counted: the rows whose value is not 0 must be there)
  nth = std::max(1u, nth);
  std::vector<Table> tab(nth, all);
  std::atomic<bool> good{true};
  std::vector<int32_t> diag_terms(nth, 0);
  F->diag.assign(size_t(n), 0.0);
  on_threads(n, nth, [&](unsigned t, int64_t r0, int64_t r1) {
    Table& T = tab[t];
    Cand* const cand = T.c.data();
    double* const diag = F->diag.data();
    int32_t dt = 0;
    for (int64_t r = r0; r < r1; ++r) {
      if ((r & 4095) == 0 && !good.load(std::memory_order_relaxed)) return;
      for (int k = 0; k <= nterms; ++k) {
        const int64_t q0 = mats[k].rp[r], q1 = mats[k].rp[r + 1];
        const int32_t* const col = mats[k].col;
        const double* const val = mats[k].val;
        for (int64_t q = q0; q < q1; ++q) {
          const uint32_t off = uint32_t(int64_t(col[q]) ^ r);
          if (off == 0) {
            dt |= 1 << k;
            diag[r] = val[2 * q];
            if (val[2 * q + 1] == 0.0) continue;
            good.store(false);
            return;
          }
          const int i = T.c.empty() ? -1 : T.at(T.guess[k], cand, off, k, q - q0);
          if (i >= 0) {
            Cand& c = cand[i];
            const uint32_t p = parity32(uint32_t(r) & c.pmask);
            bool same = value_of(val + 2 * q) == c.v[p];
            if (!same) {  // a zero of the other sign
              double v[2];
              c.v[p].get(v);
              same = v[0] == val[2 * q] && v[1] == val[2 * q + 1];
            }
            if (same) {
              c.count += c.nonzero[p];
              continue;
            }
          }
          good.store(false);
          return;
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
  if (F->diag_term < 0) F->diag.clear();
  for (size_t i = 0; i < all.c.size(); ++i) {
    Cand& k = all.c[i];
    for (const Table& T : tab) k.count += T.c[i].count;
    if (k.count != (n / 2) * (k.nonzero[0] + k.nonzero[1])) return false;
  }
  std::sort(all.c.begin(), all.c.end(), [](const Cand& a, const Cand& b) {
    return a.off != b.off ? a.off < b.off : a.term < b.term;
  });
  for (const Cand& k : all.c) {
    ParityTerm p{k.off, k.pmask, k.term, {0.0, 0.0}, {0.0, 0.0}};
    k.v[0].get(p.v0);
    k.v[1].get(p.v1);
    if (p.v0[1] != 0.0 || p.v1[1] != 0.0) F->real = false;
    F->terms.push_back(p);
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
