// Where a double-precision kernel finds what it needs of the cards.
#pragma once

#include "check.h"
#include "kernels.h"

namespace rwgt {

// Up to kArgCards of them are arguments of the launch (at most 2 KB of the 4 KB
// a launch may carry, one scalar load each): no copy goes ahead of the kernel,
// which for 10,000 events took as long as the kernel itself (with that and the
// count of non-finite outputs made by the kernel, rwgt_eval of 10,000
// e+ e- -> mu+ mu- events takes 11 us instead of 20).  More are a table that
// the caller uploaded.
template <class C> struct ArgCards {
  C c[kArgCards];
  __device__ __forceinline__ const C& operator()(int k) const { return c[k]; }
};
template <class C> struct TableCards {
  const C* p;
  int n;
  __device__ __forceinline__ const C& operator()(int k) const { return RWGT_AT(p, k, n); }
};


template <class C, class OF>
inline size_t card_table(const CardPair* cards, int n, void* out, OF of) {
  static_assert(sizeof(C) <= sizeof(CardPair) && kArgCards * sizeof(C) <= 2048, "fits the upload and the launch");
  for (int k = 0; k < n; ++k) static_cast<C*>(out)[k] = of(cards[k].d);
  return size_t(n) * sizeof(C);
}

// f(source) with the call's cards as arguments or as the uploaded table.
template <class C, class OF, class F>
inline hipError_t with_cards(const Fp64Call& a, OF of, F f) {
  if (a.ncards > kArgCards) return f(TableCards<C>{static_cast<const C*>(a.table), a.ncards});
  ArgCards<C> c{};
  card_table<C>(a.cards, a.ncards, c.c, of);
  return f(c);
}

}  // namespace rwgt
