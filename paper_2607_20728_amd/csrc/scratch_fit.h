// How kept scratch grows, and what it falls back to when the device is nearly
// full.  Host only; the allocations come in as callables.
#pragma once
#include <algorithm>

#include "../../include/bsex.h"

namespace bsex {

// Lengths in elements.  A workspace of `have` that has to hold `need` grows by
// more than was asked, so that a solver's growing products do not replace it at
// every step, but only where that fits: alloc(length) is asked for `need` alone
// when the longer one is out of memory.
template <class Alloc>
int grow_scratch(long have, long need, Alloc&& alloc) {
  const long roomy = std::max(need, std::min(2 * have, have + (4L << 20)));
  const int rc = alloc(roomy);
  return rc == BSE_ENOMEM && roomy > need ? alloc(need) : rc;
}

// Scratch for `want` sets at a time, or for one where that is out of memory:
// drop() then gives back everything that a failed alloc(want) left, and *limit
// (0: none yet) keeps later calls from trying again.  *sets: what there is.
template <class Alloc, class Drop>
int fit_sets(int want, int* limit, Alloc&& alloc, Drop&& drop, int* sets) {
  *sets = *limit > 0 ? std::min(want, *limit) : want;
  const int rc = alloc(*sets);
  if (rc != BSE_ENOMEM || *sets == 1) return rc;
  drop();
  *limit = *sets = 1;
  return alloc(1);
}

}  // namespace bsex
