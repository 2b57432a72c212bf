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

}  // namespace bsex
