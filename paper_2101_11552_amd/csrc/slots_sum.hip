// The slot aggregation (slots.h): sums, one weight per edge or none.
#include "slots.h"

namespace tfg {
namespace rows {

void slots_sum(int vec, int lps, bool narrow, const SlotLists& L, int waves, const RowArgs& a,
               hipStream_t s) {
  if (a.w != nullptr) {
    if (vec == 4) by_lps<4, kSum, kEdge>(lps, narrow, L, waves, a, s);
    else run<1, 4, kSum, kEdge>(narrow, L, waves, a, s);
  } else {
    if (vec == 4) by_lps<4, kSum, kNone>(lps, narrow, L, waves, a, s);
    else run<1, 4, kSum, kNone>(narrow, L, waves, a, s);
  }
}

}  // namespace rows
}  // namespace tfg
