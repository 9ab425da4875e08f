// The slot aggregation (slots.h): masked sums, the gather of the max gradient.
#include "slots.h"

namespace tfg {
namespace rows {

void slots_masked(int vec, int lps, bool narrow, const SlotLists& L, int waves, const RowArgs& a,
                  hipStream_t s) {
  if (a.w != nullptr && a.H > 1) {
    if (vec == 4) by_lps<4, kMasked, kHeads>(lps, narrow, L, waves, a, s);
    else by_lps<1, kMasked, kHeads>(lps, narrow, L, waves, a, s);
  } else if (a.w != nullptr) {
    if (vec == 4) by_lps<4, kMasked, kEdge>(lps, narrow, L, waves, a, s);
    else run<1, 4, kMasked, kEdge>(narrow, L, waves, a, s);
  } else {
    if (vec == 4) by_lps<4, kMasked, kNone>(lps, narrow, L, waves, a, s);
    else run<1, 4, kMasked, kNone>(narrow, L, waves, a, s);
  }
}

}  // namespace rows
}  // namespace tfg
