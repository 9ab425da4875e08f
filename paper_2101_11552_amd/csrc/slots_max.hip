// The slot aggregation (slots.h): maxima with argmax, one weight per edge or none.
#include "slots.h"

namespace tfg {
namespace rows {

void slots_max(bool ties, int vec, int lps, bool narrow, const SlotLists& L, int waves,
               const RowArgs& a, hipStream_t s) {
  if (a.w != nullptr) {
    if (vec == 4 && ties) by_lps<4, kMaxTies, kEdge>(lps, narrow, L, waves, a, s);
    else if (vec == 4) by_lps<4, kMax, kEdge>(lps, narrow, L, waves, a, s);
    else run<1, 4, kMaxTies, kEdge>(narrow, L, waves, a, s);
  } else {
    if (vec == 4 && ties) by_lps<4, kMaxTies, kNone>(lps, narrow, L, waves, a, s);
    else if (vec == 4) by_lps<4, kMax, kNone>(lps, narrow, L, waves, a, s);
    else run<1, 4, kMaxTies, kNone>(narrow, L, waves, a, s);
  }
}

}  // namespace rows
}  // namespace tfg
