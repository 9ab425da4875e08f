// The slot aggregation (slots.h) with one weight per edge and head.
#include "slots.h"

namespace tfg {
namespace rows {

void slots_heads(bool mx, int vec, int lps, bool narrow, const SlotLists& L, int waves,
                 const RowArgs& a, hipStream_t s) {
  if (mx) {
    if (vec == 4) by_lps<4, kMaxTies, kHeads>(lps, narrow, L, waves, a, s);
    else by_lps<1, kMaxTies, kHeads>(lps, narrow, L, waves, a, s);
  } else {
    if (vec == 4) by_lps<4, kSum, kHeads>(lps, narrow, L, waves, a, s);
    else if (vec == 2) by_lps<2, kSum, kHeads>(lps, narrow, L, waves, a, s);
    else by_lps<1, kSum, kHeads>(lps, narrow, L, waves, a, s);
  }
}

}  // namespace rows
}  // namespace tfg
