// The fused attention kernel (gat_slots.h) with scaled dot-product scores.
#include "gat_slots.h"

namespace tfg {
namespace rows {

void gat_dot(const GatShape& t, bool narrow, const SlotLists& L, int waves, const int* col, int H,
             int D, const Scores& S, const float* h, const GatOut& O, hipStream_t s) {
  gat_dispatch<true>(t, narrow, L, waves, col, H, D, S, h, O, s);
}

}  // namespace rows
}  // namespace tfg
