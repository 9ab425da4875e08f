// Shared by the kernels of the message aggregation (gfx950, wave64):
//
// out[t, :] = reduce over the edges k of row t of w_k * x[col_k, :].
//
// The slot kernel (slots.h) serves every form of it; sums over the part plan of
// 128-column rows go one item per wavefront (spmm_wide, aggregate.hip). A row
// is a work item, or the chunks of at most `chunk` edges of a long row are, or
// its (row, source part) segments; items that are not whole rows leave partial
// rows that fixup_rows combines in a fixed order. Partial chains are short and
// combined pairwise, so the float32 error stays small for long rows too. No
// floating-point atomics: every output is reproducible bit for bit.
#pragma once

#include "wave.h"

namespace tfg {
namespace rows {

// Vectors of a row's columns. gfx950's global loads and stores need dword
// alignment only, so they serve rows of any width and leading dimension.
typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int i2 __attribute__((ext_vector_type(2), aligned(4)));
typedef int i4 __attribute__((ext_vector_type(4), aligned(4)));

template <int V>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[V]) {
  if constexpr (V == 4) {
    f4 t = *reinterpret_cast<const f4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (V == 2) {
    f2 t = *reinterpret_cast<const f2*>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *p;
  }
}

// The same, for data read once (streamed past the L2).
template <int V>
__device__ __forceinline__ void load_row_once(const float* __restrict__ p, float (&v)[V]) {
  if constexpr (V == 4) {
    f4 t = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (V == 2) {
    f2 t = __builtin_nontemporal_load(reinterpret_cast<const f2*>(p));
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = __builtin_nontemporal_load(p);
  }
}

template <int V>
__device__ __forceinline__ void load_irow(const int* __restrict__ p, int (&v)[V]) {
  if constexpr (V == 4) {
    i4 t = *reinterpret_cast<const i4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (V == 2) {
    i2 t = *reinterpret_cast<const i2*>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *p;
  }
}

template <int V>
__device__ __forceinline__ void store_row(float* __restrict__ p, const float (&v)[V]) {
  if constexpr (V == 4) {
    f4 t = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(t, reinterpret_cast<f4*>(p));
  } else if constexpr (V == 2) {
    f2 t = {v[0], v[1]};
    __builtin_nontemporal_store(t, reinterpret_cast<f2*>(p));
  } else {
    __builtin_nontemporal_store(v[0], p);
  }
}

template <int V>
__device__ __forceinline__ void store_irow(int* __restrict__ p, const int (&v)[V]) {
  if constexpr (V == 4) {
    i4 t = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(t, reinterpret_cast<i4*>(p));
  } else if constexpr (V == 2) {
    i2 t = {v[0], v[1]};
    __builtin_nontemporal_store(t, reinterpret_cast<i2*>(p));
  } else {
    __builtin_nontemporal_store(v[0], p);
  }
}

// Output transform of a propagation step: y = scale * sum + alpha * h[row]
// (APPNP, SGC); the identity (scale 1, no h) for a plain aggregation.
struct Epilogue {
  float scale, alpha;
  const float* h;
  int64_t ldh;
};

template <int V>
__device__ __forceinline__ void apply_epilogue(const Epilogue& ep, int row, int f, float (&v)[V]) {
  if (ep.h != nullptr) {
    float t[V];
    load_row<V>(ep.h + (int64_t)row * ep.ldh + f, t);
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = __builtin_fmaf(ep.alpha, t[i], ep.scale * v[i]);
  } else if (ep.scale != 1.0f) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = ep.scale * v[i];
  }
}

// Max with the smallest edge id winning ties; arg < 0 marks "no edge yet".
__device__ __forceinline__ void max_combine(float& v, int& a, float vb, int ab) {
  bool take = ab >= 0 && (a < 0 || vb > v || (vb == v && ab < a));
  v = take ? vb : v;
  a = take ? ab : a;
}

// Threads per block of the item kernels: one wavefront. The wavefronts are
// independent, and single-wavefront blocks let a CU start the next item as
// soon as any wavefront ends (aggregation on the power-law graph: 3.60 ms,
// against 3.65 / 3.71 / 4.10 / 4.98 ms with 128- to 1024-thread blocks).
constexpr int kRowBlock = kItemBlock;

// The kernel arguments shared by every instantiation.
struct RowArgs {
  const WorkItem* heavy;  // the items that write partial rows
  int n_heavy;
  const int* col;
  const int* perm;
  const float* w;
  int w_by_perm, H, per_head;
  const float* x;
  int64_t ldx;
  const int* mask;
  int F, mean;
  float* out;
  int* argout;
  float* part;
  int* part_arg;
  Epilogue ep;
};

// Work items in edge slots (slots.h): up to kSlotLists lists in one launch,
// an item of list i handled by split[i] neighbouring slots of one wavefront,
// waves[i] wavefronts per list.
constexpr int kSlotLists = 4;
struct SlotLists {
  const WorkItem* items[kSlotLists];
  int n[kSlotLists];
  int split[kSlotLists];
  int waves[kSlotLists];
};
// Fills L for a plan's items (pieces: those that write partials; the row plan's
// whole rows follow) and lps lanes per slot, and counts the wavefronts.
void slot_lists(const Graph& g, const WorkItem* pieces, int n_pieces, bool part_plan, int lps,
                bool heads, SlotLists& L, int* waves);
void slots_sum(int vec, int lps, bool narrow, const SlotLists& L, int waves, const RowArgs& a,
               hipStream_t s);
void slots_masked(int vec, int lps, bool narrow, const SlotLists& L, int waves, const RowArgs& a,
                  hipStream_t s);
void slots_max(bool ties, int vec, int lps, bool narrow, const SlotLists& L, int waves,
               const RowArgs& a, hipStream_t s);
void slots_heads(bool mx, int vec, int lps, bool narrow, const SlotLists& L, int waves,
                 const RowArgs& a, hipStream_t s);

}  // namespace rows
}  // namespace tfg
