// Softmax statistics merged online (device code): a pair (m, d) stands for a
// set of scores with maximum m and d = sum of exp(s - m) (in double). Adding
// a score or merging two pairs rescales d to the larger maximum, so a
// segment's maximum and denominator come out of one sweep, in any grouping;
// an empty set is (-inf, 0). Both operations are symmetric in their operands
// (IEEE addition and multiplication commute), so xor butterflies leave every
// lane with the same pair.
#pragma once

#include "wave.h"

namespace tfg {

__device__ __forceinline__ void stat_merge(float& m, double& d, float m2, double d2) {
#pragma clang fp contract(off)
  if (m2 == -__builtin_huge_valf()) return;
  if (m == -__builtin_huge_valf()) {
    m = m2;
    d = d2;
    return;
  }
  const float mn = m2 > m ? m2 : m;
  d = d * (double)expf(m - mn) + d2 * (double)expf(m2 - mn);
  m = mn;
}

// One exponential per score: t = exp(-|v - m|) is the new term when the
// maximum stays and the rescale factor of d when it grows (from m = -inf the
// factor is 0). A score of -inf adds nothing, also to an empty pair.
__device__ __forceinline__ void stat_add(float& m, double& d, float v) {
#pragma clang fp contract(off)
  const float dlt = v - m;
  const float t = v == -__builtin_huge_valf() ? 0.0f : expf(-__builtin_fabsf(dlt));
  const bool up = dlt > 0.0f;
  d = up ? d * (double)t + 1.0 : d + (double)t;
  m = up ? v : m;
}

// Rows and chunks of long rows, several per wavefront:
// an item takes a group of `lanes` neighbouring lanes, which are (slot, head)
// pairs: HP heads (a power of two) and SL = lanes / HP slots; slot step u of an item
// starting at kb is position kb + slot + u * SL. Where H is a multiple of 4 a lane
// holds K = 4 heads of an edge (16-byte accesses), and HP, H count these fours.
// One wavefront per item and one head per lane left most lanes with one or two
// values, and the butterflies, the round trips on each row's extent and the 4-byte
// accesses set the pace.
template <int K>
constexpr int group_steps() { return K == 4 ? 4 : 8; }  // slot steps held in registers

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
template <int K>
__device__ __forceinline__ void load_k(const float* __restrict__ p, float (&v)[K]) {
  if constexpr (K == 4) {
    const f4u t = *reinterpret_cast<const f4u*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    v[0] = *p;
  }
}
template <int K>
__device__ __forceinline__ void store_k(float* __restrict__ p, const float (&v)[K]) {
  if constexpr (K == 4) *reinterpret_cast<f4u*>(p) = f4u{v[0], v[1], v[2], v[3]};
  else *p = v[0];
}

// HP for H heads: every head in one pass where 64 lanes hold them, some lanes
// idle. (The largest power of two within H idles as many in its last pass and
// reads the ids and the scattered lines of the caller's order twice: 8M edges, 3
// heads, 619 us.)
inline int heads_per_pass(int H) {
  int hp = 1;
  while (hp < H && hp < kWave) hp <<= 1;
  return hp;
}

constexpr int kGroupLists = 5;
struct RowGroups {
  const WorkItem* items[kGroupLists];
  int n[kGroupLists];
  int lanes[kGroupLists];
  int waves[kGroupLists];
};

// The plan's lists, longest items first, and the number of wavefronts. A list of
// items of at most `edges` edges takes as many slots as leave a lane its steps, and
// at least 64 bytes per step of a row (or all its edges). The short rows take the
// latter only while their lanes leave part of the chip idle: many of them keep it
// busy, and slots beyond a row's edges cost a wavefront per few rows (500,000 rows of
// 2 edges, 2 heads: 49 us with eight slots each, now 16 with one, as one thread per
// row and head took before; 5,000 rows among longer ones: 1.8 us the other way).
constexpr int64_t kChipLanes = 8192 * kWave;  // 256 CUs x 4 SIMDs x 8 wavefronts
template <int K>
inline int64_t row_groups(const Graph& g, int hp, RowGroups& L) {
  int64_t total = 0;
  auto add = [&](int i, const WorkItem* items, int n, int edges, int64_t most) {
    int lanes = hp;
    while (lanes < kWave && (lanes / hp * group_steps<K>() < edges ||
                             (lanes * K < 16 && lanes / hp < edges && 2 * (int64_t)n * lanes <= most)))
      lanes <<= 1;
    L.items[i] = items;
    L.n[i] = n;
    L.lanes[i] = lanes;
    L.waves[i] = (int)(((int64_t)n * lanes + kWave - 1) / kWave);
    total += L.waves[i];
  };
  add(0, g.heavy, g.n_heavy, g.chunk, INT64_MAX);
  add(1, g.long_rows, g.n_over64, g.chunk, INT64_MAX);
  add(2, g.long_rows + g.n_over64, g.n_over32 - g.n_over64, 64, INT64_MAX);
  add(3, g.long_rows + g.n_over32, g.n_long - g.n_over32, 32, INT64_MAX);
  add(4, g.short_rows, g.n_short, kShortRow, kChipLanes);
  return total;
}

// log2 of a power of two (a scalar instruction; divisions by lane counts go as shifts).
__device__ __forceinline__ int log2_of(int v) { return __builtin_ctz((unsigned)v); }

// The item of this lane's group (no edges past the list's end) and its lane count.
// Chunks of rows of at most `fewer` chunks count as no edges (0: none).
struct GroupItem {
  int kb, ke, pslot, lanes;
};
__device__ __forceinline__ GroupItem group_item(const RowGroups& L, int wid, int fewer = 0,
                                                const int* __restrict__ rowptr = nullptr,
                                                int chunk = 1) {
  // the list's first wavefront, then its fields by scalar selects (a dynamic index
  // into the arguments would be one more round trip)
  int before[kGroupLists];
  before[0] = 0;
#pragma unroll
  for (int i = 1; i < kGroupLists; ++i) before[i] = before[i - 1] + L.waves[i - 1];
  const WorkItem* items = L.items[0];
  int n = L.n[0], lanes = L.lanes[0], first = 0;
#pragma unroll
  for (int i = 1; i < kGroupLists; ++i) {
    const bool here = wid >= before[i];
    const WorkItem* p = L.items[i];
    const int ni = L.n[i], li = L.lanes[i];
    items = here ? p : items;
    n = here ? ni : n;
    lanes = here ? li : lanes;
    first = here ? before[i] : first;
  }
  wid -= first;
  GroupItem r;
  r.lanes = lanes;
  const int lg = log2_of(lanes);
  const int i = (wid << (log2_of(kWave) - lg)) + (lane_id() >> lg);
  const bool have = i < n;
  const WorkItem it = items[have ? i : 0];
  r.kb = it.kbeg;
  r.ke = have ? it.kend : it.kbeg;
  r.pslot = have ? it.slot : -1;
  if (fewer > 0 && r.pslot >= 0 && rowptr[it.row + 1] - rowptr[it.row] <= fewer * chunk) {
    r.ke = r.kb;
    r.pslot = -1;
  }
  return r;
}

// Long rows: a second launch, one wavefront per chunk, combines the chunks'
// statistics itself; rows of more than kGiantChunks chunks (whose wavefronts would
// read more statistics than scores) go one block of kGiantWaves wavefronts each,
// in a launch made where the graph has that many chunks.
constexpr int kGiantChunks = 2048;
constexpr int kGiantWaves = 16;

// The row of a chunk: its number of chunks and the slot of its first.
struct ChunkRow {
  int nch, slot0;
};
__device__ __forceinline__ ChunkRow chunk_row(const WorkItem& it, const int* __restrict__ rowptr,
                                              int chunk) {
  const int rb = uniform(rowptr[it.row]), re = uniform(rowptr[it.row + 1]);
  return {(re - rb + chunk - 1) / chunk, it.slot - (it.kbeg - rb) / chunk};
}

// Where the per-edge values of graph position k live: at the caller's edge id
// perm[k], or (perm NULL: arrays kept in the graph order) at k itself.
__device__ __forceinline__ int edge_at(const int* __restrict__ perm, int k) {
  return perm != nullptr ? perm[k] : k;
}

// Edge ids of NST steps of [kb, ke) (-1 past ke).
template <int NST>
__device__ __forceinline__ void load_ids(const int* __restrict__ perm, int kb, int ke, int slot,
                                         int SL, int (&e)[NST]) {
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const int k = kb + slot + u * SL;
    e[u] = k < ke ? edge_at(perm, k) : -1;
  }
}

// Sum over the slots of a head (lanes l, l ^ HP, l ^ 2 HP, ... of a group of
// `lanes`). IEEE addition commutes, so every lane of a head ends with the same sum.
__device__ __forceinline__ double slots_sum(double d, int HP, int lanes) {
  for (int off = HP; off < lanes; off <<= 1) d += __shfl_xor(d, off);
  return d;
}

}  // namespace tfg
