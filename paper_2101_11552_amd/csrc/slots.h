// The slot aggregation (gfx950, wave64): several work items per wavefront.
//
// A wavefront has 64 / LPS edge slots of LPS lanes; a lane holds V neighbouring
// columns of a row. An item belongs to `split` neighbouring slots, usually one
// or two, so a wavefront works on several items at once and an item's edges are
// mostly summed inside a slot. One wavefront per item (the earlier kernel) spent
// a round trip on the item, one on its ids, one on its gathers and a tree over
// the slots on each of them, with most lanes idle on rows of a few edges; rows
// of 14 edges (169,343 of them, 40 columns) took 149 us, now 91. What bounds the
// large cases now is the gathers that miss the L2s: 10M edges of 400 bytes move
// at 6.6 TB/s (0.61 ms, before 0.83), 23M of 256 bytes by source part at 12
// TB/s (0.50 ms, before 0.70); the same with maxima 0.55 ms (before 1.97: the
// comparison with its tie rule was the bound, and is now three operations per
// column, since ids ascend along an item of one source part).
//
// The 16 ids of a round reach the lanes of a slot through DPP broadcasts that
// fold into the address addition and the multiply-add: per edge and slot one
// addition, one load and V multiply-adds. Rows need dword alignment only, and
// a last lane that steps back serves any width with 16-byte loads.
#pragma once

#include <utility>

#include "spmm.h"

namespace tfg {
namespace rows {
namespace {

// Rounds of kIds edges per slot. A slot of at least 16 lanes is made of whole
// DPP rows: lane l of each row holds edge l of the round, and edge I reaches
// every lane with one row broadcast. A slot of 4 or 8 lanes is made of quads:
// register r of lane l holds edge 4 r + l % 4, broadcast inside the quad.
constexpr int kIds = 16;
template <int LPS>
constexpr int id_regs() { return LPS >= 16 ? 1 : 4; }

template <int I, int LPS>
__device__ __forceinline__ int slot_bcast(const int (&r)[id_regs<LPS>()]) {
  if constexpr (LPS >= 16)
    return __builtin_amdgcn_update_dpp(0, r[0], 0x150 + I, 0xF, 0xF, false);
  else
    return __builtin_amdgcn_update_dpp(0, r[I / 4], (I % 4) * 0x55, 0xF, 0xF, false);
}

// v moved between lanes of a row of 16 by a DPP pattern.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Each t[u] summed over the aligned groups of G lanes (a power of two); every lane
// gets the sum.
template <int U>
__device__ __forceinline__ void lanes_sum(float (&t)[U], int G) {
  for (int o = G / 2; o >= 16; o >>= 1)
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] += __shfl_xor(t[u], o);
  if (G >= 16)
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] += dpp<0x140>(t[u]);  // row_mirror: the other half row
  if (G >= 8)
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] += dpp<0x141>(t[u]);  // row_half_mirror: the other quad
  if (G >= 4)
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] += dpp<0x4E>(t[u]);  // quad lanes ^ 2
  if (G >= 2)
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] += dpp<0xB1>(t[u]);  // quad lanes ^ 1
}

// A lane's place in the row whose id (NARROW: whose byte offset) is c.
template <bool NARROW, typename T>
__device__ __forceinline__ const T* row_at(const char* base, int c, int64_t row_bytes,
                                           unsigned lane_off) {
  if constexpr (NARROW) return reinterpret_cast<const T*>(base + ((unsigned)c + lane_off));
  else return reinterpret_cast<const T*>(base + ((int64_t)c * row_bytes + lane_off));
}

template <typename F, int... I>
__device__ __forceinline__ void each_of(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F&& f) {
  each_of(f, std::make_integer_sequence<int, N>{});
}

// The item of this lane's slot: place `sub` of the `split` slots that share it, n
// edges from kbeg (0 past the list's end: !have), and the most edges of an item of the
// wavefront. The list is chosen by scalar selects among arguments loaded together (a
// dynamic index into them would be a round trip more, a division per lane another
// twenty instructions: with rows of one or two edges that is a tenth of the time).
struct SlotItem {
  int row, kbeg, n, slot, split, sub, nmax;
  bool have;
};
template <int LPS>
__device__ __forceinline__ SlotItem slot_item(const SlotLists& L) {
  constexpr int SLOTS = kWave / LPS;
  const int wave = blockIdx.x;
  const WorkItem* items = L.items[0];
  int n_items = L.n[0], split = L.split[0], first = 0, before = 0;
#pragma unroll
  for (int i = 1; i < kSlotLists; ++i) {
    before += L.waves[i - 1];
    const bool here = wave >= before;
    const WorkItem* p = L.items[i];
    const int ni = L.n[i], si = L.split[i];
    items = here ? p : items;
    n_items = here ? ni : n_items;
    split = here ? si : split;
    first = here ? before : first;
  }
  const int q = (wave - first) * SLOTS + lane_id() / LPS;
  const int i = q >> __builtin_ctz((unsigned)split);  // a power of two
  SlotItem r;
  r.split = split;
  r.sub = q & (split - 1);
  r.have = i < n_items;
  const WorkItem w = items[r.have ? i : 0];
  r.row = w.row;
  r.kbeg = w.kbeg;
  r.slot = w.slot;
  r.n = r.have ? w.kend - w.kbeg : 0;
  r.nmax = __builtin_amdgcn_readlane(r.n, 0);
#pragma unroll
  for (int s = 1; s < SLOTS; ++s) r.nmax = max(r.nmax, __builtin_amdgcn_readlane(r.n, s * LPS));
  return r;
}

// kMax: edge ids ascend along an item (one source part per item); kMaxTies:
// they need not, equal maxima compare the ids.
enum { kSum = 0, kMax = 1, kMaxTies = 2, kMasked = 3 };
enum { kNone = 0, kEdge = 1, kHeads = 2 };  // weights: none, one per edge, one per edge and head

template <int V, int LPS, int KIND, int WM, bool NARROW>
__global__ __launch_bounds__(kItemBlock) void spmm_slots(
    SlotLists L, const int* __restrict__ col, const int* __restrict__ perm,
    const float* __restrict__ w, int w_by_perm, int H, int per_head, const float* __restrict__ x,
    int64_t ldx, const int* __restrict__ mask, int F, int mean, float* __restrict__ out,
    int* __restrict__ argout, float* __restrict__ part, int* __restrict__ part_arg, Epilogue ep) {
  constexpr int SLOTS = kWave / LPS;
  constexpr int FC = LPS * V;
  constexpr int NR = id_regs<LPS>();
  constexpr int BW = kIds / NR;  // edges per register
  constexpr bool MAX = KIND == kMax || KIND == kMaxTies, MASK = KIND == kMasked;
  constexpr int U = MASK || WM == kHeads ? 4 : 8;  // gathers in flight per slot
  const SlotItem it = slot_item<LPS>(L);
  const int kbeg = it.kbeg, n = it.n, nmax = it.nmax, split = it.split, sub = it.sub;
  const int sl = lane_id() % LPS;
  const int64_t row_bytes = ldx * (int64_t)sizeof(float);
  const bool need_perm = MAX || MASK || w_by_perm;

  for (int f0 = 0; f0 < F; f0 += FC) {
    // columns f .. f + V - 1. The last lane with columns of its own steps back
    // so that its V columns end at F (it repeats some of its neighbour's: the
    // same values, written twice); lanes past it repeat it and write nothing.
    const int fw = f0 + sl * V;
    const bool fok = fw < F;
    const int f = min(fw, F - V);
    const char* xb = reinterpret_cast<const char*>(x);
    const char* mb = reinterpret_cast<const char*>(mask);  // rows like those of x
    const unsigned lane_off = (unsigned)f * (unsigned)sizeof(float);
    const int head = WM == kHeads ? f / per_head : 0;
    const char* wb = reinterpret_cast<const char*>(w);
    const unsigned head_off = 4u * (unsigned)head;
    // Sums: chains of four edges, added up in pairs to the sum of a round, the
    // rounds in turn in two chains. (Four chains that ran through the whole item
    // were further from the sums in 64 bits: 1.17e-7 against 1.07e-7 over three
    // layers of rows of 5, 6.9e-8 against 6.6e-8 in a max gradient of 100-edge rows.)
    float tot[V], odd[V];  // (maxima: tot alone)
    int arg[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      tot[v] = odd[v] = 0.0f;
      arg[v] = -1;
    }

    // rounds of kIds edges per slot: place I of a round is edge j0 + I * split,
    // the `split` slots of an item taking neighbouring edges
    for (int r0 = 0; r0 < nmax; r0 += kIds * split) {
      const int j0 = r0 + sub;
      // ids (as byte offsets when NARROW), edge ids and weights of the round;
      // places past the item's end repeat its last edge
      int id[NR], pe[NR], wt[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        id[r] = pe[r] = wt[r] = 0;
        // (maxima repeat an item's last edge there)
        if (!MAX && r > 0 && r0 + r * BW * split >= nmax) continue;  // uniform: past every item
        const int j = min(j0 + (r * BW + sl % BW) * split, n - 1);
        id[r] = n > 0 ? col[kbeg + j] : 0;
        pe[r] = (need_perm && n > 0) ? perm[kbeg + j] : 0;
        if constexpr (WM == kEdge)
          wt[r] = __float_as_int(
              n > 0 ? w[w_by_perm ? pe[r] : kbeg + j] : 0.0f);
        if constexpr (WM == kHeads) wt[r] = n > 0 ? (w_by_perm ? pe[r] : kbeg + j) : 0;
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        if constexpr (NARROW) id[r] = id[r] * (int)row_bytes;
        // the edge's row of weights as its byte offset, up to 2^32: an unsigned
        // product, kept in a signed register for the DPP moves
        if constexpr (WM == kHeads && NARROW)
          wt[r] = (int)((unsigned)wt[r] * 4u * (unsigned)H);
      }
      float half[2][V];  // the sums of the round's first and last eight places
#pragma unroll
      for (int v = 0; v < V; ++v) half[0][v] = half[1][v] = 0.0f;
      each<kIds / U>([&](auto g_) {
        constexpr int G = decltype(g_)::value;
        if (r0 + G * U * split < nmax) {  // uniform
          float xv[U][V], wh[U];
          int mv[MASK ? U : 1][V];
          each<U>([&](auto u_) {
            constexpr int u = decltype(u_)::value, I = G * U + u;
            if constexpr (WM == kHeads && NARROW) {
              wh[u] = *reinterpret_cast<const float*>(wb + ((unsigned)slot_bcast<I, LPS>(wt) + head_off));
            } else if constexpr (WM == kHeads) {
              wh[u] = w[(int64_t)slot_bcast<I, LPS>(wt) * H + head];
            }
            const int c = slot_bcast<I, LPS>(id);
            if constexpr (MASK) {
              load_irow<V>(row_at<NARROW, int>(mb, c, row_bytes, lane_off), mv[u]);
            } else {
              load_row<V>(row_at<NARROW, float>(xb, c, row_bytes, lane_off), xv[u]);
            }
          });
          if constexpr (MASK) {
            // a row of x is read only where this edge won one of its columns
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = G * U + u;
              const int c = slot_bcast<I, LPS>(id), e = slot_bcast<I, LPS>(pe);
              bool any = false;
#pragma unroll
              for (int v = 0; v < V; ++v) any |= mv[u][v] == e;
              if (any & (j0 + I * split < n)) {
                load_row<V>(row_at<NARROW, float>(xb, c, row_bytes, lane_off), xv[u]);
#pragma unroll
                for (int v = 0; v < V; ++v) xv[u][v] = mv[u][v] == e ? xv[u][v] : 0.0f;
              } else {
#pragma unroll
                for (int v = 0; v < V; ++v) xv[u][v] = 0.0f;
              }
            });
          }
          float four[V];  // a second chain: every other four places
#pragma unroll
          for (int v = 0; v < V; ++v) four[v] = 0.0f;
          each<U>([&](auto u_) {
            constexpr int u = decltype(u_)::value, I = G * U + u;
            float we = 1.0f;
            if constexpr (WM == kHeads) we = wh[u];
            if constexpr (WM == kEdge) we = __int_as_float(slot_bcast<I, LPS>(wt));
            if constexpr (MAX) {
              // repeated last edges never win: strict comparison
              const int e = slot_bcast<I, LPS>(pe);
#pragma unroll
              for (int v = 0; v < V; ++v) {
                const float m = WM == kNone ? xv[u][v] : we * xv[u][v];
                bool take = m > tot[v];
                if (KIND == kMaxTies) take |= (m == tot[v]) & (e < arg[v]);
                if (I == 0) take |= r0 == 0;  // a slot's first edge always
                tot[v] = take ? m : tot[v];
                arg[v] = take ? e : arg[v];
              }
            } else {
              auto& c = [&]() -> float(&)[V] {
                if constexpr (I / 4 % 2 == 0) return half[I / 8];
                else return four;
              }();
              if (j0 + I * split < n)
#pragma unroll
                for (int v = 0; v < V; ++v)
                  c[v] = WM == kNone ? c[v] + xv[u][v] : __builtin_fmaf(we, xv[u][v], c[v]);
            }
          });
          if constexpr (!MAX && (U == 8 || G % 2 == 1))
#pragma unroll
            for (int v = 0; v < V; ++v) half[G * U / 8][v] += four[v];
        }
      });
      if constexpr (!MAX)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float t = odd[v] + (half[0][v] + half[1][v]);
          odd[v] = tot[v];
          tot[v] = t;
        }
    }
    if constexpr (!MAX)
#pragma unroll
      for (int v = 0; v < V; ++v) tot[v] += odd[v];
    // the slots of one item, pairwise
#pragma unroll
    for (int i = 1; i < SLOTS; i <<= 1)
      if (split > i) {  // uniform
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float ov = __shfl_xor(tot[v], LPS * i);
          if constexpr (MAX) {
            const int oa = __shfl_xor(arg[v], LPS * i);
            max_combine(tot[v], arg[v], ov, oa);
          } else {
            tot[v] += ov;
          }
        }
      }
    if (!it.have || !fok || sub != 0) continue;
    if (it.slot < 0) {
      if constexpr (MAX) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          tot[v] = n == 0 ? 0.0f : tot[v];
          arg[v] = n == 0 ? -1 : arg[v];
        }
      } else {
        if (mean && n > 0) {
          const float cnt = (float)n;
#pragma unroll
          for (int v = 0; v < V; ++v) tot[v] = tot[v] / cnt;
        }
        apply_epilogue<V>(ep, it.row, f, tot);
      }
      store_row<V>(out + (int64_t)it.row * F + f, tot);
      if (MAX && argout != nullptr) store_irow<V>(argout + (int64_t)it.row * F + f, arg);
    } else {
      store_row<V>(part + (int64_t)it.slot * F + f, tot);
      if (MAX) store_irow<V>(part_arg + (int64_t)it.slot * F + f, arg);
    }
  }
}

template <int V, int LPS, int KIND, int WM>
void run(bool narrow, const SlotLists& L, int waves, const RowArgs& a, hipStream_t s) {
#define TFG_SLOTS(N)                                                                      \
  spmm_slots<V, LPS, KIND, WM, N><<<(unsigned)waves, kItemBlock, 0, s>>>(                 \
      L, a.col, a.perm, a.w, a.w_by_perm, a.H, a.per_head, a.x, a.ldx, a.mask, a.F, a.mean, \
      a.out, a.argout, a.part, a.part_arg, a.ep)
  if (narrow) TFG_SLOTS(true);
  else TFG_SLOTS(false);
#undef TFG_SLOTS
}

template <int V, int KIND, int WM>
void by_lps(int lps, bool narrow, const SlotLists& L, int waves, const RowArgs& a, hipStream_t s) {
  switch (lps) {
    case 4: run<V, 4, KIND, WM>(narrow, L, waves, a, s); break;
    case 8: run<V, 8, KIND, WM>(narrow, L, waves, a, s); break;
    case 16: run<V, 16, KIND, WM>(narrow, L, waves, a, s); break;
    case 32: run<V, 32, KIND, WM>(narrow, L, waves, a, s); break;
    default: run<V, 64, KIND, WM>(narrow, L, waves, a, s); break;
  }
}

}  // namespace
}  // namespace rows
}  // namespace tfg
