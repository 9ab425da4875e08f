// The fused attention kernel (gfx950, wave64): for every target row the score
// map, the per-head segment softmax and the weighted per-head sum of Fig. 5(a)
// in one sweep over the row's edges, with nothing per edge written to memory.
//
// Work items in edge slots as in slots.h: a slot of LPS lanes takes an item (or
// `split` neighbouring slots share one), a lane holds V columns, all of one
// head. A head's D columns sit on G lanes (the last ones step back to end at the
// head's last column, repeating some of their neighbour's), and those need one
// score per edge between them: groups of GX = 1, 2 or 4 of these lanes share the work, lane
// g taking the edges g, g + GX, ... of a round, so each score's exponential is
// computed once per group and reaches the others through a DPP quad move that
// folds into the multiply-add. (The earlier kernel kept a running maximum on
// every lane, with an exponential, a rescaling and a double accumulation per
// edge and lane.) A round's maximum is found first, then the sums so far are
// rescaled once per round.
//
// An item's result is the triple (maximum m, denominator d in double,
// numerators); whole rows write out = acc / d, chunks of long rows and the (row,
// source part) segments of the part plan write their triples, which gat_merge
// combines. By source part the gathered rows stay near the L2s. 114.6M edges of a
// power-law graph, 8 heads of 8: 4.17 + 0.26 (merge) -> 2.81 + 0.24 ms; the row
// sums alone take 1.92, the rest is this kernel's arithmetic at five wavefronts a
// SIMD (84 to 94 registers with V = 4; held to 80 or 72 it spills, 2.95 and 3.83 ms; eight
// rows in flight, 104 registers, 3.00). 23M edges, 8 heads of 16, dot product:
// 3.07 -> 2.31. 1.2M edges, 8 heads of 16, rows of 7 on
// average: 100 + 84 (a kernel for the short rows) + 35 -> 125 + 10 us.
#pragma once

#include "gat_shape.h"
#include "slots.h"
#include "softmax_stats.h"

namespace tfg {
namespace rows {

// The two score maps. Additive (GAT): s = LeakyReLU(a_s[src, k] + a_d[t, k])
// from the node projections. Scaled dot product (the Transformer-style GAT,
// Sec. 4.2): s = scale * <q[t, k], key[src, k]> over the D columns of head k;
// a lane holds V of them, and the partial products are summed over the G =
// D / V lanes of the head (every lane of the head gets the score).
struct Scores {
  const float* as;  // additive: [N, H]
  const float* ad;
  float slope;
  const float* q;  // dot product: [N, H*D]
  const float* key;
  float scale;
};

struct GatOut {
  float* out;
  float* rm;   // row maxima and denominators [N, H] (NULL: not wanted)
  double* rd;
  float* pacc;  // partial triples, by slot
  float* pm;
  double* pd;
};

// One launch over the lists (waves[] filled); the dot product in gat_dot.hip.
void gat_additive(const GatShape& t, bool narrow, const SlotLists& L, int waves, const int* col,
                  int H, int D, const Scores& S, const float* h, const GatOut& O, hipStream_t s);
void gat_dot(const GatShape& t, bool narrow, const SlotLists& L, int waves, const int* col, int H,
             int D, const Scores& S, const float* h, const GatOut& O, hipStream_t s);

namespace {

__device__ __forceinline__ float leaky(float z, float slope) { return z >= 0.0f ? z : slope * z; }

constexpr float kNegInf = -__builtin_huge_valf();

// v from lane I of this lane's group of GX (GX lanes aligned within a quad).
template <int I, int GX>
__device__ __forceinline__ float group_bcast(float v) {
  if constexpr (GX == 1) return v;
  constexpr int i = I % GX;
  constexpr int ctrl = GX == 4 ? i * 0x55 : (i | i << 2 | (2 + i) << 4 | (2 + i) << 6);
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, false));
}

// Maximum over the GX lanes of a group.
template <int GX>
__device__ __forceinline__ float group_max(float v) {
  if constexpr (GX >= 2) { const float o = dpp<0xB1>(v); v = o > v ? o : v; }  // quad lanes ^ 1
  if constexpr (GX >= 4) { const float o = dpp<0x4E>(v); v = o > v ? o : v; }  // quad lanes ^ 2
  return v;
}

// Merges the triple (m2, d2, a2) into (m, d, a); an empty triple has m = -inf.
template <int V>
__device__ __forceinline__ void triple_merge(float& m, double& d, float (&a)[V], float m2,
                                             double d2, const float (&a2)[V]) {
#pragma clang fp contract(off)
  const float mn = m2 > m ? m2 : m;
  // (equal maxima, two empty triples among them, weigh 1)
  const float x = m == mn ? 1.0f : expf(m - mn), y = m2 == mn ? 1.0f : expf(m2 - mn);
  d = d * (double)x + d2 * (double)y;
#pragma unroll
  for (int v = 0; v < V; ++v) a[v] = a[v] * x + a2[v] * y;
  m = mn;
}

template <int V, int LPS, int GX, bool DOT, bool NARROW>
__global__ __launch_bounds__(kItemBlock) void gat_slots(SlotLists L, const int* __restrict__ col,
                                                        int H, int D, int G, Scores S,
                                                        const float* __restrict__ h, GatOut O) {
  constexpr int SLOTS = kWave / LPS;
  constexpr int NR = id_regs<LPS>();
  constexpr int BW = kIds / NR;
  constexpr int U = 4;  // rows in flight per slot
  constexpr int OWN = (DOT ? U : kIds) / GX;  // scores per lane and round (dot product: group)
  const SlotItem it = slot_item<LPS>(L);
  const int kbeg = it.kbeg, n = it.n, nmax = it.nmax, split = it.split, sub = it.sub;
  const int lane = lane_id(), sl = lane % LPS;
  const int F = H * D;
  const int64_t row_bytes = (int64_t)F * (int64_t)sizeof(float);
  const int gi = lane % GX;
  const char* hb = reinterpret_cast<const char*>(h);
  const char* kb = reinterpret_cast<const char*>(S.key);

  for (int p0 = 0; p0 < H * G; p0 += LPS) {
    const int pl = p0 + sl;  // lane of the row: lane g of head `head`
    const bool fok = pl < H * G;
    // (lanes past the row repeat the last head's and write nothing)
    const int head = min(pl / G, H - 1), g = fok ? pl - head * G : 0;
    const int f = head * D + min(g * V, D - V);
    const unsigned lane_off = (unsigned)f * (unsigned)sizeof(float);
    float qv[V], adt = 0.0f;
    if constexpr (DOT) {
#pragma unroll
      for (int v = 0; v < V; ++v) qv[v] = 0.0f;
      if (n > 0) load_row<V>(S.q + (int64_t)it.row * F + f, qv);
    } else {
      adt = n > 0 ? S.ad[(int64_t)it.row * H + head] : 0.0f;
    }
    float m = kNegInf;
    double den = 0.0;  // this lane's share of the scores
    float tot[V];  // (sums in the order of slots.h, the rounds in one chain)
#pragma unroll
    for (int v = 0; v < V; ++v) tot[v] = 0.0f;

    // Brings the sums to the maximum of m and the scores sc, and replaces the
    // scores by their exponentials. (The additive score's comes before a round's
    // first sums: its chains are still zero.)
    auto weigh = [&](float (&sc)[OWN], float (&half)[2][V]) {
      float top = sc[0];
#pragma unroll
      for (int k = 1; k < OWN; ++k) top = sc[k] > top ? sc[k] : top;
      top = group_max<GX>(top);
      const float mn = top > m ? top : m;
      const float base = mn == kNegInf ? 0.0f : mn;  // no edge yet
      if (__any(mn > m)) {
        const float x = m == mn ? 1.0f : expf(m - base);
        den *= (double)x;
#pragma unroll
        for (int v = 0; v < V; ++v) {
          tot[v] *= x;
          if constexpr (DOT) {
            half[0][v] *= x;
            half[1][v] *= x;
          }
        }
        m = mn;
      }
#pragma unroll
      for (int k = 0; k < OWN; ++k) {
        sc[k] = expf(sc[k] - base);
        den += (double)sc[k];
      }
    };

    for (int r0 = 0; r0 < nmax; r0 += kIds * split) {
      const int j0 = r0 + sub;
      int id[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int j = min(j0 + (r * BW + sl % BW) * split, n - 1);
        id[r] = n > 0 ? col[kbeg + j] : 0;
        if constexpr (NARROW) id[r] = id[r] * (int)row_bytes;
      }
      float p[OWN];
      if constexpr (!DOT) {
        // this lane's edges of the round
        int own[OWN];
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
          const int j = min(j0 + (k * GX + gi) * split, n - 1);
          own[k] = n > 0 ? col[kbeg + j] : 0;
        }
#pragma unroll
        for (int k = 0; k < OWN; ++k) {
          const bool in = j0 + (k * GX + gi) * split < n;
          // (NARROW: the projections' byte offsets fit 32 bits as well, H <= F)
          float z;
          if constexpr (NARROW)
            z = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(S.as) +
                                                4u * ((unsigned)own[k] * (unsigned)H + (unsigned)head));
          else
            z = S.as[(int64_t)own[k] * H + head];
          p[k] = in ? leaky(z + adt, S.slope) : kNegInf;
        }
      }
      float half[2][V];
#pragma unroll
      for (int v = 0; v < V; ++v) half[0][v] = half[1][v] = 0.0f;
      each<kIds / U>([&](auto g_) {
        constexpr int GR = decltype(g_)::value;
        if (r0 + GR * U * split < nmax) {  // uniform
          float xv[U][V];
          if constexpr (DOT) {
            float kv[U][V];
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              load_row<V>(row_at<NARROW, float>(kb, slot_bcast<I, LPS>(id), row_bytes, lane_off),
                          kv[u]);
            });
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              load_row<V>(row_at<NARROW, float>(hb, slot_bcast<I, LPS>(id), row_bytes, lane_off),
                          xv[u]);
            });
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              float part[1] = {0.0f};
#pragma unroll
              for (int v = 0; v < V; ++v) part[0] = __builtin_fmaf(qv[v], kv[u][v], part[0]);
              lanes_sum(part, G);
              float t = S.scale * part[0];
              t = j0 + I * split < n ? t : kNegInf;
              // lane g of the group keeps edge g
              if (u % GX == 0) p[u / GX] = t;
              else p[u / GX] = gi == u % GX ? t : p[u / GX];
            });
            weigh(p, half);
          } else {
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              load_row<V>(row_at<NARROW, float>(hb, slot_bcast<I, LPS>(id), row_bytes, lane_off),
                          xv[u]);
            });
            if constexpr (GR == 0) weigh(p, half);
          }
          float four[V];
          auto& c = [&]() -> float(&)[V] {
            if constexpr (GR % 2 == 0) return half[GR / 2];
            else return four;
          }();
          if constexpr (GR % 2 == 1)
#pragma unroll
            for (int v = 0; v < V; ++v) four[v] = 0.0f;
          each<U>([&](auto u_) {
            constexpr int u = decltype(u_)::value, I = GR * U + u;
            const float w = group_bcast<u, GX>(p[(DOT ? u : I) / GX]);
            if (j0 + I * split < n)
#pragma unroll
              for (int v = 0; v < V; ++v) c[v] = __builtin_fmaf(w, xv[u][v], c[v]);
          });
          if constexpr (GR % 2 == 1)
#pragma unroll
            for (int v = 0; v < V; ++v) half[GR / 2][v] += four[v];
        }
      });
#pragma unroll
      for (int v = 0; v < V; ++v) tot[v] += half[0][v] + half[1][v];
    }
#pragma unroll
    for (int o = 1; o < GX; o <<= 1) den += __shfl_xor(den, o);
    // the slots of one item, pairwise
#pragma unroll
    for (int i = 1; i < SLOTS; i <<= 1)
      if (split > i) {  // uniform
        float a2[V];
#pragma unroll
        for (int v = 0; v < V; ++v) a2[v] = __shfl_xor(tot[v], LPS * i);
        const float m2 = __shfl_xor(m, LPS * i);
        const double d2 = __shfl_xor(den, LPS * i);
        triple_merge<V>(m, den, tot, m2, d2, a2);
      }
    if (!it.have || !fok || sub != 0) continue;
    if (it.slot < 0) {
      float o[V];
#pragma unroll
      for (int v = 0; v < V; ++v) o[v] = n > 0 ? (float)((double)tot[v] / den) : 0.0f;
      store_row<V>(O.out + (int64_t)it.row * F + f, o);
      if (O.rm != nullptr && g == 0) {
        O.rm[(int64_t)it.row * H + head] = m;
        O.rd[(int64_t)it.row * H + head] = den;
      }
    } else {
      store_row<V>(O.pacc + (int64_t)it.slot * F + f, tot);
      if (g == 0) {
        O.pm[(int64_t)it.slot * H + head] = m;
        O.pd[(int64_t)it.slot * H + head] = den;
      }
    }
  }
}

template <int V, int GX, bool DOT>
void gat_by_lps(int lps, bool narrow, const SlotLists& L, int waves, const int* col, int H, int D,
                int G, const Scores& S, const float* h, const GatOut& O, hipStream_t s) {
#define TFG_GAT(LL)                                                                              \
  do {                                                                                           \
    if (narrow)                                                                                  \
      gat_slots<V, LL, GX, DOT, true><<<(unsigned)waves, kItemBlock, 0, s>>>(L, col, H, D, G, S, h, O); \
    else                                                                                         \
      gat_slots<V, LL, GX, DOT, false><<<(unsigned)waves, kItemBlock, 0, s>>>(L, col, H, D, G, S, h, O); \
  } while (0)
  switch (lps) {
    case 4: TFG_GAT(4); break;
    case 8: TFG_GAT(8); break;
    case 16: TFG_GAT(16); break;
    case 32: TFG_GAT(32); break;
    default: TFG_GAT(64); break;
  }
#undef TFG_GAT
}

template <bool DOT>
void gat_dispatch(const GatShape& t, bool narrow, const SlotLists& L, int waves, const int* col,
                  int H, int D, const Scores& S, const float* h, const GatOut& O, hipStream_t s) {
#define TFG_BY(V, GX) gat_by_lps<V, GX, DOT>(t.lps, narrow, L, waves, col, H, D, t.G, S, h, O, s)
  if (t.vec == 4 && t.G % 4 == 0) TFG_BY(4, 4);
  else if (t.vec == 4 && t.G % 2 == 0) TFG_BY(4, 2);
  else if (t.vec == 4) TFG_BY(4, 1);
  else if (t.vec == 2) TFG_BY(2, 1);
  else TFG_BY(1, 1);
#undef TFG_BY
}

}  // namespace
}  // namespace rows
}  // namespace tfg
