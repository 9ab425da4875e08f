// Gradients of the aggregation and of the segment softmax (gfx950, wave64).
//
// For out = aggregate(w, x) and an incoming gradient dy = dL/d out:
//   dx  (sum)  = the sum aggregation of dy over the transposed graph (rows are
//                sources, columns targets) with the same edge weights;
//   dx  (mean) = the same with w_e / deg(t_e) as weights;
//   dx  (max)  = the masked gather (slots.h): element c of dy[t] reaches
//                source s only through the edge that won the forward max;
//   dw[e, k]   = sum over the columns c of head k of g[t_e, c] x[s_e, c] with
//                g = dy, dy / deg(t) or the masked dy: one dot product per
//                edge (edge_grad_slots), walking the forward graph so that the
//                dy row of a target is loaded once.
// Segment softmax: ds = alpha * (dalpha - sum over the segment of alpha * dalpha)
// per head, the sum accumulated in double (softmax_grad_items; long rows in
// chunks whose sums are added in chunk order).
// Every result has one writer and a fixed summation order: no atomics.
#include <cstdlib>

#include "slots.h"
#include "softmax_stats.h"

namespace tfg {

namespace {

using namespace rows;

enum { kGradSum = 0, kGradMean = 1, kGradMax = 2 };

// Per-edge dot products <g[t, k], x[s, k]> (dw, and the attention's scaled dot
// products): work items in edge slots as in slots.h, the dy row of an item's
// target in registers. Head k's D columns sit on G lanes, a power of two (the
// last ones step back to end at column D and leave out what their neighbour
// has; lanes past the columns add nothing); the partial products of a group of
// four edges are summed over the G lanes with DPP moves, and lane g of a head
// keeps edge g, so that four edges go out with one store. Columns beyond 64 lanes
// go in passes inside a group; heads beyond them in passes over the edges.
// One wavefront per item, each with its own tree over the lanes, took 137 us for
// 1.35M edges and 8 heads of 16 in two launches; now 112 in one, the gathers of
// 512-byte rows at 6 TB/s. 23M edges of 64 columns by source part: 0.68 -> 0.47
// ms. Rows wider than 256 columns had one thread per edge (2M edges of 300
// columns: 2.50 -> 0.32 ms).
template <int V, int LPS, int U, int MODE, bool NARROW>
__global__ __launch_bounds__(kItemBlock) void edge_grad_slots(
    SlotLists L, const int* __restrict__ rowptr, const int* __restrict__ col,
    const int* __restrict__ perm, const float* __restrict__ x, int64_t ldx,
    const float* __restrict__ dy, const int* __restrict__ arg, int H, int D, int G,
    float* __restrict__ dw, int dw_by_perm, float scale) {
  constexpr int NR = id_regs<LPS>();
  constexpr int BW = kIds / NR;
  constexpr int Q = 4;  // edges per reduction (U: gathers in flight per slot)
  const SlotItem it = slot_item<LPS>(L);
  const int kbeg = it.kbeg, n = it.n, nmax = it.nmax, split = it.split, sub = it.sub;
  const int sl = lane_id() % LPS;
  if (nmax == 0) return;
  const int F = H * D;
  const int64_t row_bytes = ldx * (int64_t)sizeof(float);
  const char* xb = reinterpret_cast<const char*>(x);
  const bool need_perm = MODE == kGradMax || dw_by_perm;
  const float cnt = MODE == kGradMean && n > 0 ? (float)(rowptr[it.row + 1] - rowptr[it.row]) : 1.0f;

  for (int p0 = 0; p0 < H * G; p0 += LPS) {
    const int pl = p0 + sl;
    const bool hok = pl < H * G;  // a lane of an existing head
    const int head = hok ? pl / G : 0, g = hok ? pl - head * G : 0;
    // the columns of pass c0: c0 + g V .., stepped back at the head's end
    auto columns = [&](int c0, int& f, int& skip, float (&gy)[V], int (&ga)[V]) {
      const int cw = c0 + g * V, c = min(cw, D - V);
      f = head * D + c;
      skip = cw - c;  // the first columns, its neighbour's
      if (n > 0) {
        load_row<V>(dy + (int64_t)it.row * F + f, gy);
        if constexpr (MODE == kGradMax) load_irow<V>(arg + (int64_t)it.row * F + f, ga);
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        gy[v] = n > 0 ? gy[v] : 0.0f;
        if constexpr (MODE == kGradMean) gy[v] = gy[v] / cnt;
      }
    };
    const int cstep = G * V;            // columns per pass
    const bool ragged = D % cstep != 0;  // some lanes skip columns
    int f, skip;
    float gy[V];
    int ga[V];
    columns(0, f, skip, gy, ga);
    for (int r0 = 0; r0 < nmax; r0 += kIds * split) {
      const int j0 = r0 + sub;
      int id[NR], pe[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        id[r] = pe[r] = 0;
        if (r > 0 && r0 + r * BW * split >= nmax) continue;  // uniform: past every item
        const int j = min(j0 + (r * BW + sl % BW) * split, n - 1);
        id[r] = n > 0 ? col[kbeg + j] : 0;
        pe[r] = (need_perm && n > 0) ? perm[kbeg + j] : 0;
      }
      if constexpr (NARROW)
#pragma unroll
        for (int r = 0; r < NR; ++r) id[r] = id[r] * (int)row_bytes;
      each<kIds / U>([&](auto g_) {
        constexpr int GR = decltype(g_)::value;
        if (r0 + GR * U * split < nmax) {  // uniform
          float t[U];
#pragma unroll
          for (int u = 0; u < U; ++u) t[u] = 0.0f;
          for (int c0 = 0; c0 < D; c0 += cstep) {
            if (cstep < D) columns(c0, f, skip, gy, ga);  // uniform: more than one pass
            const unsigned lane_off = (unsigned)f * (unsigned)sizeof(float);
            float xv[U][V];
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              load_row<V>(row_at<NARROW, float>(xb, slot_bcast<I, LPS>(id), row_bytes, lane_off),
                          xv[u]);
            });
            if (ragged) {  // uniform; zeros on both sides, whatever x holds there
#pragma unroll
              for (int v = 0; v < V; ++v) {
                gy[v] = v < skip ? 0.0f : gy[v];
#pragma unroll
                for (int u = 0; u < U; ++u) xv[u][v] = v < skip ? 0.0f : xv[u][v];
              }
            }
            each<U>([&](auto u_) {
              constexpr int u = decltype(u_)::value, I = GR * U + u;
              const int e = MODE == kGradMax ? slot_bcast<I, LPS>(pe) : 0;
#pragma unroll
              for (int v = 0; v < V; ++v) {
                // (both sides zero where the edge did not win: x may hold -inf there)
                const bool use = MODE == kGradMax ? ga[v] == e : true;
                const float w = use ? gy[v] : 0.0f, xs = use ? xv[u][v] : 0.0f;
                t[u] = __builtin_fmaf(w, xs, t[u]);
              }
            });
          }
          lanes_sum<U>(t, G);
          // lane g of a head keeps the edges g, g + min(G, Q), ... of each Q
          const int gl = min(G, Q);
          each<U / Q>([&](auto b_) {
            constexpr int b = decltype(b_)::value * Q;
            int pq[Q];
            if (dw_by_perm)  // uniform
              each<Q>([&](auto i_) {
                constexpr int i = decltype(i_)::value;
                pq[i] = slot_bcast<GR * U + b + i, LPS>(pe);
              });
            for (int o = 0; o < Q; o += gl) {  // uniform
              const int mine = o + (g & (gl - 1));
              const int j = j0 + (GR * U + b + mine) * split;
              float val = t[b];
              int e = dw_by_perm ? pq[0] : kbeg + j;
#pragma unroll
              for (int i = 1; i < Q; ++i) {
                val = mine == i ? t[b + i] : val;
                if (dw_by_perm) e = mine == i ? pq[i] : e;
              }
              if (hok && g < gl && j < n) dw[(int64_t)e * H + head] = val * scale;
            }
          });
        }
      });
    }
  }
}

// Weights of the transposed graph for the mean gradient, in its graph order:
// wt[k, h] = w[e, h] / deg(t_k) (w = 1 when NULL) with e = perm[k] for
// weights in edge order, e = k for weights already in the transposed order;
// t_k = col[k].
__global__ __launch_bounds__(kBlock) void mean_weights(const int* __restrict__ tcol,
                                                       const int* __restrict__ tperm, unsigned n,
                                                       unsigned H, const int* __restrict__ rowptr,
                                                       const float* __restrict__ w, int by_perm,
                                                       float* __restrict__ wt) {
  const unsigned i = blockIdx.x * kBlock + threadIdx.x;  // (position, head), below 2^31
  if (i >= n) return;
  const unsigned k = i / H, h = i - k * H;
  const int t = tcol[k];
  const float cnt = (float)(rowptr[t + 1] - rowptr[t]);
  const float wv = w ? w[(by_perm ? (int64_t)tperm[k] : (int64_t)k) * H + h] : 1.0f;
  wt[i] = wv / cnt;
}

// Graph order -> caller's edge order: out[perm[k], h] = in[k, h]; K values of
// one edge per thread (E * H / K threads, below 2^31).
template <int K>
__global__ __launch_bounds__(kBlock) void to_edge_order(const int* __restrict__ perm, unsigned n,
                                                        unsigned hk, const float* __restrict__ in,
                                                        float* __restrict__ out) {
  const unsigned i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const unsigned k = i / hk, h = i - k * hk;
  float v[K];
  load_row<K>(in + (int64_t)i * K, v);
  float* o = out + ((int64_t)perm[k] * hk + h) * K;
  if constexpr (K == 4) *reinterpret_cast<f4*>(o) = f4{v[0], v[1], v[2], v[3]};
  else *o = v[0];
}

// The same scatter for one value per edge on large graphs, in two passes
// through buckets of 2^kPermBits consecutive destinations (a random 4-byte
// store moves a whole line; these passes move whole lines):
//   perm_count   per tile of kPermTile positions, the count of each bucket
//                (one column of a bucket-major table);
//   (exclusive scan of the table: every (bucket, tile) its place)
//   perm_bucket  each position's (destination mod 2^kPermBits, value) pair
//                to its bucket's place for this tile, slots taken with LDS
//                atomics (the order inside a bucket does not matter);
//   perm_place   one block per bucket: the pairs into LDS at their offsets,
//                then the bucket's 2^kPermBits destinations written in order.
// perm is a permutation, so every destination of a bucket is written once.
constexpr int kPermBits = 15;                         // destinations per bucket (128 KB of LDS)
constexpr int kPermThreads = 1024;
constexpr int kPermItems = 64;                        // positions per thread and tile
constexpr int kPermTile = kPermThreads * kPermItems;  // 65536
constexpr int kPermMaxBuckets = 8192;                 // LDS counters (32 KB)
constexpr int kPermXcds = 8;

// tiles in XCD-contiguous order (blocks are dispatched round-robin over the
// XCDs), so that the bucket runs of neighbouring tiles meet in one L2
__device__ __forceinline__ int perm_tile_of(int bid, int ntiles) {
  const int q = ntiles / kPermXcds, r = ntiles % kPermXcds;
  const int x = bid % kPermXcds, i = bid / kPermXcds;
  return x * q + min(x, r) + i;
}

__global__ __launch_bounds__(kPermThreads) void perm_count(const int* __restrict__ perm, int64_t E,
                                                       int nbuckets, int ntiles,
                                                       int* __restrict__ table) {
  __shared__ int cnt[kPermMaxBuckets];
  for (int b = threadIdx.x; b < nbuckets; b += kPermThreads) cnt[b] = 0;
  __syncthreads();
  const int tile = perm_tile_of((int)blockIdx.x, ntiles);
  const int64_t base = (int64_t)tile * kPermTile;
  const int n = (int)min<int64_t>(kPermTile, E - base);
  for (int i0 = 0; i0 < kPermItems; i0 += 16) {
    int d[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int p = (i0 + i) * kPermThreads + (int)threadIdx.x;
      d[i] = p < n ? __builtin_nontemporal_load(perm + base + p) : -1;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (d[i] >= 0) atomicAdd(&cnt[d[i] >> kPermBits], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbuckets; b += kPermThreads)
    table[(int64_t)b * ntiles + tile] = cnt[b];
}

__global__ __launch_bounds__(kPermThreads) void perm_bucket(const int* __restrict__ perm,
                                                        const float* __restrict__ in, int64_t E,
                                                        int nbuckets, int ntiles,
                                                        const int* __restrict__ table,
                                                        int2* __restrict__ pairs) {
  __shared__ int cur[kPermMaxBuckets];
  const int tile = perm_tile_of((int)blockIdx.x, ntiles);
  for (int b = threadIdx.x; b < nbuckets; b += kPermThreads)
    cur[b] = table[(int64_t)b * ntiles + tile];
  __syncthreads();
  const int64_t base = (int64_t)tile * kPermTile;
  const int n = (int)min<int64_t>(kPermTile, E - base);
  for (int i0 = 0; i0 < kPermItems; i0 += 16) {
    int d[16];
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int p = (i0 + i) * kPermThreads + (int)threadIdx.x;
      d[i] = p < n ? __builtin_nontemporal_load(perm + base + p) : -1;
      v[i] = p < n ? __builtin_nontemporal_load(in + base + p) : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (d[i] >= 0) {
        const int slot = atomicAdd(&cur[d[i] >> kPermBits], 1);
        pairs[slot] = make_int2(d[i] & ((1 << kPermBits) - 1), __float_as_int(v[i]));
      }
  }
}

__global__ __launch_bounds__(kPermThreads) void perm_place(const int2* __restrict__ pairs,
                                                       const int* __restrict__ table, int ntiles,
                                                       int64_t E, int nbuckets,
                                                       float* __restrict__ out) {
  __shared__ float buf[1 << kPermBits];
  const int b = (int)blockIdx.x;
  const int64_t start = table[(int64_t)b * ntiles];
  const int64_t end = b + 1 < nbuckets ? table[(int64_t)(b + 1) * ntiles] : E;
  typedef int i2v __attribute__((ext_vector_type(2)));
  const i2v* pv = reinterpret_cast<const i2v*>(pairs);
  for (int64_t j0 = start; j0 < end; j0 += 8 * kPermThreads) {
    i2v pr[8];  // eight loads in flight per thread
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t j = j0 + u * kPermThreads + threadIdx.x;
      pr[u] = j < end ? __builtin_nontemporal_load(pv + j) : i2v{-1, 0};
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (pr[u].x >= 0) buf[pr[u].x] = __int_as_float(pr[u].y);
  }
  __syncthreads();
  const int64_t o = (int64_t)b << kPermBits;
  const int n = (int)min<int64_t>(int64_t(1) << kPermBits, E - o);
  for (int j = threadIdx.x; j < n; j += kPermThreads) __builtin_nontemporal_store(buf[j], out + o + j);
}

// Caller's edge order -> graph order: out[k, h] = in[perm[k], h].
template <int K>
__global__ __launch_bounds__(kBlock) void to_graph_order(const int* __restrict__ perm, unsigned n,
                                                         unsigned hk, const float* __restrict__ in,
                                                         float* __restrict__ out) {
  const unsigned i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const unsigned k = i / hk, h = i - k * hk;
  float v[K];
  load_row<K>(in + ((int64_t)perm[k] * hk + h) * K, v);
  float* o = out + (int64_t)i * K;
  if constexpr (K == 4) *reinterpret_cast<f4*>(o) = f4{v[0], v[1], v[2], v[3]};
  else *o = v[0];
}

// Launches one of the two over E edges of H values (E * H below 2^31).
template <bool TO_EDGE>
void launch_reorder(const int* perm, int64_t E, int H, const float* in, float* out, hipStream_t s) {
  const int K = H % 4 == 0 ? 4 : 1;
  const unsigned hk = (unsigned)(H / K), n = (unsigned)(E * hk);
  const unsigned nb = (unsigned)(((int64_t)n + kBlock - 1) / kBlock);
#define TFG_REORDER(KK)                                                        \
  do {                                                                         \
    if (TO_EDGE) to_edge_order<KK><<<nb, kBlock, 0, s>>>(perm, n, hk, in, out); \
    else to_graph_order<KK><<<nb, kBlock, 0, s>>>(perm, n, hk, in, out);        \
  } while (0)
  if (K == 4) TFG_REORDER(4);
  else TFG_REORDER(1);
#undef TFG_REORDER
}

// Softmax gradient ds = alpha * (dalpha - sum over the row of alpha *
// dalpha), per head, with the products summed in double (exact products of
// floats), in the layouts of the softmax (softmax_stats.h): lane groups with
// their values in registers, and the chunks of split rows in two launches, the
// first of which stores their sums (pdot).

// alpha and dalpha of the heads h for the registers' ids (0 where there is none)
template <int NST, int K>
__device__ __forceinline__ void grad_load(const float* __restrict__ alpha,
                                          const float* __restrict__ da, int H, int h, bool act,
                                          const int (&e)[NST], float (&a)[NST][K],
                                          float (&g)[NST][K]) {
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const bool ok = act && e[u] >= 0;
    if (ok) {
      load_k<K>(alpha + ((int64_t)e[u] * H + h) * K, a[u]);
      load_k<K>(da + ((int64_t)e[u] * H + h) * K, g[u]);
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
      a[u][i] = ok ? a[u][i] : 0.0f;
      g[u][i] = ok ? g[u][i] : 0.0f;
    }
  }
}

template <int NST, int K>
__device__ __forceinline__ double grad_dot(const float (&a)[NST][K], const float (&g)[NST][K],
                                           int i, int HP, int lanes) {
  double dot = 0.0;
#pragma unroll
  for (int u = 0; u < NST; ++u) dot += (double)a[u][i] * (double)g[u][i];
  return slots_sum(dot, HP, lanes);
}

template <int NST, int K>
__device__ __forceinline__ void grad_write(const float (&a)[NST][K], const float (&g)[NST][K],
                                           const int (&e)[NST], const double (&dot)[K], int H,
                                           int h, bool act, float* __restrict__ ds) {
#pragma unroll
  for (int u = 0; u < NST; ++u)
    if (act && e[u] >= 0) {
      float v[K];
#pragma unroll
      for (int i = 0; i < K; ++i) v[i] = (float)((double)a[u][i] * ((double)g[u][i] - dot[i]));
      store_k<K>(ds + ((int64_t)e[u] * H + h) * K, v);
    }
}

// A whole item's sum over [kb, ke) for head h, loading the values (the items
// longer than group_steps() slot steps), and its ds from a second sweep.
constexpr int kGradSweep = 4;  // values in flight
__device__ __forceinline__ double grad_sweep_dot(const int* __restrict__ perm,
                                                 const float* __restrict__ alpha,
                                                 const float* __restrict__ da, int H, int h,
                                                 bool act, int kb, int ke, int slot, int SL,
                                                 int HP) {
  double dot = 0.0;
  for (int k = kb + slot; k < ke; k += kGradSweep * SL) {
    int e[kGradSweep];
    float a[kGradSweep][1], g[kGradSweep][1];
    load_ids<kGradSweep>(perm, k, ke, 0, SL, e);
    grad_load<kGradSweep, 1>(alpha, da, H, h, act, e, a, g);
#pragma unroll
    for (int u = 0; u < kGradSweep; ++u) dot += (double)a[u][0] * (double)g[u][0];
  }
  return slots_sum(dot, HP, kWave);
}

__device__ __forceinline__ void grad_sweep_write(const int* __restrict__ perm,
                                                 const float* __restrict__ alpha,
                                                 const float* __restrict__ da, int H, int h,
                                                 bool act, int kb, int ke, int slot, int SL,
                                                 double dot, float* __restrict__ ds) {
  const double d[1] = {dot};
  for (int k = kb + slot; k < ke; k += kGradSweep * SL) {
    int e[kGradSweep];
    float a[kGradSweep][1], g[kGradSweep][1];
    load_ids<kGradSweep>(perm, k, ke, 0, SL, e);
    grad_load<kGradSweep, 1>(alpha, da, H, h, act, e, a, g);
    grad_write<kGradSweep, 1>(a, g, e, d, H, h, act, ds);
  }
}

template <int NST, int K>
__device__ __forceinline__ void grad_item_regs(const int* __restrict__ perm,
                                               const float* __restrict__ alpha,
                                               const float* __restrict__ da, int H, int HP,
                                               const GroupItem& it, float* __restrict__ ds,
                                               double* __restrict__ pdot) {
  const int SL = it.lanes >> log2_of(HP);
  const int slot = (lane_id() & (it.lanes - 1)) >> log2_of(HP), hh = lane_id() & (HP - 1);
  int e[NST];
  load_ids<NST>(perm, it.kb, it.ke, slot, SL, e);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    float a[NST][K], g[NST][K];
    double dot[K];
    grad_load<NST, K>(alpha, da, H, h, act, e, a, g);
#pragma unroll
    for (int i = 0; i < K; ++i) dot[i] = grad_dot<NST, K>(a, g, i, HP, it.lanes);
    if (it.pslot < 0) {
      grad_write<NST, K>(a, g, e, dot, H, h, act, ds);
    } else if (slot == 0 && act) {
#pragma unroll
      for (int i = 0; i < K; ++i) pdot[((int64_t)it.pslot * H + h) * K + i] = dot[i];
    }
  }
}

// 1.35M edges and 8 heads, rows of 8 on average: 62 us with one wavefront per row of
// over 8 edges and one head per lane, now 31.
template <int K>
__global__ __launch_bounds__(kItemBlock) void softmax_grad_items(
    RowGroups L, const int* __restrict__ rowptr, int chunk, int fewer,
    const int* __restrict__ perm, const float* __restrict__ alpha, const float* __restrict__ da,
    int H, int HP, float* __restrict__ ds, double* __restrict__ pdot) {
  const GroupItem it = group_item(L, blockIdx.x, fewer, rowptr, chunk);
  const int SL = it.lanes >> log2_of(HP), n = it.ke - it.kb;
  if (!__any(n > SL)) {
    grad_item_regs<1, K>(perm, alpha, da, H, HP, it, ds, pdot);
  } else if (!__any(n > 2 * SL)) {
    grad_item_regs<2, K>(perm, alpha, da, H, HP, it, ds, pdot);
  } else if (!__any(n > 4 * SL)) {
    grad_item_regs<4, K>(perm, alpha, da, H, HP, it, ds, pdot);
  } else if (K == 1 && !__any(n > 8 * SL)) {
    grad_item_regs<K == 1 ? 8 : 1, K>(perm, alpha, da, H, HP, it, ds, pdot);
  } else {  // groups of 64 lanes: one item; single heads
    const int H1 = H * K, hp = min(HP * K, kWave), sl1 = kWave >> log2_of(hp);
    const int slot = lane_id() >> log2_of(hp), hh = lane_id() & (hp - 1);
    for (int hb = 0; hb < H1; hb += hp) {
      const int h = hb + hh;
      const bool act = h < H1;
      const double dot = grad_sweep_dot(perm, alpha, da, H1, h, act, it.kb, it.ke, slot, sl1, hp);
      if (it.pslot < 0)
        grad_sweep_write(perm, alpha, da, H1, h, act, it.kb, it.ke, slot, sl1, dot, ds);
      else if (slot == 0 && act)
        pdot[(int64_t)it.pslot * H1 + h] = dot;
    }
  }
}

// A split row's sum for head h from its chunks' sums (p at the head), a share
// per slot, four in flight, then over the slots.
__device__ __forceinline__ double row_dot(const double* __restrict__ p, int nch, int H, bool act,
                                          int slot, int SL, int HP) {
  constexpr int U = 4;
  double dot = 0.0;
  if (act)
    for (int c = slot; c < nch; c += U * SL) {
      double q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = p[(int64_t)min(c + u * SL, nch - 1) * H];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u * SL < nch) dot += q[u];
    }
  return slots_sum(dot, HP, kWave);
}

// ds of the chunks of split rows, one wavefront per chunk (NST = 0: the values
// loaded one by one). One block of 16 wavefronts per split row: 30 us for 1,400
// chunks of 460 rows, now 8.
template <int NST, int K>
__device__ __forceinline__ void grad_chunk_write(const int* __restrict__ perm,
                                                 const float* __restrict__ alpha,
                                                 const float* __restrict__ da, int H, int HP,
                                                 const WorkItem& it, const ChunkRow& r,
                                                 const double* __restrict__ pdot,
                                                 float* __restrict__ ds) {
  const int SL = kWave >> log2_of(HP);
  const int slot = lane_id() >> log2_of(HP), hh = lane_id() & (HP - 1);
  constexpr int R = NST > 0 ? NST : 1;
  int e[R];
  if constexpr (NST > 0) load_ids<NST>(perm, it.kbeg, it.kend, slot, SL, e);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    float a[R][K], g[R][K];
    double dot[K];
    if constexpr (NST > 0) grad_load<NST, K>(alpha, da, H, h, act, e, a, g);
#pragma unroll
    for (int i = 0; i < K; ++i)
      dot[i] = row_dot(pdot + ((int64_t)r.slot0 * H + h) * K + i, r.nch, H * K, act, slot, SL, HP);
    if constexpr (NST > 0)
      grad_write<NST, K>(a, g, e, dot, H, h, act, ds);
    else
      grad_sweep_write(perm, alpha, da, H, h, act, it.kbeg, it.kend, slot, SL, dot[0], ds);
  }
}

template <int K>
__global__ __launch_bounds__(kItemBlock) void softmax_grad_chunks(
    const WorkItem* __restrict__ heavy, const int* __restrict__ rowptr, int chunk, int fewer,
    const int* __restrict__ perm, const float* __restrict__ alpha, const float* __restrict__ da,
    int H, int HP, const double* __restrict__ pdot, float* __restrict__ ds) {
  const WorkItem it = heavy[blockIdx.x];
  const ChunkRow r = chunk_row(it, rowptr, chunk);
  if (r.nch > kGiantChunks || r.nch <= fewer) return;
  const int SL = kWave >> log2_of(HP), cst = (chunk + SL - 1) >> log2_of(SL);
  if (cst <= 2) {
    grad_chunk_write<2, K>(perm, alpha, da, H, HP, it, r, pdot, ds);
  } else if (cst <= 4) {
    grad_chunk_write<4, K>(perm, alpha, da, H, HP, it, r, pdot, ds);
  } else if (K == 1 && cst <= 8) {
    grad_chunk_write<K == 1 ? 8 : 2, K>(perm, alpha, da, H, HP, it, r, pdot, ds);
  } else {  // single heads
    grad_chunk_write<0, 1>(perm, alpha, da, H * K, min(HP * K, kWave), it, r, pdot, ds);
  }
}

// A row of more than kGiantChunks chunks by a block of `waves` wavefronts: the sums
// added once per wavefront, and wavefront w writes chunks w, w + waves, ...
__device__ __forceinline__ void grad_giant_row(const SplitRow& sr, int w, int waves,
                                               const int* __restrict__ rowptr, int chunk,
                                               const int* __restrict__ perm,
                                               const float* __restrict__ alpha,
                                               const float* __restrict__ da, int H, int HP,
                                               const double* __restrict__ pdot,
                                               float* __restrict__ ds) {
  const int rb = uniform(rowptr[sr.row]), re = uniform(rowptr[sr.row + 1]);
  const int SL = kWave >> log2_of(HP), slot = lane_id() >> log2_of(HP), hh = lane_id() & (HP - 1);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    const double dot = row_dot(pdot + (int64_t)sr.slot0 * H + h, sr.nchunks, H, act, slot, SL, HP);
    for (int c = w; c < sr.nchunks; c += waves) {
      const int kb = rb + c * chunk, ke = min(re, kb + chunk);
      grad_sweep_write(perm, alpha, da, H, h, act, kb, ke, slot, SL, dot, ds);
    }
  }
}

__global__ __launch_bounds__(kGiantWaves * kWave) void softmax_grad_giant(
    const SplitRow* __restrict__ split, const int* __restrict__ rowptr, int chunk,
    const int* __restrict__ perm, const float* __restrict__ alpha, const float* __restrict__ da,
    int H, int HP, const double* __restrict__ pdot, float* __restrict__ ds) {
  const SplitRow sr = split[blockIdx.x];
  if (sr.nchunks <= kGiantChunks) return;
  const int w = uniform((int)threadIdx.x / kWave);
  grad_giant_row(sr, w, kGiantWaves, rowptr, chunk, perm, alpha, da, H, HP, pdot, ds);
}

// Split rows of at most kRowWaves chunks in the caller's order, one block each and a
// wavefront per chunk, whose values stay in registers while the chunks' sums meet in
// LDS. What bounds this order is the lines that scattered values move, and the two
// launches above read alpha and dalpha twice: 8M edges of a power-law graph, one head,
// 404 us before them, with them 561, now 400. Not where the two arrays fit the L2s (460
// rows of 1,400 chunks, 1.35M edges: 30 us, with them 8) or a value's line holds several
// heads. Two blocks share a CU (58 registers; with 70 one block, whose wavefronts past
// the row's chunks leave it idle: 4 heads, 398 us, now 302). The longest rows go in the
// same launch: one more of as many blocks costs 12 us where it finds nothing to do.
constexpr int kRowWaves = 16;
constexpr int kRowHeads = 4;
constexpr int kRowSteps = 8;  // values a lane holds
bool grad_by_rows(const Graph& g, int H, bool graph_order) {
  return !graph_order && H <= kRowHeads && g.n_split > 0 &&
         g.chunk * heads_per_pass(H) <= kRowSteps * kWave &&
         8.0 * (double)g.E * (double)H >= 32.0 * (1 << 20);
}
template <int NST>
__device__ __forceinline__ void grad_row(const int* __restrict__ perm,
                                         const float* __restrict__ alpha,
                                         const float* __restrict__ da, int H, int HP, int kb,
                                         int ke, int nch, int w, double (&sums)[kRowWaves][kRowHeads],
                                         float* __restrict__ ds) {
  const int SL = kWave >> log2_of(HP);
  const int slot = lane_id() >> log2_of(HP), h = lane_id() & (HP - 1);
  int e[NST];
  float a[NST][1], g[NST][1];
  load_ids<NST>(perm, kb, ke, slot, SL, e);
  grad_load<NST, 1>(alpha, da, H, h, h < H, e, a, g);
  const double dot = grad_dot<NST, 1>(a, g, 0, HP, kWave);
  if (slot == 0) sums[w][h] = dot;
  __syncthreads();
  double total[1] = {0.0};
  for (int c = 0; c < nch; ++c) total[0] += sums[c][h];
  grad_write<NST, 1>(a, g, e, total, H, h, h < H, ds);
}
__global__ __launch_bounds__(kRowWaves * kWave, 8) void softmax_grad_rows(
    const SplitRow* __restrict__ split, const int* __restrict__ rowptr, int chunk,
    const int* __restrict__ perm, const float* __restrict__ alpha, const float* __restrict__ da,
    int H, int HP, const double* __restrict__ pdot, float* __restrict__ ds) {
  __shared__ double sums[kRowWaves][kRowHeads];
  const SplitRow sr = split[blockIdx.x];
  const int re = uniform(rowptr[sr.row + 1]), w = uniform((int)threadIdx.x / kWave);
  if (sr.nchunks > kRowWaves) {  // uniform
    if (sr.nchunks > kGiantChunks)
      grad_giant_row(sr, w, kRowWaves, rowptr, chunk, perm, alpha, da, H, HP, pdot, ds);
    return;
  }
  // (wavefronts past the row's chunks hold no edges)
  const int kb = min(re, uniform(rowptr[sr.row]) + w * chunk), ke = min(re, kb + chunk);
  const int steps = chunk * HP;  // of a whole chunk, times the wavefront
  if (steps <= 2 * kWave) grad_row<2>(perm, alpha, da, H, HP, kb, ke, sr.nchunks, w, sums, ds);
  else if (steps <= 4 * kWave) grad_row<4>(perm, alpha, da, H, HP, kb, ke, sr.nchunks, w, sums, ds);
  else grad_row<kRowSteps>(perm, alpha, da, H, HP, kb, ke, sr.nchunks, w, sums, ds);
}

template <int MODE>
int launch_edge_grad(const Graph& g, const float* x, int64_t ldx, const float* dy,
                     const int* arg, int64_t F, int H, float* dw, int by_perm, hipStream_t s,
                     float scale = 1.0f) {
  const int D = (int)(F / H);
  const int vec = D >= 4 ? 4 : 1;
  int G = 1;  // lanes per head
  while (G < kWave && G * vec < D) G <<= 1;
  int lps = 4, waves;
  while (lps < std::min<int64_t>((int64_t)H * G, kWave)) lps <<= 1;
  SlotLists L{};
  const bool part_plan = use_part_plan(g, F);
  slot_lists(g, part_plan ? g.pexec : g.heavy, part_plan ? g.n_pexec : g.n_heavy, part_plan, lps,
             true, L, &waves);
  if (waves == 0) return TFG_OK;
  const bool narrow = (double)g.N_src * (double)ldx * 4.0 < 2147483648.0;
  // Four gathers per slot instead of eight where items have few edges and fill the
  // wavefront's lanes in one pass: places past an item's end repeat its last row, and
  // half the registers let eight wavefronts stay in flight for five (500,000 rows of 2
  // edges of 200 columns 322 -> 253 us; rows of 14 edges of 128 columns 199 and 206).
  const int items = part_plan ? g.n_pexec : g.n_heavy + g.n_long + g.n_short;
  const bool few = lps >= 32 && G * vec >= D && g.E <= 8 * (int64_t)items;
#define TFG_EG(VV, LL, UU)                                                                    \
  do {                                                                                        \
    if (narrow)                                                                               \
      edge_grad_slots<VV, LL, UU, MODE, true><<<(unsigned)waves, kItemBlock, 0, s>>>(         \
          L, g.rowptr, g.col, g.perm, x, ldx, dy, arg, H, D, G, dw, by_perm, scale);          \
    else                                                                                      \
      edge_grad_slots<VV, LL, UU, MODE, false><<<(unsigned)waves, kItemBlock, 0, s>>>(        \
          L, g.rowptr, g.col, g.perm, x, ldx, dy, arg, H, D, G, dw, by_perm, scale);          \
  } while (0)
#define TFG_EG_LPS(VV)                      \
  switch (lps) {                            \
    case 4: TFG_EG(VV, 4, 8); break;        \
    case 8: TFG_EG(VV, 8, 8); break;        \
    case 16: TFG_EG(VV, 16, 8); break;      \
    case 32: TFG_EG(VV, 32, 8); break;      \
    default: TFG_EG(VV, 64, 8); break;      \
  }
  if (vec == 4 && few && lps == 32) TFG_EG(4, 32, 4);
  else if (vec == 4 && few) TFG_EG(4, 64, 4);
  else if (vec == 4) TFG_EG_LPS(4)
  else TFG_EG_LPS(1)
#undef TFG_EG_LPS
#undef TFG_EG
  TFG_LAUNCHED("edge_grad_slots");
  return TFG_OK;
}

}  // namespace

// Bytes of the bucketed scatter's scratch (pairs, bucket table, scan sums);
// 0 where the plain scatter runs (several values per edge, small or very
// large graphs).
size_t perm_scatter_ws_bytes(int64_t E, int H) {
  if (H != 1 || E < (int64_t(1) << 20)) return 0;
  if (const char* v = std::getenv("TFG_PERM_BUCKETS"))  // "0": the plain scatter
    if (v[0] == '0') return 0;
  const int64_t nbuckets = (E + (int64_t(1) << kPermBits) - 1) >> kPermBits;
  if (nbuckets > kPermMaxBuckets) return 0;
  const int64_t ntiles = (E + kPermTile - 1) / kPermTile;
  const int64_t entries = nbuckets * ntiles;
  return align_up(sizeof(int2) * (size_t)E, 256) + align_up(sizeof(int) * (size_t)entries, 256) +
         align_up(sizeof(int) * (size_t)exclusive_scan_sums(entries), 256);
}

// out[perm[k], h] = in[k, h]; bucketed when ws holds perm_scatter_ws_bytes.
int launch_perm_scatter(const int* perm, int64_t E, int H, const float* in, float* out, void* ws,
                        size_t ws_bytes, hipStream_t s) {
  const int64_t n = E * H;
  if (n == 0) return TFG_OK;
  const size_t need = perm_scatter_ws_bytes(E, H);
  if (need == 0 || ws == nullptr || ws_bytes < need) {
    launch_reorder<true>(perm, E, H, in, out, s);
    TFG_LAUNCHED("to_edge_order");
    return TFG_OK;
  }
  const int nbuckets = (int)((E + (int64_t(1) << kPermBits) - 1) >> kPermBits);
  const int ntiles = (int)((E + kPermTile - 1) / kPermTile);
  const int64_t entries = (int64_t)nbuckets * ntiles;
  char* c = static_cast<char*>(ws);
  int2* pairs = reinterpret_cast<int2*>(c);
  c += align_up(sizeof(int2) * (size_t)E, 256);
  int* table = reinterpret_cast<int*>(c);
  c += align_up(sizeof(int) * (size_t)entries, 256);
  int* sums = reinterpret_cast<int*>(c);
  perm_count<<<ntiles, kPermThreads, 0, s>>>(perm, E, nbuckets, ntiles, table);
  TFG_LAUNCHED("perm_count");
  if (int rc = exclusive_scan(table, table, entries, sums, s)) return rc;
  perm_bucket<<<ntiles, kPermThreads, 0, s>>>(perm, in, E, nbuckets, ntiles, table, pairs);
  TFG_LAUNCHED("perm_bucket");
  perm_place<<<nbuckets, kPermThreads, 0, s>>>(pairs, table, ntiles, E, nbuckets, out);
  TFG_LAUNCHED("perm_place");
  return TFG_OK;
}


int launch_edge_dot(const Graph& g, const float* q, const float* key, int64_t ldk, int64_t F,
                    int H, float scale, float* out, int by_perm, hipStream_t s) {
  if (g.E == 0 || F == 0) return TFG_OK;
  return launch_edge_grad<kGradSum>(g, key, ldk, q, nullptr, F, H, out, by_perm, s, scale);
}

// Graph -> graph goes through edge order in the first E * H floats of ws;
// the scatter's scratch follows.
size_t edge_reorder_ws_bytes(int64_t E, int H, bool from, bool to) {
  const size_t tmp = (from && to) ? align_up(sizeof(float) * (size_t)std::max<int64_t>(E * H, 1), 256) : 0;
  return tmp + (from ? perm_scatter_ws_bytes(E, H) : 0);
}

int launch_edge_reorder(const int* perm_from, const int* perm_to, int64_t E, int H,
                        const float* in, float* out, void* ws, size_t ws_bytes, hipStream_t s) {
  const int64_t n = E * H;
  if (n == 0) return TFG_OK;
  if (perm_from != nullptr && perm_to != nullptr) {
    const size_t tb = align_up(sizeof(float) * (size_t)n, 256);
    float* tmp = static_cast<float*>(ws);
    const int rc = launch_perm_scatter(perm_from, E, H, in, tmp, static_cast<char*>(ws) + tb,
                                       ws_bytes > tb ? ws_bytes - tb : 0, s);
    if (rc) return rc;
    launch_reorder<false>(perm_to, E, H, tmp, out, s);
  } else if (perm_from != nullptr) {
    return launch_perm_scatter(perm_from, E, H, in, out, ws, ws_bytes, s);
  } else {
    launch_reorder<false>(perm_to, E, H, in, out, s);
  }
  TFG_LAUNCHED("edge reorder");
  return TFG_OK;
}

size_t aggregate_backward_ws_bytes(const Graph& g, const Graph* gt, int64_t F, int64_t H,
                                   int reduce, int w_order, bool has_w) {
  size_t b = 256;
  if (gt == nullptr) return b;
  const int64_t parts = use_part_plan(*gt, F) ? gt->n_pexec : gt->n_heavy;
  b += aggregate_partial_bytes(parts, F, TFG_SUM);
  const size_t ew = align_up(sizeof(float) * (size_t)std::max<int64_t>(g.E * H, 1), 256);
  // weights moved to edge order (and the bucketed scatter's scratch)
  if (has_w && w_order == TFG_CSR) b += ew + perm_scatter_ws_bytes(g.E, (int)H);
  if (reduce == TFG_MEAN) b += ew;           // weights / degree in transposed order
  return b;
}

int launch_aggregate_backward(const Graph& g, const Graph* gt, const float* w, int H, int w_order,
                              const float* x, int64_t ldx, const float* dy, int64_t F,
                              int reduce, const int32_t* argmax, float* dx, float* dw,
                              int dw_order, void* ws, hipStream_t s) {
  const int64_t EH = g.E * H;
  const unsigned eb = (unsigned)((EH + kBlock - 1) / kBlock);
  char* base = static_cast<char*>(ws);
  size_t off = 256;
  if (dx != nullptr && gt != nullptr) {
    const int64_t parts = use_part_plan(*gt, F) ? gt->n_pexec : gt->n_heavy;
    void* part = base + off;
    off += aggregate_partial_bytes(parts, F, TFG_SUM);
    const size_t ew = align_up(sizeof(float) * (size_t)std::max<int64_t>(EH, 1), 256);
    // weights for the gather over gt: in edge order (read through gt's perm)
    // or already in gt's order (read in sequence)
    const float* wg = w;
    int wg_order = w_order == TFG_CSR_T ? TFG_CSR : TFG_COO;
    if (w != nullptr && w_order == TFG_CSR && EH > 0) {
      float* t = reinterpret_cast<float*>(base + off);
      off += ew;
      const size_t sb = perm_scatter_ws_bytes(g.E, H);
      const int rc = launch_perm_scatter(g.perm, g.E, H, w, t, sb ? base + off : nullptr, sb, s);
      if (rc) return rc;
      off += sb;
      wg = t;
    }
    if (gt->N > 0 && F > 0) {
      int rc;
      if (reduce == TFG_MEAN) {
        float* wt = reinterpret_cast<float*>(base + off);
        off += ew;
        if (EH > 0) {
          mean_weights<<<eb, kBlock, 0, s>>>(gt->col, gt->perm, (unsigned)EH, (unsigned)H, g.rowptr, wg,
                                             wg_order == TFG_COO ? 1 : 0, wt);
          TFG_LAUNCHED("mean_weights");
        }
        rc = launch_aggregate(*gt, wt, H, TFG_CSR, dy, F, F, TFG_SUM, dx, nullptr, part, s);
      } else {
        rc = launch_aggregate(*gt, wg, wg ? H : 1, wg_order, dy, F, F, TFG_SUM, dx, nullptr, part,
                              s, 1.0f, 0.0f, nullptr, 0, reduce == TFG_MAX ? argmax : nullptr);
      }
      if (rc) return rc;
    }
  }
  if (dw != nullptr && EH > 0 && F > 0) {
    const int by_perm = dw_order == TFG_COO ? 1 : 0;
    int rc;
    if (reduce == TFG_MEAN)
      rc = launch_edge_grad<kGradMean>(g, x, ldx, dy, nullptr, F, H, dw, by_perm, s);
    else if (reduce == TFG_MAX)
      rc = launch_edge_grad<kGradMax>(g, x, ldx, dy, argmax, F, H, dw, by_perm, s);
    else
      rc = launch_edge_grad<kGradSum>(g, x, ldx, dy, nullptr, F, H, dw, by_perm, s);
    if (rc) return rc;
  }
  return TFG_OK;
}

int launch_segment_softmax_backward(const Graph& g, const float* alpha, const float* dalpha,
                                    int H, float* ds, void* ws, hipStream_t s, bool graph_order) {
  if (g.N == 0 || g.E == 0 || H == 0) return TFG_OK;
  const int* perm = graph_order ? nullptr : g.perm;  // alpha, dalpha, ds in the graph order
  const int hp = heads_per_pass(H);
  // the double part of the per-chunk statistics (row_stats_bytes layout)
  double* pdot = reinterpret_cast<double*>(
      static_cast<char*>(ws) +
      align_up(sizeof(float) * (size_t)std::max<int64_t>((int64_t)g.n_heavy * H, 1), 256));
  const int fewer = grad_by_rows(g, H, graph_order) ? kRowWaves : 0;
  const auto run = [&](auto k_) {
    constexpr int K = decltype(k_)::value;
    const int hk = H / K, hpk = heads_per_pass(hk);
    RowGroups L;
    const int64_t waves = row_groups<K>(g, hpk, L);
    if (waves > INT32_MAX) return fail(TFG_ERR_TOO_LARGE, "softmax gradient: too many work items");
    if (waves > 0) {
      softmax_grad_items<K><<<(unsigned)waves, kItemBlock, 0, s>>>(
          L, g.rowptr, g.chunk, fewer, perm, alpha, dalpha, hk, hpk, ds, pdot);
      TFG_LAUNCHED("softmax_grad_items");
    }
    if (g.n_heavy > 0) {
      softmax_grad_chunks<K><<<(unsigned)g.n_heavy, kItemBlock, 0, s>>>(
          g.heavy, g.rowptr, g.chunk, fewer, perm, alpha, dalpha, hk, hpk, pdot, ds);
      TFG_LAUNCHED("softmax_grad_chunks");
    }
    return (int)TFG_OK;
  };
  const int rc = H % 4 == 0 ? run(std::integral_constant<int, 4>{})
                            : run(std::integral_constant<int, 1>{});
  if (rc) return rc;
  if (fewer > 0) {
    softmax_grad_rows<<<(unsigned)g.n_split, kRowWaves * kWave, 0, s>>>(
        g.split, g.rowptr, g.chunk, perm, alpha, dalpha, H, hp, pdot, ds);
    TFG_LAUNCHED("softmax_grad_rows");
  } else if (g.n_heavy > kGiantChunks) {
    softmax_grad_giant<<<(unsigned)g.n_split, kGiantWaves * kWave, 0, s>>>(
        g.split, g.rowptr, g.chunk, perm, alpha, dalpha, H, hp, pdot, ds);
    TFG_LAUNCHED("softmax_grad_giant");
  }
  return TFG_OK;
}

}  // namespace tfg
