// Graph pooling over a sorted node -> graph index (gfx950): segment bounds
// from the sorted index (with range and order checks), then one wavefront per
// graph reducing its contiguous node rows (sum / mean / max + argmax); and its
// gradient, four nodes and a column vector per thread.
#include "wave.h"

namespace tfg {
namespace {

// four columns of a row at dword alignment (any width and leading dimension: the
// last lane of a row steps back to end at its last column)
typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int i4 __attribute__((ext_vector_type(4), aligned(4)));

__global__ void zero_ints(int* __restrict__ p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

__device__ __forceinline__ int64_t clamp_gid(int64_t g, int64_t G) {
  return g < -1 ? -1 : (g > G - 1 ? G - 1 : g);
}

// goff[g] = first node of graph g, goff[G] = Nb. Node n writes the starts of
// the graphs (gi[n-1], gi[n]]; the thread n = Nb writes the empty tail graphs.
// With valid sorted input every entry is written exactly once. Otherwise the
// error flag is set (unless err is NULL), and every entry is still written (so goff needs no
// clearing first) with a value in [0, Nb]: the clamped ids run from -1 (before
// node 0) to G (after node Nb - 1), so each g in [0, G] lies in (prev, cur] for
// the first n whose cur reaches g.
template <typename IdxT>
__global__ __launch_bounds__(kBlock) void segment_bounds(const IdxT* __restrict__ gi, int64_t Nb,
                                                         int64_t G, int* __restrict__ goff,
                                                         int* __restrict__ err) {
  int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n > Nb) return;
  int64_t prev = n > 0 ? (int64_t)gi[n - 1] : -1;
  int64_t cur;
  if (n < Nb) {
    cur = (int64_t)gi[n];
    int bad = 0;
    if (cur < 0 || cur >= G) bad |= kErrIndex;
    if (n > 0 && cur < prev) bad |= kErrUnsorted;
    if (bad != 0 && err != nullptr) atomicOr(err, bad);
  } else {
    cur = G;  // the tail: graphs after the last node's graph start at Nb
  }
  int64_t a = clamp_gid(prev, G), b = n < Nb ? clamp_gid(cur, G) : G;
  for (int64_t g = a + 1; g <= b; ++g) goff[g] = (int)n;
}

template <int V>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[V]) {
  if constexpr (V == 4) {
    f4 t = *reinterpret_cast<const f4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    v[0] = *p;
  }
}

template <int V>
__device__ __forceinline__ void store_row(float* __restrict__ p, const float (&v)[V]) {
  if constexpr (V == 4) __builtin_nontemporal_store(f4{v[0], v[1], v[2], v[3]}, reinterpret_cast<f4*>(p));
  else __builtin_nontemporal_store(v[0], p);
}

__device__ __forceinline__ void max_combine(float& v, int& a, float vb, int ab) {
  bool take = ab >= 0 && (a < 0 || vb > v || (vb == v && ab < a));
  v = take ? vb : v;
  a = take ? ab : a;
}

// One wavefront per graph; SLOTS node slots of 64/SLOTS lanes, U nodes in
// flight per slot, pairwise combination (as in the aggregation kernel).
template <int V, int SLOTS, bool MAX>
__global__ __launch_bounds__(kItemBlock) void pool_rows(const float* __restrict__ x, int64_t ldx,
                                                    int F, const int* __restrict__ goff, int64_t G,
                                                    int64_t Nb, int mean, float* __restrict__ out,
                                                    int* __restrict__ argout) {
  constexpr int LPS = kWave / SLOTS;
  constexpr int FC = LPS * V;
  constexpr int U = SLOTS * 8 <= kWave ? 8 : kWave / SLOTS;
  const int64_t g = (int64_t)blockIdx.x * (kItemBlock / kWave) + threadIdx.x / kWave;
  if (g >= G) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int slot = lane / LPS, sl = lane % LPS;
  int b = uniform(goff[g]), e = uniform(goff[g + 1]);
  b = b < 0 ? 0 : (b > Nb ? (int)Nb : b);
  e = e < b ? b : (e > Nb ? (int)Nb : e);
  for (int f0 = 0; f0 < F; f0 += FC) {
    const int fw = f0 + sl * V, f = min(fw, F - V);
    const bool fok = fw < F;
    float acc[U][V];
    int arg[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        acc[u][v] = 0.0f;
        arg[u][v] = -1;
      }
    for (int n0 = b; n0 < e; n0 += SLOTS * U) {
      float xv[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int n = n0 + u * SLOTS + slot;
        if (n < e && fok) {
          load_row<V>(x + (int64_t)n * ldx + f, xv[u]);
        } else {
#pragma unroll
          for (int v = 0; v < V; ++v) xv[u][v] = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int n = n0 + u * SLOTS + slot;
        if (n < e) {
#pragma unroll
          for (int v = 0; v < V; ++v) {
            if constexpr (MAX) {
              if (arg[u][v] < 0 || xv[u][v] > acc[u][v]) {
                acc[u][v] = xv[u][v];
                arg[u][v] = n;
              }
            } else {
              acc[u][v] += xv[u][v];
            }
          }
        }
      }
    }
#pragma unroll
    for (int step = 1; step < U; step <<= 1)
#pragma unroll
      for (int u = 0; u + step < U; u += 2 * step)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          if constexpr (MAX)
            max_combine(acc[u][v], arg[u][v], acc[u + step][v], arg[u + step][v]);
          else
            acc[u][v] += acc[u + step][v];
        }
#pragma unroll
    for (int off = LPS; off < kWave; off <<= 1)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float ov = __shfl_xor(acc[0][v], off);
        if constexpr (MAX) {
          const int oa = __shfl_xor(arg[0][v], off);
          max_combine(acc[0][v], arg[0][v], ov, oa);
        } else {
          acc[0][v] += ov;
        }
      }
    if (slot == 0 && fok) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        float r = acc[0][v];
        if (!MAX && mean && e > b) r = r / (float)(e - b);
        if (MAX && arg[0][v] < 0) r = 0.0f;
        out[g * F + f + v] = r;
        if (MAX && argout != nullptr) argout[g * F + f + v] = arg[0][v];
      }
    }
  }
}

template <int V, bool MAX>
void launch_pool_slots(int slots, dim3 grid, hipStream_t s, const float* x, int64_t ldx, int F,
                       const int* goff, int64_t G, int64_t Nb, int mean, float* out, int* argout) {
  switch (slots) {
    case 1: pool_rows<V, 1, MAX><<<grid, kItemBlock, 0, s>>>(x, ldx, F, goff, G, Nb, mean, out, argout); break;
    case 2: pool_rows<V, 2, MAX><<<grid, kItemBlock, 0, s>>>(x, ldx, F, goff, G, Nb, mean, out, argout); break;
    case 4: pool_rows<V, 4, MAX><<<grid, kItemBlock, 0, s>>>(x, ldx, F, goff, G, Nb, mean, out, argout); break;
    case 8: pool_rows<V, 8, MAX><<<grid, kItemBlock, 0, s>>>(x, ldx, F, goff, G, Nb, mean, out, argout); break;
    default: pool_rows<V, 16, MAX><<<grid, kItemBlock, 0, s>>>(x, ldx, F, goff, G, Nb, mean, out, argout); break;
  }
}

template <bool MAX>
void launch_pool_vec(int vec, int slots, dim3 grid, hipStream_t s, const float* x, int64_t ldx,
                     int F, const int* goff, int64_t G, int64_t Nb, int mean, float* out,
                     int* argout) {
  if (vec == 4)
    launch_pool_slots<4, MAX>(slots, grid, s, x, ldx, F, goff, G, Nb, mean, out, argout);
  else
    launch_pool_slots<1, MAX>(slots, grid, s, x, ldx, F, goff, G, Nb, mean, out, argout);
}

}  // namespace

namespace {

// Gradient of the pooling: dx[n, c] = dy[g, c] (sum), dy[g, c] / count(g) (mean),
// or dy[g, c] where node n won the forward max of (g, c), else 0. g = the clamped
// graph id; the counts come from the segment bounds. A thread takes V columns of
// kGradNodes nodes, lpr neighbouring threads a row, the chains from graph id to
// dy row of its nodes in flight together, and the stores stream past the L2s.
// Without the index check sum and max need no segment bounds. 1.05M nodes of 64
// columns: 63 us with one node per thread and a 64-bit division, now 46 (5.9 TB/s
// of stores); of 63 columns 151, now 60; 143,000 nodes 20, now 13.
constexpr int kGradNodes = 4;
template <typename IdxT, int V>
__global__ __launch_bounds__(kBlock) void pool_grad(const float* __restrict__ dy, int64_t G,
                                                    int F, const IdxT* __restrict__ gi,
                                                    int64_t Nb, const int* __restrict__ goff,
                                                    int reduce, const int* __restrict__ arg,
                                                    float* __restrict__ dx, int64_t ldx, int lpr, int lg,
                                                    int rows) {
  // (lg: log2 of lpr, or -1; rows: per block and step)
  const int r = lg >= 0 ? (int)threadIdx.x >> lg : (int)threadIdx.x / lpr;
  const int sub = (int)threadIdx.x - r * lpr;
  if (r >= rows) return;
  const int64_t n0 = (int64_t)blockIdx.x * (kGradNodes * rows) + r;
  int64_t g[kGradNodes];
  float cnt[kGradNodes];
#pragma unroll
  for (int u = 0; u < kGradNodes; ++u) {
    const int64_t n = n0 + u * rows;
    g[u] = n < Nb ? clamp_gid((int64_t)gi[n], G) : -1;
  }
#pragma unroll
  for (int u = 0; u < kGradNodes; ++u)
    cnt[u] = reduce == TFG_MEAN && g[u] >= 0 ? (float)(goff[g[u] + 1] - goff[g[u]]) : 1.0f;
  for (int fw = sub * V; fw < F; fw += V * lpr) {
    const int f = min(fw, F - V);
    float v[kGradNodes][V];
#pragma unroll
    for (int u = 0; u < kGradNodes; ++u) {
#pragma unroll
      for (int j = 0; j < V; ++j) v[u][j] = 0.0f;
      if (g[u] >= 0) load_row<V>(dy + g[u] * F + f, v[u]);
    }
    if (reduce == TFG_MEAN) {
#pragma unroll
      for (int u = 0; u < kGradNodes; ++u)
#pragma unroll
        for (int j = 0; j < V; ++j) v[u][j] = cnt[u] > 0.0f ? v[u][j] / cnt[u] : 0.0f;
    } else if (reduce == TFG_MAX) {
#pragma unroll
      for (int u = 0; u < kGradNodes; ++u)
        if (g[u] >= 0) {
          int a[V];
          if constexpr (V == 4) {
            const i4 t = *reinterpret_cast<const i4*>(arg + g[u] * F + f);
            a[0] = t.x; a[1] = t.y; a[2] = t.z; a[3] = t.w;
          } else {
            a[0] = arg[g[u] * F + f];
          }
#pragma unroll
          for (int j = 0; j < V; ++j) v[u][j] = a[j] == (int)(n0 + u * rows) ? v[u][j] : 0.0f;
        }
    }
#pragma unroll
    for (int u = 0; u < kGradNodes; ++u)
      if (n0 + u * rows < Nb) store_row<V>(dx + (n0 + u * rows) * ldx + f, v[u]);
  }
}

template <typename IdxT>
void launch_pool_grad(const float* dy, int64_t G, int F, const void* gi, int64_t Nb,
                      const int* goff, int reduce, const int* arg, float* dx, int64_t ldx,
                      hipStream_t s) {
  const int vec = F >= 4 ? 4 : 1;
  // threads per row: a power of two within a wavefront, else as many as it has
  // vectors, whole rows side by side in a block (143,000 nodes of 300 columns: two
  // passes of a wavefront 53 us, three rows of 75 threads 41)
  const int lanes = (F + vec - 1) / vec;
  int lg = 0;
  while (1 << lg < lanes && lg < 6) ++lg;
  int lpr = 1 << lg;
  if (lanes > kWave) {
    lpr = std::min(lanes, kBlock);
    lg = -1;
  }
  const int rows = kBlock / lpr;
  const int64_t per = (int64_t)kGradNodes * rows;
  const unsigned nb = (unsigned)((Nb + per - 1) / per);
  const IdxT* g = static_cast<const IdxT*>(gi);
  if (vec == 4)
    pool_grad<IdxT, 4><<<nb, kBlock, 0, s>>>(dy, G, F, g, Nb, goff, reduce, arg, dx, ldx, lpr, lg, rows);
  else
    pool_grad<IdxT, 1><<<nb, kBlock, 0, s>>>(dy, G, F, g, Nb, goff, reduce, arg, dx, ldx, lpr, lg, rows);
}

// The segment bounds (err NULL: nobody reads the flag).
int launch_segment_bounds(const void* graph_index, int index_type, int64_t Nb, int64_t G,
                          int* goff, int* err, hipStream_t s) {
  const unsigned nb = (unsigned)((Nb + 1 + kBlock - 1) / kBlock);
  if (index_type == TFG_I64)
    segment_bounds<int64_t><<<nb, kBlock, 0, s>>>(static_cast<const int64_t*>(graph_index), Nb, G,
                                                   goff, err);
  else
    segment_bounds<int32_t><<<nb, kBlock, 0, s>>>(static_cast<const int32_t*>(graph_index), Nb, G,
                                                   goff, err);
  TFG_LAUNCHED("segment_bounds");
  return TFG_OK;
}

}  // namespace

int launch_segment_pool_backward(const float* dy, int64_t G, int64_t F, const void* graph_index,
                                 int index_type, int64_t Nb, int reduce, const int32_t* argmax,
                                 float* dx, int64_t ldx, int* goff, int* err, hipStream_t s) {
  if (err != nullptr) zero_ints<<<1, 64, 0, s>>>(err, 1);
  if (Nb == 0 || F == 0) return TFG_OK;
  // the bounds: for the mean's counts, and where the index is to be checked
  if (err != nullptr || reduce == TFG_MEAN)
    if (int rc = launch_segment_bounds(graph_index, index_type, Nb, G, goff, err, s)) return rc;
  if (index_type == TFG_I64)
    launch_pool_grad<int64_t>(dy, G, (int)F, graph_index, Nb, goff, reduce, argmax, dx, ldx, s);
  else
    launch_pool_grad<int32_t>(dy, G, (int)F, graph_index, Nb, goff, reduce, argmax, dx, ldx, s);
  TFG_LAUNCHED("pool_grad");
  return TFG_OK;
}

int launch_segment_pool(const float* x, int64_t Nb, int64_t F, int64_t ldx, const void* graph_index,
                        int index_type, int64_t G, int reduce, float* out, int32_t* argmax,
                        int* goff, int* err, hipStream_t s) {
  if (err != nullptr) zero_ints<<<1, 64, 0, s>>>(err, 1);
  if (G == 0 || F == 0) return TFG_OK;
  if (int rc = launch_segment_bounds(graph_index, index_type, Nb, G, goff, err, s)) return rc;
  // Four columns a lane, any width; but where rows are no whole vectors of four, one
  // for sums of few nodes (200,000 graphs of 3 nodes, 31 columns: 55 us, with four 66),
  // for maxima of odd widths (30,000 graphs of 63 columns 53 us, with four 61), and for
  // maxima of even ones unless a graph's nodes fill its slots a few times (3 nodes of 30
  // columns 84 us, with four 181; 10,000 nodes 479 and 197)
  const auto slots_of = [&](int v) {
    const int lanes = (int)std::min<int64_t>((F + v - 1) / v, kWave);
    int p2 = 1;
    while (p2 < lanes) p2 <<= 1;
    return std::min(kWave / p2, 16);
  };
  int vec = F >= 4 ? 4 : 1;
  if (F % 4 != 0 && (reduce != TFG_MAX ? Nb < 16 * G : F % 2 != 0 || Nb < 32 * slots_of(4) * G)) vec = 1;
  const int slots = slots_of(vec);
  dim3 grid((unsigned)((G + kItemBlock / kWave - 1) / (kItemBlock / kWave)));
  if (reduce == TFG_MAX)
    launch_pool_vec<true>(vec, slots, grid, s, x, ldx, (int)F, goff, G, Nb, 0, out, argmax);
  else
    launch_pool_vec<false>(vec, slots, grid, s, x, ldx, (int)F, goff, G, Nb,
                           reduce == TFG_MEAN, out, argmax);
  TFG_LAUNCHED("pool_rows");
  return TFG_OK;
}

}  // namespace tfg
