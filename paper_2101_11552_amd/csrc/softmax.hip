// Attention map -> reduce -> map (gfx950):
//   gat scores: per node and head, the dot products with a_src / a_dst; per
//               edge, LeakyReLU of their sum (the first map);
//   segment softmax: per target row and head, the maximum and the sum of the
//               shifted exponentials (the reduce, in one online sweep) and the
//               division (the last map), several work items of the graph's row
//               plan per wavefront.
#include <type_traits>

#include "softmax_stats.h"

namespace tfg {
namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

// a_s[n, k] = sum_d a_src[k, d] h[n, k*D + d]; a_d likewise (float32, d ascending).
__global__ __launch_bounds__(kBlock) void node_projections(const float* __restrict__ h, int64_t N,
                                                           int H, int D,
                                                           const float* __restrict__ a_src,
                                                           const float* __restrict__ a_dst,
                                                           float* __restrict__ as,
                                                           float* __restrict__ ad) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (node, head)
  if (i >= N * H) return;
  const int k = (int)(i % H);
  const float* hv = h + i * D;  // h[n, k*D ...] == h + (n*H + k) * D
  const float* s = a_src + (int64_t)k * D;
  const float* t = a_dst + (int64_t)k * D;
  float x = 0.0f, y = 0.0f;
  for (int d = 0; d < D; ++d) {
    const float v = hv[d];
    x = __builtin_fmaf(s[d], v, x);
    y = __builtin_fmaf(t[d], v, y);
  }
  as[i] = x;
  ad[i] = y;
}

// The same projections with lanes = (node, V columns): 64 / LPS nodes per
// wave, the V-column partial dots summed over the G = D / V lanes of each
// head with xor butterflies (G a power of two dividing LPS).
template <int V>
__global__ __launch_bounds__(kBlock) void node_projections_vec(
    const float* __restrict__ h, int64_t N, int H, int D, int LPS, int G,
    const float* __restrict__ a_src, const float* __restrict__ a_dst, float* __restrict__ as,
    float* __restrict__ ad) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int64_t n = wave * (kWave / LPS) + lane / LPS;
  const int sl = lane % LPS;
  const int F = H * D;
  const int f = sl * V;
  const bool ok = n < N && f < F;
  float x = 0.0f, y = 0.0f;
  if (ok) {
    float t[V];
    const float* hv = h + n * F + f;
    if constexpr (V == 4) {
      const f4 q = *reinterpret_cast<const f4*>(hv);
      t[0] = q.x; t[1] = q.y; t[2] = q.z; t[3] = q.w;
    } else if constexpr (V == 2) {
      const f2 q = *reinterpret_cast<const f2*>(hv);
      t[0] = q.x; t[1] = q.y;
    } else {
      t[0] = hv[0];
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      x = __builtin_fmaf(a_src[f + v], t[v], x);
      y = __builtin_fmaf(a_dst[f + v], t[v], y);
    }
  }
  for (int off = 1; off < G; off <<= 1) {
    x += __shfl_xor(x, off);
    y += __shfl_xor(y, off);
  }
  if (ok && sl % G == 0) {
    as[n * H + sl / G] = x;
    ad[n * H + sl / G] = y;
  }
}

// Launches the vectorised projections when the shape allows, else the simple ones.
void projections(const float* h, int64_t N, int H, int D, const float* a_src, const float* a_dst,
                 float* as, float* ad, hipStream_t s) {
  const int F = H * D;
  int vec = 1;
  for (int v : {4, 2}) {
    if (D % v == 0 && reinterpret_cast<uintptr_t>(h) % (4 * v) == 0) {
      vec = v;
      break;
    }
  }
  const int G = D / vec;
  const int lanes = F / vec;
  if ((G & (G - 1)) == 0 && lanes <= kWave) {
    int lps = 1;
    while (lps < lanes) lps <<= 1;
    const int64_t waves = (N + kWave / lps - 1) / (kWave / lps);
    const unsigned nb = (unsigned)((waves * kWave + kBlock - 1) / kBlock);
    if (vec == 4)
      node_projections_vec<4><<<nb, kBlock, 0, s>>>(h, N, H, D, lps, G, a_src, a_dst, as, ad);
    else if (vec == 2)
      node_projections_vec<2><<<nb, kBlock, 0, s>>>(h, N, H, D, lps, G, a_src, a_dst, as, ad);
    else
      node_projections_vec<1><<<nb, kBlock, 0, s>>>(h, N, H, D, lps, G, a_src, a_dst, as, ad);
  } else {
    node_projections<<<(unsigned)((N * H + kBlock - 1) / kBlock), kBlock, 0, s>>>(h, N, H, D, a_src,
                                                                                 a_dst, as, ad);
  }
}

template <typename IdxT>
__global__ __launch_bounds__(kBlock) void edge_scores(const IdxT* __restrict__ src,
                                                      const IdxT* __restrict__ tgt, int64_t E,
                                                      int64_t N, int H,
                                                      const float* __restrict__ as,
                                                      const float* __restrict__ ad, float slope,
                                                      float* __restrict__ out,
                                                      int* __restrict__ err) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (edge, head)
  if (i >= E * H) return;
  const int64_t e = i / H;
  const int k = (int)(i - e * H);
  int64_t s = (int64_t)src[e], t = (int64_t)tgt[e];
  if (s < 0 || s >= N || t < 0 || t >= N) {
    atomicOr(err, kErrIndex);
    s = (s < 0 || s >= N) ? 0 : s;
    t = (t < 0 || t >= N) ? 0 : t;
  }
  const float z = as[s * H + k] + ad[t * H + k];
  out[i] = z >= 0.0f ? z : slope * z;
}

// The same scores over a graph handle: one thread per graph position and K
// heads, the source from col, the target from the stored sort key (target *
// parts + part), written at the position (graph order) or at the edge id
// perm[k] (the caller's order). Same operands and operations as edge_scores.
// (E * H is below 2^31 here. One thread per head and a 64-bit division took 37 us
// for 1.35M edges and 8 heads.)
template <int K>
__global__ __launch_bounds__(kBlock) void edge_scores_graph(const int* __restrict__ col,
                                                            const int* __restrict__ key,
                                                            const int* __restrict__ perm,
                                                            int parts, unsigned n, unsigned hk,
                                                            const float* __restrict__ as,
                                                            const float* __restrict__ ad,
                                                            float slope, float* __restrict__ out) {
  const unsigned i = blockIdx.x * kBlock + threadIdx.x;  // (position, K heads)
  if (i >= n) return;
  const unsigned k = i / hk, h = i - k * hk;
  const int64_t sv = col[k], t = parts == 1 ? key[k] : key[k] / parts;
  const float* a = as + (sv * hk + h) * K;
  const float* b = ad + (t * hk + h) * K;
  float* o = out + ((int64_t)edge_at(perm, (int)k) * hk + h) * K;
  float z[K];
  if constexpr (K == 4) {
    const f4 u = *reinterpret_cast<const f4*>(a), v = *reinterpret_cast<const f4*>(b);
    z[0] = u.x + v.x; z[1] = u.y + v.y; z[2] = u.z + v.z; z[3] = u.w + v.w;
  } else {
    z[0] = a[0] + b[0];
  }
#pragma unroll
  for (int j = 0; j < K; ++j) z[j] = z[j] >= 0.0f ? z[j] : slope * z[j];
  if constexpr (K == 4) *reinterpret_cast<f4*>(o) = f4{z[0], z[1], z[2], z[3]};
  else o[0] = z[0];
}

// Rows and the chunks of long rows go in lane groups (softmax_stats.h).
// Items of at most group_steps() slot steps are swept once, over NST steps (a power
// of two, a template argument chosen per wavefront): their edge ids and scores
// are loaded together and stay in registers, the maximum comes from the
// registers and a butterfly over the slots, then each score is replaced by
// exp(s - m) and summed (butterfly again), and alpha is written from the
// registers. Items of more than group_steps() * 64 / HP edges (over 64 at 5 to 7, 12
// and 16 heads, over 32 at 9 to 15 and 20 to 32; a whole row or chunk has at most 128)
// keep a running pair instead (stat_add: maximum and rescaled sum in one sweep of
// loads) and load the scores again to write alpha.
constexpr int kSmSteps = 4;  // slot steps per round of loads (the running sweep)

// Scores of the heads h for the ids (-inf where there is no edge or no head).
template <int NST, int K>
__device__ __forceinline__ void load_scores(const float* __restrict__ s, int H, int h, bool act,
                                            const int (&e)[NST], float (&v)[NST][K]) {
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const bool ok = act && e[u] >= 0;
    if (ok) load_k<K>(s + ((int64_t)e[u] * H + h) * K, v[u]);
#pragma unroll
    for (int i = 0; i < K; ++i) v[u][i] = ok ? v[u][i] : -__builtin_huge_valf();
  }
}

__device__ __forceinline__ float slots_max(float m, int HP, int lanes) {
  for (int off = HP; off < lanes; off <<= 1) {
    const float o = __shfl_xor(m, off);
    m = o > m ? o : m;
  }
  return m;
}

__device__ __forceinline__ void slots_merge(float& m, double& d, int HP) {
  for (int off = HP; off < kWave; off <<= 1) {
    const float m2 = __shfl_xor(m, off);
    const double d2 = __shfl_xor(d, off);
    stat_merge(m, d, m2, d2);
  }
}

// Maximum of the registers of head i, over all slots of the head.
template <int NST, int K>
__device__ __forceinline__ float regs_max(const float (&v)[NST][K], int i, int HP, int lanes) {
  float m = -__builtin_huge_valf();
#pragma unroll
  for (int u = 0; u < NST; ++u) m = v[u][i] > m ? v[u][i] : m;
  return slots_max(m, HP, lanes);
}

// The registers' exp(v - m) (a missing edge, v = -inf, gives 0; with no maximum
// yet every score is -inf or NaN, and stays 0 or NaN), and their sum over all slots
// of the head: a lane's terms (at most 8) in float, or (WIDE) in a pair of floats.
__device__ __forceinline__ float exp_base(float m) { return m == -__builtin_huge_valf() ? 0.0f : m; }
template <bool WIDE, int NST, int K>
__device__ __forceinline__ double regs_exp_sum(float (&v)[NST][K], int i, float m, int HP,
                                               int lanes) {
  const float base = exp_base(m);
  float sum = 0.0f, low = 0.0f;  // low: what the float sum has lost
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    v[u][i] = expf(v[u][i] - base);
    const float t = sum + v[u][i];
    if constexpr (WIDE) {  // (exact: Knuth's two-sum)
      const float b = t - sum;
      low += (sum - (t - b)) + (v[u][i] - b);
    }
    sum = t;
  }
  return slots_sum(WIDE ? (double)sum + (double)low : (double)sum, HP, lanes);
}

// alpha = x * r for the registers' edges (x = exp(s - m), r = 1 / sum).
template <typename R, int NST, int K>
__device__ __forceinline__ void regs_write(float (&x)[NST][K], const int (&e)[NST],
                                           const R (&r)[K], int kb, int slot, int SL, int H,
                                           int h, bool act, float* __restrict__ out,
                                           float* __restrict__ out_csr) {
#pragma unroll
  for (int u = 0; u < NST; ++u)
    if (act && e[u] >= 0) {
#pragma unroll
      for (int i = 0; i < K; ++i) x[u][i] = (float)((R)x[u][i] * r[i]);
      store_k<K>(out + ((int64_t)e[u] * H + h) * K, x[u]);
      if (out_csr) store_k<K>(out_csr + ((int64_t)(kb + slot + u * SL) * H + h) * K, x[u]);
    }
}

// kSmSteps slot steps (positions k0, k0 + SL, ...) at a time: the edge ids,
// then the scores, issued together (e < 0: past the item or an inactive head).
__device__ __forceinline__ void load_steps(const int* __restrict__ perm,
                                           const float* __restrict__ s, int H, int h, bool act,
                                           int k0, int SL, int ke, int64_t (&e)[kSmSteps],
                                           float (&v)[kSmSteps]) {
#pragma unroll
  for (int u = 0; u < kSmSteps; ++u) {
    const int k = k0 + u * SL;
    e[u] = (act && k < ke) ? (int64_t)edge_at(perm, k) : -1;
  }
#pragma unroll
  for (int u = 0; u < kSmSteps; ++u) v[u] = e[u] >= 0 ? s[e[u] * H + h] : 0.0f;
}

// The running pair of [kb, ke) for head h, combined over the slots.
__device__ __forceinline__ void sweep_stats(const int* __restrict__ perm,
                                            const float* __restrict__ s, int H, int h, bool act,
                                            int kb, int ke, int slot, int SL, int HP, float& m,
                                            double& d) {
  m = -__builtin_huge_valf();
  d = 0.0;
  for (int k0 = kb + slot; k0 < ke; k0 += kSmSteps * SL) {
    int64_t e[kSmSteps];
    float v[kSmSteps];
    load_steps(perm, s, H, h, act, k0, SL, ke, e, v);
#pragma unroll
    for (int u = 0; u < kSmSteps; ++u)
      if (e[u] >= 0) stat_add(m, d, v[u]);
  }
  slots_merge(m, d, HP);
}

// alpha = exp(s - m) * r over [kb, ke), loading the scores again.
__device__ __forceinline__ void sweep_write(const int* __restrict__ perm,
                                            const float* __restrict__ s, int H, int h, bool act,
                                            int kb, int ke, int slot, int SL, float m, double r,
                                            float* __restrict__ out,
                                            float* __restrict__ out_csr) {
  for (int k0 = kb + slot; k0 < ke; k0 += kSmSteps * SL) {
    int64_t e[kSmSteps];
    float v[kSmSteps];
    load_steps(perm, s, H, h, act, k0, SL, ke, e, v);
#pragma unroll
    for (int u = 0; u < kSmSteps; ++u)
      if (e[u] >= 0) {
        const float a = (float)((double)expf(v[u] - m) * r);
        out[e[u] * H + h] = a;
        if (out_csr) out_csr[(int64_t)(k0 + u * SL) * H + h] = a;
      }
  }
}

// One item per group from the registers: a whole row (pslot < 0) writes alpha,
// a chunk of a split row its pair. WIDE: the sum and its reciprocal in double, as in
// the running sweep (in float they cost 3% of alpha's accuracy); short rows, whose
// sums have few terms, take them in float (4 to 10% of the time at 8 to 16 heads).
template <int NST, int K, bool WIDE = false>
__device__ __forceinline__ void item_regs(const int* __restrict__ perm,
                                          const float* __restrict__ s, int H, int HP,
                                          const GroupItem& it, float* __restrict__ out,
                                          float* __restrict__ out_csr, float* __restrict__ pm,
                                          double* __restrict__ pd) {
  const int SL = it.lanes >> log2_of(HP);
  const int slot = (lane_id() & (it.lanes - 1)) >> log2_of(HP), hh = lane_id() & (HP - 1);
  int e[NST];
  load_ids<NST>(perm, it.kb, it.ke, slot, SL, e);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    float v[NST][K], m[K];
    double d[K];
    load_scores<NST, K>(s, H, h, act, e, v);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      m[i] = regs_max<NST, K>(v, i, HP, it.lanes);
      d[i] = regs_exp_sum<WIDE, NST, K>(v, i, m[i], HP, it.lanes);
    }
    if (it.pslot < 0) {
      using RT = typename std::conditional<WIDE, double, float>::type;
      RT r[K];
#pragma unroll
      for (int i = 0; i < K; ++i) r[i] = (RT)(1.0 / d[i]);
      regs_write<RT, NST, K>(v, e, r, it.kb, slot, SL, H, h, act, out, out_csr);
    } else if (slot == 0 && act) {
#pragma unroll
      for (int i = 0; i < K; ++i) {
        pm[((int64_t)it.pslot * H + h) * K + i] = m[i];
        pd[((int64_t)it.pslot * H + h) * K + i] = d[i];
      }
    }
  }
}

// 1.35M edges and 8 heads, rows of 8 on average: 35 us with one wavefront per row of
// over 8 edges and one head per lane, now 27.
template <int K>
__global__ __launch_bounds__(kItemBlock) void softmax_items(
    RowGroups L, const int* __restrict__ perm, const float* __restrict__ s, int H, int HP,
    float* __restrict__ out, float* __restrict__ out_csr, float* __restrict__ pm,
    double* __restrict__ pd) {
  const GroupItem it = group_item(L, blockIdx.x);
  const int SL = it.lanes >> log2_of(HP), n = it.ke - it.kb;
  if (!__any(n > SL)) {
    item_regs<1, K>(perm, s, H, HP, it, out, out_csr, pm, pd);
  } else if (!__any(n > 2 * SL)) {
    item_regs<2, K>(perm, s, H, HP, it, out, out_csr, pm, pd);
  } else if (K == 4 && it.lanes == kWave && n <= 4 * SL) {  // more than 512 values
    item_regs<4, K, true>(perm, s, H, HP, it, out, out_csr, pm, pd);
  } else if (!__any(n > 4 * SL)) {
    item_regs<4, K>(perm, s, H, HP, it, out, out_csr, pm, pd);
  } else if (K == 1 && !__any(n > 8 * SL)) {
    item_regs<K == 1 ? 8 : 1, K>(perm, s, H, HP, it, out, out_csr, pm, pd);
  } else {  // groups of 64 lanes: one item; single heads
    const int H1 = H * K, hp = min(HP * K, kWave), sl1 = kWave >> log2_of(hp);
    const int slot = lane_id() >> log2_of(hp), hh = lane_id() & (hp - 1);
    for (int hb = 0; hb < H1; hb += hp) {
      const int h = hb + hh;
      const bool act = h < H1;
      float m;
      double d;
      sweep_stats(perm, s, H1, h, act, it.kb, it.ke, slot, sl1, hp, m, d);
      if (it.pslot < 0) {
        sweep_write(perm, s, H1, h, act, it.kb, it.ke, slot, sl1, m, 1.0 / d, out, out_csr);
      } else if (slot == 0 && act) {
        pm[(int64_t)it.pslot * H1 + h] = m;
        pd[(int64_t)it.pslot * H1 + h] = d;
      }
    }
  }
}

// The pair of a split row for head h from its chunks' pairs, a share per slot,
// then over the slots: the maximum, then the sums weighed to it, four pairs in
// flight.
__device__ __forceinline__ void row_pair(const float* __restrict__ pm,
                                         const double* __restrict__ pd, int nch, int H, bool act,
                                         int slot, int SL, int HP, float& m, double& d) {
  constexpr int U = 4;
  m = -__builtin_huge_valf();
  d = 0.0;
  if (act)
    for (int c = slot; c < nch; c += U * SL) {
      float t[U];
#pragma unroll
      for (int u = 0; u < U; ++u) t[u] = pm[(int64_t)min(c + u * SL, nch - 1) * H];
#pragma unroll
      for (int u = 0; u < U; ++u) m = t[u] > m ? t[u] : m;
    }
  m = slots_max(m, HP, kWave);
  if (act)
    for (int c = slot; c < nch; c += U * SL) {
      float t[U];
      double q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t j = (int64_t)min(c + u * SL, nch - 1) * H;
        t[u] = pm[j];
        q[u] = pd[j];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u * SL < nch) d += q[u] * (double)(t[u] == m ? 1.0f : expf(t[u] - m));
    }
  d = slots_sum(d, HP, kWave);
}

// Alpha of the chunks of split rows, one wavefront per chunk. (One block of 16
// wavefronts per split row, with the chunks' pairs combined behind barriers: 24
// us for 1,400 chunks of 460 rows, now 11.)
template <int NST, int K>
__device__ __forceinline__ void chunk_write(const int* __restrict__ perm,
                                            const float* __restrict__ s, int H, int HP,
                                            const WorkItem& it, const ChunkRow& r,
                                            const float* __restrict__ pm,
                                            const double* __restrict__ pd,
                                            float* __restrict__ out,
                                            float* __restrict__ out_csr) {
  const int SL = kWave >> log2_of(HP);
  const int slot = lane_id() >> log2_of(HP), hh = lane_id() & (HP - 1);
  constexpr int R = NST > 0 ? NST : 1;  // registers (NST = 0: the scores loaded in rounds)
  int e[R];
  if constexpr (NST > 0) load_ids<NST>(perm, it.kbeg, it.kend, slot, SL, e);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    float v[R][K], m[K];
    double inv[K];
    if constexpr (NST > 0) load_scores<NST, K>(s, H, h, act, e, v);
    const int64_t p0 = ((int64_t)r.slot0 * H + h) * K;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      double d;
      row_pair(pm + p0 + i, pd + p0 + i, r.nch, H * K, act, slot, SL, HP, m[i], d);
      if constexpr (NST > 0) inv[i] = 1.0 / d;
      else sweep_write(perm, s, H, h, act, it.kbeg, it.kend, slot, SL, m[i], 1.0 / d, out, out_csr);
    }
    if constexpr (NST > 0) {
#pragma unroll
      for (int u = 0; u < NST; ++u)
#pragma unroll
        for (int i = 0; i < K; ++i) v[u][i] = expf(v[u][i] - m[i]);
      regs_write<double, NST, K>(v, e, inv, it.kbeg, slot, SL, H, h, act, out, out_csr);
    }
  }
}

template <int K>
__global__ __launch_bounds__(kItemBlock) void softmax_chunks(
    const WorkItem* __restrict__ heavy, const int* __restrict__ rowptr, int chunk,
    const int* __restrict__ perm, const float* __restrict__ s, int H, int HP,
    const float* __restrict__ pm, const double* __restrict__ pd, float* __restrict__ out,
    float* __restrict__ out_csr) {
  const WorkItem it = heavy[blockIdx.x];
  const ChunkRow r = chunk_row(it, rowptr, chunk);
  if (r.nch > kGiantChunks) return;
  const int SL = kWave >> log2_of(HP), cst = (chunk + SL - 1) >> log2_of(SL);
  if (cst <= 2) {
    chunk_write<2, K>(perm, s, H, HP, it, r, pm, pd, out, out_csr);
  } else if (cst <= 4) {
    chunk_write<4, K>(perm, s, H, HP, it, r, pm, pd, out, out_csr);
  } else if (K == 1 && cst <= 8) {
    chunk_write<K == 1 ? 8 : 2, K>(perm, s, H, HP, it, r, pm, pd, out, out_csr);
  } else {  // single heads
    chunk_write<0, 1>(perm, s, H * K, min(HP * K, kWave), it, r, pm, pd, out, out_csr);
  }
}

// Rows of more than kGiantChunks chunks: the pairs combined once per wavefront
// of the row's block, and wavefront w writes chunks w, w + kGiantWaves, ...
__global__ __launch_bounds__(kGiantWaves * kWave) void softmax_giant(
    const SplitRow* __restrict__ split, const int* __restrict__ rowptr, int chunk,
    const int* __restrict__ perm, const float* __restrict__ s, int H, int HP,
    const float* __restrict__ pm, const double* __restrict__ pd, float* __restrict__ out,
    float* __restrict__ out_csr) {
  const SplitRow sr = split[blockIdx.x];
  if (sr.nchunks <= kGiantChunks) return;
  const int rb = uniform(rowptr[sr.row]), re = uniform(rowptr[sr.row + 1]);
  const int w = uniform((int)threadIdx.x / kWave);
  const int SL = kWave >> log2_of(HP), slot = lane_id() >> log2_of(HP), hh = lane_id() & (HP - 1);
  for (int hb = 0; hb < H; hb += HP) {
    const int h = hb + hh;
    const bool act = h < H;
    float m;
    double d;
    const int64_t p0 = (int64_t)sr.slot0 * H + h;
    row_pair(pm + p0, pd + p0, sr.nchunks, H, act, slot, SL, HP, m, d);
    for (int c = w; c < sr.nchunks; c += kGiantWaves) {
      const int kb = rb + c * chunk, ke = min(re, kb + chunk);
      sweep_write(perm, s, H, h, act, kb, ke, slot, SL, m, 1.0 / d, out, out_csr);
    }
  }
}

}  // namespace

int launch_node_projections(const float* h, int64_t N, int H, int D, const float* a_src,
                            const float* a_dst, float* as, float* ad, hipStream_t s) {
  if (N * H == 0) return TFG_OK;
  projections(h, N, H, D, a_src, a_dst, as, ad, s);
  TFG_LAUNCHED("node_projections");
  return TFG_OK;
}

int launch_gat_scores(const void* edge_index, int index_type, int64_t E, const float* h, int64_t N,
                      int H, int D, const float* a_src, const float* a_dst, float slope,
                      float* out, float* proj, int* err, hipStream_t s) {
  float* as = proj;
  float* ad = proj + N * H;
  if (N * H > 0) {
    projections(h, N, H, D, a_src, a_dst, as, ad, s);
    TFG_LAUNCHED("node_projections");
  }
  if (E * H > 0) {
    const unsigned nb = (unsigned)((E * H + kBlock - 1) / kBlock);
    if (index_type == TFG_I64) {
      const int64_t* ei = static_cast<const int64_t*>(edge_index);
      edge_scores<int64_t><<<nb, kBlock, 0, s>>>(ei, ei + E, E, N, H, as, ad, slope, out, err);
    } else {
      const int32_t* ei = static_cast<const int32_t*>(edge_index);
      edge_scores<int32_t><<<nb, kBlock, 0, s>>>(ei, ei + E, E, N, H, as, ad, slope, out, err);
    }
    TFG_LAUNCHED("edge_scores");
  }
  return TFG_OK;
}

int launch_gat_graph_scores(const Graph& g, const float* h, int H, int D, const float* a_src,
                            const float* a_dst, float slope, float* out, int by_perm,
                            float* proj, hipStream_t s) {
  float* as = proj;
  float* ad = proj + g.N * H;
  if (g.N * H > 0) {
    projections(h, g.N, H, D, a_src, a_dst, as, ad, s);
    TFG_LAUNCHED("node_projections");
  }
  if (g.E * H > 0) {
    // (16-byte accesses: the projections sit in the workspace, rows of 4-head groups)
    const int K = H % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0 && g.N * H % 4 == 0 ? 4 : 1;
    const unsigned hk = (unsigned)(H / K), n = (unsigned)(g.E * hk);
    const unsigned nb = (unsigned)(((int64_t)n + kBlock - 1) / kBlock);
    const int* perm = by_perm ? g.perm : nullptr;
    if (K == 4)
      edge_scores_graph<4><<<nb, kBlock, 0, s>>>(g.col, g.key, perm, g.parts, n, hk, as, ad, slope, out);
    else
      edge_scores_graph<1><<<nb, kBlock, 0, s>>>(g.col, g.key, perm, g.parts, n, hk, as, ad, slope, out);
    TFG_LAUNCHED("edge_scores_graph");
  }
  return TFG_OK;
}

size_t row_stats_bytes(int64_t n_chunks, int64_t H) {
  const size_t n = (size_t)std::max<int64_t>(n_chunks * H, 1);
  return align_up(sizeof(float) * n, 256) + align_up(sizeof(double) * n, 256);
}

int launch_segment_softmax(const Graph& g, const float* scores, int H, float* out, float* out_csr,
                           void* ws, hipStream_t s, bool graph_order) {
  if (g.N == 0 || g.E == 0 || H == 0) return TFG_OK;
  // scores and alpha in the graph order: position k is edge k, one output
  const int* perm = graph_order ? nullptr : g.perm;
  if (graph_order) out_csr = nullptr;
  const int hp = heads_per_pass(H);
  float* pm = static_cast<float*>(ws);
  double* pd = reinterpret_cast<double*>(
      static_cast<char*>(ws) + align_up(sizeof(float) * (size_t)std::max<int64_t>((int64_t)g.n_heavy * H, 1), 256));
  const auto run = [&](auto k_) {
    constexpr int K = decltype(k_)::value;
    const int hk = H / K, hpk = heads_per_pass(hk);
    RowGroups L;
    const int64_t waves = row_groups<K>(g, hpk, L);
    if (waves > INT32_MAX) return fail(TFG_ERR_TOO_LARGE, "segment softmax: too many work items");
    if (waves > 0) {
      softmax_items<K><<<(unsigned)waves, kItemBlock, 0, s>>>(L, perm, scores, hk, hpk, out,
                                                              out_csr, pm, pd);
      TFG_LAUNCHED("softmax_items");
    }
    if (g.n_heavy > 0) {
      softmax_chunks<K><<<(unsigned)g.n_heavy, kItemBlock, 0, s>>>(
          g.heavy, g.rowptr, g.chunk, perm, scores, hk, hpk, pm, pd, out, out_csr);
      TFG_LAUNCHED("softmax_chunks");
    }
    return (int)TFG_OK;
  };
  const int rc = H % 4 == 0 ? run(std::integral_constant<int, 4>{})
                            : run(std::integral_constant<int, 1>{});
  if (rc) return rc;
  if (g.n_heavy > kGiantChunks) {
    softmax_giant<<<(unsigned)g.n_split, kGiantWaves * kWave, 0, s>>>(
        g.split, g.rowptr, g.chunk, perm, scores, H, hp, pm, pd, out, out_csr);
    TFG_LAUNCHED("softmax_giant");
  }
  return TFG_OK;
}

}  // namespace tfg
