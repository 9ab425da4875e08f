// Fused attention layers (gfx950): the sweep over the edges (gat_slots.h), the
// merge of the rows that went in pieces, and the optional coefficients
// alpha = exp(s - m) / d in a pass of their own. For the additive score the node
// projections a_s = a_src . h and a_d = a_dst . h come from node_projections()
// (softmax.hip) and sit in the workspace.
#include "gat_slots.h"

namespace tfg {
namespace rows {

void gat_additive(const GatShape& t, bool narrow, const SlotLists& L, int waves, const int* col,
                  int H, int D, const Scores& S, const float* h, const GatOut& O, hipStream_t s) {
  gat_dispatch<false>(t, narrow, L, waves, col, H, D, S, h, O, s);
}

}  // namespace rows

namespace {

using namespace rows;

constexpr int kMaxHeads = 64;

// Score of edge (c -> t) at head k, all D columns by one thread.
template <bool DOT>
__device__ __forceinline__ float edge_score(const Scores& sc, int64_t c, int64_t t, int k, int H,
                                            int D) {
  if constexpr (DOT) {
    const int64_t F = (int64_t)H * D;
    const float* qa = sc.q + t * F + (int64_t)k * D;
    const float* ka = sc.key + c * F + (int64_t)k * D;
    float acc = 0.0f;
    for (int d = 0; d < D; ++d) acc = __builtin_fmaf(qa[d], ka[d], acc);
    return sc.scale * acc;
  } else {
    return leaky(sc.as[c * H + k] + sc.ad[t * H + k], sc.slope);
  }
}

// Rows reduced from partial triples, `share` neighbouring slots of lps lanes per
// row: the row's maximum first, then the pieces weighed to it, kMergeU in flight
// and in no serial chain (the earlier running merge took an exponential per
// piece one after the other: 35 us for a hub of 190 pieces).
constexpr int kMergeU = 4;
template <int V>
__global__ __launch_bounds__(kItemBlock) void gat_merge(const SplitRow* __restrict__ split,
                                                        int n_split, int H, int D, int G, int lps,
                                                        int share, GatOut O) {
  const int lane = lane_id();
  const int q = blockIdx.x * (kWave / lps) + lane / lps;
  const int i = q / share, sub = q - i * share;
  const bool have = i < n_split;
  const SplitRow sr = split[have ? i : 0];
  const int nch = have ? sr.nchunks : 0;
  const int F = H * D;
  for (int p0 = 0; p0 < H * G; p0 += lps) {  // the lanes of gat_slots
    const int pl = p0 + (lane & (lps - 1));
    const bool fok = pl < H * G;
    const int head = min(pl / G, H - 1), g = fok ? pl - head * G : 0;
    const int f = head * D + min(g * V, D - V);
    const float* pm = O.pm + (int64_t)sr.slot0 * H + head;
    const double* pd = O.pd + (int64_t)sr.slot0 * H + head;
    const float* pa = O.pacc + (int64_t)sr.slot0 * F + f;
    float m = kNegInf;
    for (int j0 = sub; j0 < nch; j0 += kMergeU * share) {
      float t[kMergeU];
#pragma unroll
      for (int u = 0; u < kMergeU; ++u) t[u] = pm[(int64_t)min(j0 + u * share, nch - 1) * H];
#pragma unroll
      for (int u = 0; u < kMergeU; ++u) m = t[u] > m ? t[u] : m;
    }
    for (int o = lps; o < lps * share; o <<= 1) {
      const float t = __shfl_xor(m, o);
      m = t > m ? t : m;
    }
    double d = 0.0;
    float part[kMergeU][V];  // a chain per place, added up in pairs
#pragma unroll
    for (int u = 0; u < kMergeU; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) part[u][v] = 0.0f;
    for (int j0 = sub; j0 < nch; j0 += kMergeU * share) {
      float t[kMergeU], a[kMergeU][V];
      double e[kMergeU];
#pragma unroll
      for (int u = 0; u < kMergeU; ++u) {
        const int64_t j = min(j0 + u * share, nch - 1);
        t[u] = pm[j * H];
        e[u] = pd[j * H];
        load_row_once<V>(pa + j * F, a[u]);
      }
#pragma unroll
      for (int u = 0; u < kMergeU; ++u)
        if (j0 + u * share < nch) {
          const float w = t[u] == m ? 1.0f : expf(t[u] - m);
          d += e[u] * (double)w;
#pragma unroll
          for (int v = 0; v < V; ++v) part[u][v] = __builtin_fmaf(w, a[u][v], part[u][v]);
        }
    }
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v)
      acc[v] = (part[0][v] + part[1][v]) + (part[2][v] + part[3][v]);
    for (int o = lps; o < lps * share; o <<= 1) {
      d += __shfl_xor(d, o);
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += __shfl_xor(acc[v], o);
    }
    if (!have || !fok || sub != 0) continue;
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = nch > 0 ? (float)((double)acc[v] / d) : 0.0f;
    store_row<V>(O.out + (int64_t)sr.row * F + f, acc);
    if (O.rm != nullptr && g == 0) {
      O.rm[(int64_t)sr.row * H + head] = m;
      O.rd[(int64_t)sr.row * H + head] = d;
    }
  }
}

// Attention coefficients, one thread per graph position and K heads, written
// at the caller's edge ids.
template <bool DOT, int K>
__global__ __launch_bounds__(kBlock) void gat_alpha(const int* __restrict__ col,
                                                    const int* __restrict__ key,
                                                    const int* __restrict__ perm, int parts,
                                                    int64_t E, int H, int D, Scores S,
                                                    const float* __restrict__ rm,
                                                    const double* __restrict__ rd,
                                                    float* __restrict__ alpha_out) {
  const unsigned hk = (unsigned)H / K;  // groups of heads per position
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= E * hk) return;
  const int64_t k = i / hk;
  const int hh = (int)(i - k * hk) * K;
  const int64_t c = col[k], t = parts == 1 ? key[k] : key[k] / parts;
  float sc[K], m[K];
  double d[K];
  if constexpr (DOT) {
#pragma unroll
    for (int j = 0; j < K; ++j) sc[j] = edge_score<DOT>(S, c, t, hh + j, H, D);
  } else {
    float a[K], b[K];
    load_row<K>(S.as + c * H + hh, a);
    load_row<K>(S.ad + t * H + hh, b);
#pragma unroll
    for (int j = 0; j < K; ++j) sc[j] = leaky(a[j] + b[j], S.slope);
  }
  load_row<K>(rm + t * H + hh, m);
#pragma unroll
  for (int j = 0; j < K; ++j) d[j] = rd[t * H + hh + j];
#pragma unroll
  for (int j = 0; j < K; ++j) sc[j] = (float)((double)expf(sc[j] - m[j]) / d[j]);
  // (ordinary stores: scattered, the L2s join those of one line)
  float* o = alpha_out + (int64_t)perm[k] * H + hh;
#pragma unroll
  for (int j = 0; j < K; ++j) o[j] = sc[j];
}

struct GatLayout {
  size_t as, ad, rm, rd, pacc, pm, pd, total;
};

GatLayout gat_layout(int64_t N, int64_t H, int64_t F, int64_t n_partials) {
  GatLayout L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const size_t nh = (size_t)std::max<int64_t>(N * H, 1);
  L.as = take(sizeof(float) * nh);
  L.ad = take(sizeof(float) * nh);
  L.rm = take(sizeof(float) * nh);
  L.rd = take(sizeof(double) * nh);
  L.pacc = take(sizeof(float) * (size_t)std::max<int64_t>(n_partials * F, 1));
  L.pm = take(sizeof(float) * (size_t)std::max<int64_t>(n_partials * H, 1));
  L.pd = take(sizeof(double) * (size_t)std::max<int64_t>(n_partials * H, 1));
  L.total = off + 256;
  return L;
}

// The part plan where the gathered table (both tables of the dot product) is
// much larger than the L2s, as in the aggregation.
bool gat_part_plan(const Graph& g, int64_t F, bool dot) { return use_part_plan(g, dot ? 2 * F : F); }

int64_t gat_partials(const Graph& g, int64_t F, bool dot) {
  return gat_part_plan(g, F, dot) ? g.n_pexec : g.n_heavy;
}

template <bool DOT>
int run_attention(const Graph& g, int H, int D, const Scores& S, const float* h, float* out,
                  float* alpha_out, void* ws, hipStream_t s) {
  const int F = H * D;
  const bool part_plan = gat_part_plan(g, F, DOT);
  const GatLayout W = gat_layout(g.N, H, F, gat_partials(g, F, DOT));
  char* base = static_cast<char*>(ws);
  GatOut O{};
  O.out = out;
  if (alpha_out != nullptr) {
    O.rm = reinterpret_cast<float*>(base + W.rm);
    O.rd = reinterpret_cast<double*>(base + W.rd);
  }
  O.pacc = reinterpret_cast<float*>(base + W.pacc);
  O.pm = reinterpret_cast<float*>(base + W.pm);
  O.pd = reinterpret_cast<double*>(base + W.pd);
  const GatShape t = gat_shape(H, D, DOT);
  SlotLists L{};
  int waves;
  slot_lists(g, part_plan ? g.pexec : g.heavy, part_plan ? g.n_pexec : g.n_heavy, part_plan, t.lps,
             true, L, &waves);
  const bool narrow = (double)g.N_src * (double)F * 4.0 < 2147483648.0;
  if (waves > 0) {
    if (DOT) gat_dot(t, narrow, L, waves, g.col, H, D, S, h, O, s);
    else gat_additive(t, narrow, L, waves, g.col, H, D, S, h, O, s);
    TFG_LAUNCHED("gat_slots");
  }
  const SplitRow* rows = part_plan ? g.prows : g.split;
  const int n_rows = part_plan ? (int)g.N : g.n_split;
  if (n_rows > 0) {
    // the long rows of the row plan by a whole wavefront each
    const int share = part_plan ? 1 : kWave / t.lps;
    const unsigned nb = (unsigned)(((int64_t)n_rows * share * t.lps + kWave - 1) / kWave);
#define TFG_MERGE(V) gat_merge<V><<<nb, kItemBlock, 0, s>>>(rows, n_rows, H, D, t.G, t.lps, share, O)
    if (t.vec == 4) TFG_MERGE(4);
    else if (t.vec == 2) TFG_MERGE(2);
    else TFG_MERGE(1);
#undef TFG_MERGE
    TFG_LAUNCHED("gat_merge");
  }
  if (alpha_out != nullptr && g.E > 0) {
    const int K = H % 4 == 0 ? 4 : 1;
    const unsigned nb = (unsigned)((g.E * (H / K) + kBlock - 1) / kBlock);
    if (K == 4)
      gat_alpha<DOT, 4><<<nb, kBlock, 0, s>>>(g.col, g.key, g.perm, g.parts, g.E, H, D, S, O.rm,
                                              O.rd, alpha_out);
    else
      gat_alpha<DOT, 1><<<nb, kBlock, 0, s>>>(g.col, g.key, g.perm, g.parts, g.E, H, D, S, O.rm,
                                              O.rd, alpha_out);
    TFG_LAUNCHED("gat_alpha");
  }
  return TFG_OK;
}

}  // namespace

size_t gat_aggregate_ws_bytes(const Graph& g, int64_t H, int64_t D) {
  const int64_t F = H * D;
  return gat_layout(g.N, H, F, std::max(gat_partials(g, F, false), gat_partials(g, F, true))).total;
}

int max_fused_heads() { return kMaxHeads; }

int launch_gat_aggregate(const Graph& g, const float* h, int H, int D, const float* a_src,
                         const float* a_dst, float slope, float* out, float* alpha_out, void* ws,
                         hipStream_t s) {
  if (g.N == 0 || H == 0 || D == 0) return TFG_OK;
  const GatLayout W = gat_layout(g.N, H, (int64_t)H * D, gat_partials(g, (int64_t)H * D, false));
  float* as = reinterpret_cast<float*>(static_cast<char*>(ws) + W.as);
  float* ad = reinterpret_cast<float*>(static_cast<char*>(ws) + W.ad);
  Scores S{};
  S.as = as;
  S.ad = ad;
  S.slope = slope;
  const int rc = launch_node_projections(h, g.N, H, D, a_src, a_dst, as, ad, s);
  if (rc) return rc;
  return run_attention<false>(g, H, D, S, h, out, alpha_out, ws, s);
}

bool dot_attention_shape_ok(int64_t D) { return D >= 1 && D <= 64 && (D & (D - 1)) == 0; }

int launch_gat_dot_aggregate(const Graph& g, const float* q, const float* key, const float* v,
                             int H, int D, float scale, float* out, float* alpha_out, void* ws,
                             hipStream_t s) {
  if (g.N == 0 || H == 0 || D == 0) return TFG_OK;
  Scores S{};
  S.q = q;
  S.key = key;
  S.scale = scale;
  return run_attention<true>(g, H, D, S, v, out, alpha_out, ws, s);
}

}  // namespace tfg
