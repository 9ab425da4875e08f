// Message aggregation over the CSR-by-target graph (gfx950, wave64):
// out[t, :] = reduce over the edges k of row t of w_k * x[col_k, :].
// The work items of the graph's plan go to the slot kernel (slots.h) or to
// spmm_wide; long rows and source-part segments leave partial rows that
// fixup_rows combines in a fixed order. No floating-point atomics: every
// output is reproducible bit for bit.
#include <cstdlib>
#include <mutex>

#include "spmm.h"

namespace tfg {
namespace {

// Device memory of the no-allocation aggregation (tfg_aggregate_noalloc): the
// partial rows that tfg_aggregate keeps in its workspace. Every GPU the
// library runs on holds its own copy until the process ends. In host code the
// name only stands for the symbol: kernels get the device address that
// hipGetSymbolAddress returns for the current device.
__device__ __align__(256) unsigned char scratch[TFG_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

using namespace rows;

// Combines the partial results of each split row: `share` neighbouring slots of
// lps lanes take a row's partials in turn, each kFixAcc partial rows in flight (sums
// with one accumulator each, combined pairwise; maxima with the tie rule), and are
// combined pairwise themselves. A lane covers V consecutive features; the last lane
// with features of its own steps back to end at F (it repeats some of its
// neighbour's). What bounds a hub row is the chain of loads over its partials: one
// slot took 1.78 ms for an aggregation with the maxima of 4,700 partials of 4 columns
// (one wavefront without column vectors 0.86), sixteen slots 0.14.
constexpr int kFixAcc = 8;
template <bool MAX, int V>
__global__ __launch_bounds__(kItemBlock) void fixup_rows(const SplitRow* __restrict__ split,
                                                     int n_split, const float* __restrict__ part,
                                                     const int* __restrict__ part_arg, int F,
                                                     int mean, float* __restrict__ out,
                                                     int* __restrict__ argout, Epilogue ep,
                                                     int lps, int share) {
  const int lane = threadIdx.x & (kWave - 1);
  const int per = kWave / (lps * share);  // rows per wavefront
  const int wid = blockIdx.x * per + lane / (lps * share);
  const bool have = wid < n_split;
  const SplitRow sr = split[have ? wid : 0];
  const int row = sr.row, slot0 = sr.slot0, nch = have ? sr.nchunks : 0, deg = sr.deg;
  const int sub = lane / lps & (share - 1);
  for (int f0 = 0; f0 < F; f0 += lps * V) {
    const int fw = f0 + (lane & (lps - 1)) * V;
    const bool fok = fw < F;
    const int f = min(fw, F - V);
    if constexpr (MAX) {
      constexpr int U = kFixAcc / 2;  // two rows each: values and edge ids
      float best[V];
      int a[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        best[v] = 0.0f;
        a[v] = -1;
      }
      for (int j = sub; j < nch; j += U * share) {
        float t[U][V];
        int e[U][V];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          // places past the row's partials repeat the last one, which never wins again
          const int64_t o = (int64_t)(slot0 + min(j + i * share, nch - 1)) * F + f;
          load_row_once<V>(part + o, t[i]);
          load_irow<V>(part_arg + o, e[i]);
        }
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
          for (int v = 0; v < V; ++v) max_combine(best[v], a[v], t[i][v], e[i][v]);
      }
      for (int o = lps; o < lps * share; o <<= 1)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float t = __shfl_xor(best[v], o);
          const int e = __shfl_xor(a[v], o);
          max_combine(best[v], a[v], t, e);
        }
#pragma unroll
      for (int v = 0; v < V; ++v) best[v] = a[v] < 0 ? 0.0f : best[v];
      if (have && fok && sub == 0) {
        store_row<V>(out + (int64_t)row * F + f, best);
        if (argout != nullptr) store_irow<V>(argout + (int64_t)row * F + f, a);
      }
    } else {
      // kFixAcc partial rows in flight, one accumulator each
      float a4[kFixAcc][V];
#pragma unroll
      for (int i = 0; i < kFixAcc; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) a4[i][v] = 0.0f;
      for (int j = sub; j < nch; j += kFixAcc * share) {
        float t[kFixAcc][V];
#pragma unroll
        for (int i = 0; i < kFixAcc; ++i) {
          if (j + i * share < nch) {
            load_row_once<V>(part + (int64_t)(slot0 + j + i * share) * F + f, t[i]);
          } else {
#pragma unroll
            for (int v = 0; v < V; ++v) t[i][v] = 0.0f;
          }
        }
#pragma unroll
        for (int i = 0; i < kFixAcc; ++i)
#pragma unroll
          for (int v = 0; v < V; ++v) a4[i][v] += t[i][v];
      }
#pragma unroll
      for (int step = 1; step < kFixAcc; step <<= 1)
#pragma unroll
        for (int i = 0; i + step < kFixAcc; i += 2 * step)
#pragma unroll
          for (int v = 0; v < V; ++v) a4[i][v] += a4[i + step][v];
      for (int o = lps; o < lps * share; o <<= 1)
#pragma unroll
        for (int v = 0; v < V; ++v) a4[0][v] += __shfl_xor(a4[0][v], o);
      if (have && fok && sub == 0) {
        float s[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          s[v] = a4[0][v];
          if (mean && deg > 0) s[v] = s[v] / (float)deg;
        }
        apply_epilogue<V>(ep, row, f, s);
        store_row<V>(out + (int64_t)row * F + f, s);
      }
    }
  }
}

// Sum and mean over the part plan (every item writes a partial) with scalar edge
// ids: one wavefront per work item, two edge slots of 32 lanes, lane l of a slot holding columns 4 l ..
// 4 l + 3 of a 128-column row. The item's edge ids and weights come in with one
// coalesced load per 64 edges and are read out edge by edge into scalar
// registers (readlane); the scalar unit forms each row's 32-bit byte offset
// (NARROW: the table below 2 GB; else 64-bit per lane), so a lane adds its own
// offset and selects between the slots' values, and the load takes the table's
// base from scalar registers. Edges go in groups of kWideU per slot (4: 3.51 ms
// on the power-law graph; 8: 3.69, 2: 3.51), every load of a group issued
// before its first multiply-add; the last group repeats the item's last edge in
// its unused places (a row already loaded) and adds only the item's own edges.
// One accumulator chain per group place, combined pairwise, then across the
// slots.
constexpr int kWideU = 4;
template <bool NARROW>
__global__ __launch_bounds__(kRowBlock) void spmm_wide(
    const WorkItem* __restrict__ items, int n_items, const int* __restrict__ col,
    const int* __restrict__ perm, const float* __restrict__ w, int w_by_perm,
    const float* __restrict__ x, int64_t ldx, int F, float* __restrict__ part) {
  constexpr int V = 4, SL = 2, U = kWideU, LPS = kWave / SL;
  const int wid = uniform(blockIdx.x * (kRowBlock / kWave) + threadIdx.x / kWave);
  if (wid >= n_items) return;
  const int lane = lane_id();
  const int slot = lane / LPS, sl = lane % LPS;
  const WorkItem* itp = items + wid;
  const int kbeg = uniform(itp->kbeg), kend = uniform(itp->kend), pslot = uniform(itp->slot);
  const char* xb = reinterpret_cast<const char*>(x);
  const int64_t row_bytes = ldx * (int64_t)sizeof(float);
  const int f = sl * V;
  const unsigned lane_off = (unsigned)f * (unsigned)sizeof(float);
  float acc[U][V];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[u][v] = 0.0f;
  for (int kb = kbeg; kb < kend; kb += kWave) {
    const int n = min(kWave, kend - kb);
    const bool lok = lane < n;
    const int cj = lok ? __builtin_nontemporal_load(col + kb + lane) : 0;
    float wf = 1.0f;
    if (w != nullptr && lok)  // weights in graph order, or in the caller's edge order
      wf = w_by_perm ? w[__builtin_nontemporal_load(perm + kb + lane)]
                     : __builtin_nontemporal_load(w + kb + lane);
    const int wj = __float_as_int(wf);
    auto group = [&](int j0, bool tail) {
      float xv[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ja = j0 + u * SL;
        const int ca = __builtin_amdgcn_readlane(cj, tail ? min(ja, n - 1) : ja);
        const int cb = __builtin_amdgcn_readlane(cj, tail ? min(ja + 1, n - 1) : ja + 1);
        if constexpr (NARROW) {
          const unsigned off =
              (unsigned)(slot ? cb * (int)row_bytes : ca * (int)row_bytes) + lane_off;
          load_row<V>(reinterpret_cast<const float*>(xb + off), xv[u]);
        } else {
          const int64_t off = (int64_t)(slot ? cb : ca) * row_bytes + lane_off;
          load_row<V>(reinterpret_cast<const float*>(xb + off), xv[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ja = j0 + u * SL;
        if (tail && ja >= n) continue;  // uniform
        const int wa = __builtin_amdgcn_readlane(wj, ja);
        const int wb = __builtin_amdgcn_readlane(wj, tail ? min(ja + 1, n - 1) : ja + 1);
        const float wt = __int_as_float(slot ? wb : wa);
        if (!tail || ja + slot < n)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[u][v] = __builtin_fmaf(wt, xv[u][v], acc[u][v]);
      }
    };
    int j0 = 0;
    for (; j0 + U * SL <= n; j0 += U * SL) group(j0, false);
    if (j0 < n) group(j0, true);
  }
#pragma unroll
  for (int step = 1; step < U; step <<= 1)
#pragma unroll
    for (int u = 0; u + step < U; u += 2 * step)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[u][v] += acc[u + step][v];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[0][v] += __shfl_xor(acc[0][v], LPS);
  if (slot != 0) return;
  // partial rows are read back once, by the fix-up, long after: streamed
  // past the L2, which they would otherwise share with the gathered rows
  store_row<V>(part + (int64_t)pslot * F + f, acc[0]);
}

// Whether a sum or mean over the part plan goes through spmm_wide: rows of 128
// columns, which its two slots of 32 lanes of four columns fill. There it beats a
// segment per slot (3.49 against 3.67 ms on 114.6M edges; both slots on one segment
// keep fewer segments in flight, and the gathered window stays closer to the L2s);
// narrower rows leave lanes idle and wider ones take passes, and the slots are as
// fast or faster there (256 columns 2.39 against 2.41 ms on 23M edges, 200 columns
// 1.95 against 2.31), as on the row plan. TFG_WIDE_ROWS=0 keeps every aggregation on
// the slots.
constexpr int kWideColumns = 128;
bool use_wide(int64_t F, bool plain_sum, bool part_plan) {
  if (!plain_sum || !part_plan || F != kWideColumns) return false;
  if (const char* v = std::getenv("TFG_WIDE_ROWS"))
    if (v[0] == '0') return false;
  return true;
}

void launch_wide(int n_items, hipStream_t s, const RowArgs& a, int64_t n_src) {
  // the whole table within 32-bit byte offsets of its base
  const bool narrow = (double)n_src * (double)a.ldx * 4.0 < 2147483648.0;
  const dim3 grid((unsigned)n_items);
#define TFG_WIDE(NN)                                                                          \
  spmm_wide<NN><<<grid, dim3(kRowBlock), 0, s>>>(a.heavy, n_items, a.col, a.perm, a.w,        \
                                                 a.w_by_perm, a.x, a.ldx, a.F, a.part)
  if (narrow) TFG_WIDE(true); else TFG_WIDE(false);
#undef TFG_WIDE
}

// The slot aggregation (slots.h) over the plan's items: V columns per lane,
// the fewest lanes per slot (a power of two, at least 4) that hold a row, and
// per list the number of neighbouring slots that share an item.
//
// Row plan, items of over 32 edges: at least max(4, 32 / lanes) slots. The ids
// and weights of an item are then read in longer runs: with one item per slot,
// the id streams of a wavefront's 64 / lanes items fall out of the L1 between
// rounds (16 columns on 23M edges, 4 lanes: 0.36 ms with one slot per item,
// 0.29 / 0.26 / 0.24 with two, four, eight). 9..32 edges: two (16 columns on
// 2.3M edges of rows of 14: 41.7 -> 38.6 us), one with per-head weights (64
// columns: 102 -> 96 us). Part plan: one (segments of 16 edges, 64 columns: 0.50
// ms, two slots 0.55). Beyond that, while the items leave part of the chip idle,
// an item takes more slots until each has one round of edges.
constexpr int kIdRound = 16;      // edges a slot takes per round of ids
constexpr int kChipWaves = 8192;  // wavefronts in flight: 256 CUs x 4 SIMDs x 8
}  // namespace

namespace rows {
void slot_lists(const Graph& g, const WorkItem* pieces, int n_pieces, bool part_plan, int lps,
                bool heads, SlotLists& L, int* waves) {
  const int slots = kWave / lps;
  // edges: of the list's longest item; least, total: see above (total items)
  auto add = [&](int i, const WorkItem* items, int n, int edges, int least, int total) {
    L.items[i] = items;
    L.n[i] = n;
    int sp = 1;
    while (sp < slots && sp * kIdRound < edges &&
           (sp < least || (int64_t)total * sp < (int64_t)kChipWaves * slots))
      sp <<= 1;
    L.split[i] = sp;
    L.waves[i] = (int)(((int64_t)n * sp + slots - 1) / slots);
  };
  if (part_plan) {
    add(0, pieces, n_pieces, g.chunk, 1, n_pieces);
  } else {
    const int total = n_pieces + g.n_long + g.n_short, least = std::max(4, 32 / lps);
    add(0, pieces, n_pieces, g.chunk, least, total);
    add(1, g.long_rows, g.n_over32, g.chunk, least, total);
    add(2, g.long_rows + g.n_over32, g.n_long - g.n_over32, 32, heads ? 1 : 2, total);
    add(3, g.short_rows, g.n_short, kShortRow, 1, total);
  }
  *waves = 0;
  for (int i = 0; i < kSlotLists; ++i) *waves += L.waves[i];
}
}  // namespace rows

namespace {
void launch_slots(const Graph& g, const RowArgs& a, bool mx, bool heads, bool masked,
                  bool part_plan, hipStream_t s) {
  // (heads of columns that are no multiple of 4: a lane's columns stay in one head)
  int v = a.F >= 4 ? 4 : 1;
  if (heads && a.per_head % 4 != 0) v = a.per_head % 2 == 0 && !mx && !masked ? 2 : 1;
  SlotLists L{};
  const int need = std::min((a.F + v - 1) / v, kWave);
  int lps = 4, waves;
  while (lps < need) lps <<= 1;
  slot_lists(g, a.heavy, a.n_heavy, part_plan, lps, heads, L, &waves);
  if (waves == 0) return;
  // byte offsets in 32 bits: rows of x, and per-head weights (past the last item's
  // end by up to a round: a margin of 2^20 rows)
  const bool narrow = (double)g.N_src * (double)a.ldx * 4.0 < 2147483648.0 &&
                      (!heads || ((double)g.E + 1048576.0) * (double)a.H * 4.0 < 4294967296.0);
  if (masked) slots_masked(v, lps, narrow, L, waves, a, s);
  else if (heads) slots_heads(mx, v, lps, narrow, L, waves, a, s);
  else if (mx) slots_max(!part_plan && g.parts > 1, v, lps, narrow, L, waves, a, s);
  else slots_sum(v, lps, narrow, L, waves, a, s);
}

}  // namespace

int noalloc_scratch(void** ptr) {
  int dev = 0;
  TFG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(TFG_ERR_INVALID_ARG, "device id out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_addr[dev] == nullptr) {
    void* p = nullptr;
    TFG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return fail(TFG_ERR_HIP, "no device address for the static scratch");
    g_scratch_addr[dev] = p;
  }
  *ptr = g_scratch_addr[dev];
  return TFG_OK;
}

size_t aggregate_partial_bytes(int64_t n_partials, int64_t F, int reduce) {
  size_t per = sizeof(float) + (reduce == TFG_MAX ? sizeof(int) : 0);
  return align_up((size_t)std::max<int64_t>(n_partials, 1) * (size_t)F * per + 256, 256);
}

bool use_part_plan(const Graph& g, int64_t F) {
  if (g.parts <= 1 || g.n_pexec == 0) return false;
  const char* v = std::getenv("TFG_PART_PLAN");  // "0": never, "1": always, unset: by size
  if (v && v[0] == '0') return false;
  if (v && v[0] == '1') return true;
  // the gathered table must be much larger than the L2 caches (8 x 4 MB)
  return (double)g.N_src * (double)F * 4.0 >= 32.0 * (1 << 20);
}

int launch_aggregate(const Graph& g, const float* w, int H, int w_order, const float* x,
                     int64_t F, int64_t ldx, int reduce, float* out, int32_t* argmax, void* ws,
                     hipStream_t s, float scale, float alpha, const float* h, int64_t ldh,
                     const int32_t* mask) {
  if (g.N == 0 || F == 0) return TFG_OK;
  if (mask != nullptr && reduce != TFG_SUM) return fail(TFG_ERR_INVALID_ARG, "masked max");
  if (mask != nullptr && ldx != F) return fail(TFG_ERR_INVALID_ARG, "masked rows must be dense");
  const bool heads = H > 1 && w != nullptr;
  const bool mx = reduce == TFG_MAX;
  const bool part_plan = use_part_plan(g, F);

  RowArgs a;
  a.col = g.col;
  a.perm = g.perm;
  a.w = w;
  a.w_by_perm = (w != nullptr && w_order == TFG_COO) ? 1 : 0;
  a.H = H;
  a.per_head = (int)(F / H);
  a.x = x;
  a.ldx = ldx;
  a.mask = mask;
  a.F = (int)F;
  a.mean = reduce == TFG_MEAN;
  a.out = out;
  a.argout = argmax;
  a.ep = Epilogue{scale, alpha, h, ldh};
  const int n_partials = part_plan ? g.n_pexec : g.n_heavy;
  a.part = static_cast<float*>(ws);
  a.part_arg = reinterpret_cast<int*>(a.part + (size_t)std::max(n_partials, 1) * F);
  // part plan: every (part, row) item writes a partial, each row is reduced in
  // part order; row plan: whole rows write the output, chunks partials
  a.heavy = part_plan ? g.pexec : g.heavy;
  a.n_heavy = n_partials;
  const SplitRow* rows = part_plan ? g.prows : g.split;
  const int n_rows = part_plan ? (int)g.N : g.n_split;
  if (use_wide(F, !mx && !heads && mask == nullptr, part_plan) && a.n_heavy > 0)
    launch_wide(a.n_heavy, s, a, g.N_src);
  else
    launch_slots(g, a, mx, heads, mask != nullptr, part_plan, s);
  TFG_LAUNCHED("aggregation");
  if (n_rows > 0) {
    int flps = 4;  // lanes per slot
    while (flps < kWave && flps * (F >= 4 ? 4 : 1) < F) flps <<= 1;
    // slots per row: one by source part (a row has at most a few partials per part);
    // split rows the average number of partials a row, at least four
    int share = 1;
    if (!part_plan)
      while (share < kWave / flps && (share < 4 || (int64_t)share * n_rows < n_partials)) share <<= 1;
    const int64_t lanes = (int64_t)n_rows * flps * share;
    dim3 fgrid((unsigned)((lanes + kWave - 1) / kWave));
#define TFG_FIXUP(M, VV)                                                                      \
  fixup_rows<M, VV><<<fgrid, dim3(kItemBlock), 0, s>>>(rows, n_rows, a.part, a.part_arg, a.F, \
                                                       a.mean, out, argmax, a.ep, flps, share)
    if (mx && F >= 4) TFG_FIXUP(true, 4);
    else if (mx) TFG_FIXUP(true, 1);
    else if (F >= 4) TFG_FIXUP(false, 4);
    else TFG_FIXUP(false, 1);
#undef TFG_FIXUP
    TFG_LAUNCHED("fixup_rows");
  }
  return TFG_OK;
}

}  // namespace tfg
