// The paper's precision (Section 5.1.2): float32 edge weights with FP64
// hashtable values, weighted degrees K, community totals Sigma, 2m and
// modularity.  The steps are those of the integer path (batch edit, Alg. 7,
// Alg. 1, Alg. 4-6) with Eq. 2 evaluated as printed in FP64:
//     ΔQ(i: d -> c) = (K_{i->c} - K_{i->d}) / m - K_i (K_i + Σ_c - Σ_d) / (2 m^2)
// in ASYNC mode (a move's membership and totals are visible at once to
// later readers; the iteration runs the integer path's sub-rounds).
//
// Work mapping (wave64): rows up to 256 arcs take one wavefront with an LDS
// table of 512 (community, FP64 weight) slots; rows up to 2048 arcs one
// workgroup with a 4096-slot LDS table; longer rows one wide workgroup with
// an 8192-slot LDS table, or one of 2 x deg slots in the workspace pool where
// a row's communities exceed that.  The frontier is a bitmask; movers push
// their neighbours.  Aggregation gives each community one workgroup, whose
// table (LDS, or pool slots for a large community of a level of many) sums
// the members' arcs by neighbouring community in FP64; the
// sums are stored as float32 weights of a slack CSR whose row capacities
// are the member volumes.
#include <cfloat>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>

#include "lv_internal.hpp"

namespace lv {
namespace {

constexpr int kFWaveMax = 256;
constexpr int kFWaveSlots = 2 * kFWaveMax;
constexpr int kFBlockMax = 2048;
constexpr int kFBlockSlots = 2 * kFBlockMax;
constexpr int kFNW = kBlock / kWave;
enum FBin { FB_WAVE = 0, FB_BLOCK, FB_HUB, FB_N };

// Counter block (int64 slots, one 128-byte line each where contended):
// errors, list counts, pool reservations, the batch edit's statistics, and
// kFReps replicas of the per-iteration statistics.
constexpr int kFReps = 32;
enum FCtr {
  F_ERR = 0,
  F_LIST0 = 1 * kCtrLine,   // three lines: items per bin
  F_POOL = 4 * kCtrLine,    // pool slots handed out in this round
  F_AUX = 5 * kCtrLine,     // scratch count (compaction rows)
  F_BSUM = 6 * kCtrLine,    // batch: FP64 Σ w_ins (slot 0), Σ w_del (slot 1) as doubles
  F_STATS = 8 * kCtrLine,   // kFReps replicas of a line: the statistics below
  F_COUNT = F_STATS + kFReps * kCtrLine
};
enum FStat { FS_MOVERS = 0, FS_ARCS, FS_PROCESSED, FS_EXPAND, FS_AFFECTED, FS_DQ /* double */, FS_SUM /* double */,
             FS_SUM2 /* double */ };

__device__ __forceinline__ int64_t* rep(int64_t* ctr) { return ctr + F_STATS + (blockIdx.x % kFReps) * kCtrLine; }
__device__ __forceinline__ void stat_i(int64_t* ctr, int k, int64_t v) {
  if (v) atomicAdd(reinterpret_cast<unsigned long long*>(rep(ctr) + k), static_cast<unsigned long long>(v));
}
__device__ __forceinline__ void stat_d(int64_t* ctr, int k, double v) {
  if (v != 0.0) atomicAdd(reinterpret_cast<double*>(rep(ctr) + k), v);
}
__device__ __forceinline__ void flag(int64_t* ctr, int64_t code) {
  atomicCAS(reinterpret_cast<unsigned long long*>(&ctr[F_ERR]), 0ull, static_cast<unsigned long long>(code));
}
template <class T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double wave_sum_d(double v) {
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  return v;
}
__device__ __forceinline__ bool better_f(double g1, int32_t c1, double g0, int32_t c0) {
  return g1 > g0 || (g1 == g0 && c1 < c0);
}
template <int S = 1>
__device__ __forceinline__ void wave_arg(double& g, int32_t& c) {
  if constexpr (S < kWave) {
    const double og = other_half<S>(g);
    const int32_t oc = other_half<S>(c);
    if (better_f(og, oc, g, c)) {
      g = og;
      c = oc;
    }
    wave_arg<2 * S>(g, c);
  }
}
__device__ __forceinline__ bool weight_ok(float w) { return isfinite(w) && w > 0.0f; }

struct FG {  // a level graph
  int32_t n;
  const int64_t* row_start;
  const int32_t* row_len;
  const int32_t* col;
  const float* w;
};

// ---------------------------------------------------------------------------
// Call start, row sums, totals
// ---------------------------------------------------------------------------
__global__ void k_f_begin(int64_t* __restrict__ ctr, uint32_t* __restrict__ a, uint32_t* __restrict__ b,
                          uint32_t* __restrict__ ever, int64_t words, const double* __restrict__ two_m) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t t0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  for (int64_t k = t0; k < words; k += stride) {
    a[k] = 0;
    b[k] = 0;
    ever[k] = 0;
  }
  for (int64_t k = t0; k < F_COUNT; k += stride) {
    int64_t v = 0;
    if (k == F_ERR) v = (*two_m > 0.0 && isfinite(*two_m)) ? 0 : LV_EEMPTY;
    ctr[k] = v;
  }
}

// K_i = FP64 row sum (Sigma = K, C = identity, size = 1 when given); the
// total (2m) and, with C, the weight of arcs inside communities go to the
// statistics replicas.  One wavefront per row.
__global__ void __launch_bounds__(kBlock) k_f_rows(FG g, const int32_t* __restrict__ C, double* __restrict__ K,
                                                 double* __restrict__ Sigma, int32_t* __restrict__ Cinit,
                                                 int32_t* __restrict__ size, int64_t* __restrict__ ctr) {
  const int lane = lane_id();
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kFNW;
  double tot = 0.0, intra = 0.0;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kFNW) + threadIdx.x / kWave; i < g.n; i += nw) {
    const int64_t s = g.row_start[i];
    const int32_t len = g.row_len[i];
    const int32_t ci = C ? C[i] : 0;
    double acc = 0.0, in = 0.0;
    for (int32_t k = lane; k < len; k += kWave) {
      const double x = static_cast<double>(g.w[s + k]);
      acc += x;
      if (C && C[g.col[s + k]] == ci) in += x;
    }
    acc = wave_sum_d(acc);
    in = wave_sum_d(in);
    if (lane == 0) {
      if (K) K[i] = acc;
      if (Sigma) Sigma[i] = acc;
      if (Cinit) Cinit[i] = static_cast<int32_t>(i);
      if (size) size[i] = 1;
      tot += acc;
      intra += in;
    }
  }
  if (lane == 0) {
    stat_d(ctr, FS_SUM, tot);
    stat_d(ctr, FS_SUM2, intra);
  }
}

// tot[C_i] += K_i (community totals), FP64 atomics
__global__ void k_f_totals(const int32_t* __restrict__ C, const double* __restrict__ K, int32_t n,
                           double* __restrict__ tot, int64_t* __restrict__ ctr) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t c = C[i];
    if (c < 0 || c >= n)
      flag(ctr, LV_EINVAL);
    else if (K[i] != 0.0)
      atomicAdd(&tot[c], K[i]);
  }
}

// every membership lies in [0, n)
constexpr int64_t kBadMember = -1000;  // (reported as LV_EINVAL, with a message of its own)
__global__ void k_f_check_c(const int32_t* __restrict__ C, int32_t n, int64_t* __restrict__ ctr) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    if (C[i] < 0 || C[i] >= n) flag(ctr, kBadMember);
}

// Σ_c tot_c^2 into the statistics (slot FS_SUM)
__global__ void k_f_sumsq(const double* __restrict__ tot, int32_t n, int64_t* __restrict__ ctr) {
  double s = 0.0;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    s += tot[i] * tot[i];
  s = wave_sum_d(s);
  if (lane_id() == 0) stat_d(ctr, FS_SUM, s);
}

__global__ void k_f_zero_d(double* __restrict__ p, int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// Graph build
// ---------------------------------------------------------------------------
__global__ void k_f_count(const int32_t* __restrict__ u, const int32_t* __restrict__ v, const float* __restrict__ w,
                          int64_t m, int32_t n, int32_t* __restrict__ deg, int64_t* __restrict__ ctr) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < m;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t a = u[k], b = v[k];
    if (a < 0 || b < 0 || a >= n || b >= n || a == b || !weight_ok(w[k])) {
      flag(ctr, LV_EINVAL);
      continue;
    }
    atomicAdd(&deg[a], 1);
    atomicAdd(&deg[b], 1);
  }
}

__global__ void k_f_scatter(const int32_t* __restrict__ u, const int32_t* __restrict__ v,
                            const float* __restrict__ w, int64_t m, const int64_t* __restrict__ row_start,
                            int32_t* __restrict__ row_len, int32_t* __restrict__ col, float* __restrict__ wt) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < m;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t a = u[k], b = v[k];
    const int64_t pa = row_start[a] + atomicAdd(&row_len[a], 1);
    const int64_t pb = row_start[b] + atomicAdd(&row_len[b], 1);
    col[pa] = b;
    wt[pa] = w[k];
    col[pb] = a;
    wt[pb] = w[k];
  }
}

__global__ void k_f_set_two_m(double* __restrict__ two_m, const int64_t* __restrict__ ctr, int add) {
  double s = 0.0;
  for (int r = 0; r < kFReps; ++r) s += reinterpret_cast<const double*>(ctr + F_STATS + r * kCtrLine)[FS_SUM];
  if (add) {  // batch: 2 (Σ w_ins - Σ w_del)
    const double* b = reinterpret_cast<const double*>(ctr + F_BSUM);
    *two_m += 2.0 * (b[0] - b[1]);
  } else {
    *two_m = s;
  }
}

// ---------------------------------------------------------------------------
// Batch edit (Section 3.4), all-or-nothing.  A table of the batch's pairs
// (tagged deletion / insertion) finds repeats; a table of touched rows
// counts the arcs each row gains and loses, for the capacity check.
// ---------------------------------------------------------------------------
struct FBatch {
  const int32_t *du, *dv;
  const float* dw;
  int64_t nd;
  const int32_t *iu, *iv;
  const float* iw;
  int64_t ni;
};
struct FBTab {
  unsigned long long* pkey;  // pair tables: (canonical pair << 1 | is_insertion) + 1, 0 = empty
  int32_t* pzero;            // deletions: 1 when the arc's whole weight goes
  int64_t psize;             // power of two
  int32_t* rkey;             // row table: row + 1, 0 = empty
  int32_t* rapp;             // arcs appended to the row
  int32_t* rzero;            // arcs removed from the row
  int64_t rsize;
  int32_t* dpos;             // per deletion: arc offsets in row u and row v
  int32_t* imode;            // per insertion: 1 merge, 0 append
};

__device__ __forceinline__ unsigned long long pair_tag(int32_t a, int32_t b, int ins) {
  const unsigned long long lo = static_cast<uint32_t>(min(a, b)), hi = static_cast<uint32_t>(max(a, b));
  return (((lo << 32) | hi) << 1 | static_cast<unsigned long long>(ins)) + 1ull;
}
__device__ __forceinline__ uint32_t mixh(unsigned long long k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  return static_cast<uint32_t>(k);
}
// find-or-insert; returns (slot, inserted now)
__device__ __forceinline__ int64_t pair_slot(const FBTab& t, unsigned long long key, bool* fresh) {
  int64_t h = mixh(key) & (t.psize - 1);
  for (int64_t p = 0; p < t.psize; ++p) {
    const unsigned long long old = atomicCAS(&t.pkey[h], 0ull, key);
    if (old == 0ull || old == key) {
      *fresh = old == 0ull;
      return h;
    }
    h = (h + 1) & (t.psize - 1);
  }
  return -1;
}
__device__ __forceinline__ int64_t pair_find(const FBTab& t, unsigned long long key) {
  int64_t h = mixh(key) & (t.psize - 1);
  for (int64_t p = 0; p < t.psize; ++p) {
    const unsigned long long k = ld_agent(&t.pkey[h]);
    if (k == key) return h;
    if (k == 0ull) return -1;
    h = (h + 1) & (t.psize - 1);
  }
  return -1;
}
__device__ __forceinline__ int64_t row_slot(const FBTab& t, int32_t r) {
  int64_t h = mixh(static_cast<unsigned long long>(r) + 0x9E3779B97F4A7C15ull) & (t.rsize - 1);
  for (int64_t p = 0; p < t.rsize; ++p) {
    const int32_t old = atomicCAS(&t.rkey[h], 0, r + 1);
    if (old == 0 || old == r + 1) return h;
    h = (h + 1) & (t.rsize - 1);
  }
  return -1;
}
__device__ __forceinline__ int32_t find_arc(const int32_t* col, int64_t s, int32_t len, int32_t j) {
  for (int32_t k = 0; k < len; ++k)
    if (col[s + k] == j) return k;
  return -1;
}

// V1: deletions -- ids, weights, repeats, presence and weight; records the
// arc offsets and whether the whole weight goes (the row then loses it).
__global__ void k_f_val_del(FBatch b, lv_graph_f g, FBTab t, int64_t* __restrict__ ctr) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < b.nd;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t u = b.du[k], v = b.dv[k];
    const float x = b.dw[k];
    if (u < 0 || v < 0 || u >= g.n || v >= g.n || u == v || !weight_ok(x)) {
      flag(ctr, LV_EINVAL);
      continue;
    }
    bool fresh = false;
    const int64_t h = pair_slot(t, pair_tag(u, v, 0), &fresh);
    if (h < 0 || !fresh) {
      flag(ctr, h < 0 ? LV_EWORKSPACE : LV_EINVAL);
      continue;
    }
    const int32_t pu = find_arc(g.col, g.row_start[u], g.row_len[u], v);
    const int32_t pv = find_arc(g.col, g.row_start[v], g.row_len[v], u);
    if (pu < 0 || pv < 0 || g.w[g.row_start[u] + pu] < x) {
      flag(ctr, LV_ENOEDGE);
      continue;
    }
    t.dpos[2 * k] = pu;
    t.dpos[2 * k + 1] = pv;
    const bool whole = g.w[g.row_start[u] + pu] - x <= 0.0f;
    t.pzero[h] = whole ? 1 : 0;
    if (whole) {
      const int64_t ru = row_slot(t, u), rv = row_slot(t, v);
      if (ru < 0 || rv < 0) {
        flag(ctr, LV_EWORKSPACE);
        continue;
      }
      atomicAdd(&t.rzero[ru], 1);
      atomicAdd(&t.rzero[rv], 1);
    }
    atomicAdd(reinterpret_cast<double*>(ctr + F_BSUM) + 1, static_cast<double>(x));
  }
}

// V2: insertions -- ids, weights, repeats; merge into a present arc that
// the batch's deletions leave, else append (the rows gain an arc).
__global__ void k_f_val_ins(FBatch b, lv_graph_f g, FBTab t, int64_t* __restrict__ ctr) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < b.ni;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t u = b.iu[k], v = b.iv[k];
    const float x = b.iw[k];
    if (u < 0 || v < 0 || u >= g.n || v >= g.n || u == v || !weight_ok(x)) {
      flag(ctr, LV_EINVAL);
      continue;
    }
    bool fresh = false;
    const int64_t h = pair_slot(t, pair_tag(u, v, 1), &fresh);
    if (h < 0 || !fresh) {
      flag(ctr, h < 0 ? LV_EWORKSPACE : LV_EINVAL);
      continue;
    }
    bool merge = find_arc(g.col, g.row_start[u], g.row_len[u], v) >= 0;
    if (merge) {
      const int64_t hd = pair_find(t, pair_tag(u, v, 0));
      if (hd >= 0 && ld_agent(&t.pzero[hd])) merge = false;  // deleted whole first
    }
    t.imode[k] = merge ? 1 : 0;
    if (!merge) {
      const int64_t ru = row_slot(t, u), rv = row_slot(t, v);
      if (ru < 0 || rv < 0) {
        flag(ctr, LV_EWORKSPACE);
        continue;
      }
      atomicAdd(&t.rapp[ru], 1);
      atomicAdd(&t.rapp[rv], 1);
    }
    atomicAdd(reinterpret_cast<double*>(ctr + F_BSUM), static_cast<double>(x));
  }
}

// V3: every touched row fits its capacity after the batch
__global__ void k_f_val_cap(lv_graph_f g, FBTab t, int64_t* __restrict__ ctr) {
  for (int64_t h = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; h < t.rsize;
       h += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t key = t.rkey[h];
    if (!key) continue;
    const int32_t r = key - 1;
    const int64_t cap = g.row_start[r + 1] - g.row_start[r];
    if (static_cast<int64_t>(g.row_len[r]) - t.rzero[h] + t.rapp[h] > cap) flag(ctr, LV_ENOSLACK);
  }
}

// A1: deletions subtract their weight from both arcs
__global__ void k_f_del(FBatch b, lv_graph_f g, FBTab t, const int64_t* __restrict__ ctr) {
  if (ctr[F_ERR]) return;
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < b.nd;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    g.w[g.row_start[b.du[k]] + t.dpos[2 * k]] -= b.dw[k];
    g.w[g.row_start[b.dv[k]] + t.dpos[2 * k + 1]] -= b.dw[k];
  }
}

// A2: rows that lost arcs drop the ones of weight 0 (one lane per row)
__global__ void k_f_compact(lv_graph_f g, FBTab t, const int64_t* __restrict__ ctr) {
  if (ctr[F_ERR]) return;
  for (int64_t h = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; h < t.rsize;
       h += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t key = t.rkey[h];
    if (!key || t.rzero[h] == 0) continue;
    const int32_t r = key - 1;
    const int64_t s = g.row_start[r];
    const int32_t len = g.row_len[r];
    int32_t o = 0;
    for (int32_t q = 0; q < len; ++q) {
      const float x = g.w[s + q];
      if (x > 0.0f) {
        g.col[s + o] = g.col[s + q];
        g.w[s + o] = x;
        ++o;
      }
    }
    g.row_len[r] = o;
  }
}

// A3: insertions merge or append, in both directions
__global__ void k_f_ins(FBatch b, lv_graph_f g, FBTab t, const int64_t* __restrict__ ctr) {
  if (ctr[F_ERR]) return;
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < b.ni;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int32_t e[2][2] = {{b.iu[k], b.iv[k]}, {b.iv[k], b.iu[k]}};
    for (int q = 0; q < 2; ++q) {
      const int32_t a = e[q][0], c = e[q][1];
      const int64_t s = g.row_start[a];
      if (t.imode[k]) {
        const int32_t p = find_arc(g.col, s, g.row_len[a], c);
        if (p >= 0) atomicAdd(&g.w[s + p], b.iw[k]);
      } else {
        const int64_t p = s + atomicAdd(&g.row_len[a], 1);
        g.col[p] = c;
        g.w[p] = b.iw[k];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// updateWeights (Alg. 7) in FP64 and DF marking (Alg. 1)
// ---------------------------------------------------------------------------
__global__ void k_f_update(FBatch b, int32_t n, const int32_t* __restrict__ C, double* __restrict__ K,
                           double* __restrict__ Sigma, uint32_t* __restrict__ fr, int64_t* __restrict__ ctr) {
  if (ctr[F_ERR]) return;
  const int64_t total = b.nd + b.ni;
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < total;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const bool del = k < b.nd;
    const int32_t u = del ? b.du[k] : b.iu[k - b.nd];
    const int32_t v = del ? b.dv[k] : b.iv[k - b.nd];
    if (u < 0 || v < 0 || u >= n || v >= n || u == v) {  // not the batch apply_batch_f took
      flag(ctr, LV_EINVAL);
      continue;
    }
    const double x = del ? -static_cast<double>(b.dw[k]) : static_cast<double>(b.iw[k - b.nd]);
    const int32_t cu = C[u], cv = C[v];
    atomicAdd(&K[u], x);
    atomicAdd(&K[v], x);
    atomicAdd(&Sigma[cu], x);
    atomicAdd(&Sigma[cv], x);
    if (fr && (cu == cv) == del) {
      set_bit(fr, u);
      set_bit(fr, v);
    }
  }
}

// ---------------------------------------------------------------------------
// Local moving (Alg. 5), ASYNC
// ---------------------------------------------------------------------------
struct FMove {
  FG g;
  int32_t* C;
  const double* K;
  double* Sigma;
  int32_t* size;
  uint32_t* next;
  const int32_t* list[FB_N];
  int64_t cnt[FB_N];  // rows per bin (-1: in the counter block)
  const double* two_m;
  int32_t guard;
  int64_t* ctr;
  int64_t pool_slots;
  int32_t* pkeys;
  double* pvals;
};

__device__ __forceinline__ int64_t rows_in(const FMove& M, int b) {
  return M.cnt[b] >= 0 ? M.cnt[b] : M.ctr[F_LIST0 + b * kCtrLine];
}

__device__ __forceinline__ double dq_of(double m, double kic, double kid, double Ki, double Sc, double Sd) {
  return (kic - kid) / m - Ki * (Ki + Sc - Sd) / (2.0 * m * m);
}

// the move of vertex i (one thread): returns whether it moved
__device__ __forceinline__ bool commit(const FMove& M, int32_t i, int32_t d, int32_t c, double dq, double Ki) {
  if (c == INT_MAX || !(dq > 0.0)) return false;
  if (M.guard && M.size[d] == 1 && M.size[c] == 1 && c > d) return false;
  M.C[i] = c;
  atomicAdd(&M.Sigma[d], -Ki);
  atomicAdd(&M.Sigma[c], Ki);
  atomicSub(&M.size[d], 1);
  atomicAdd(&M.size[c], 1);
  return true;
}

// Table insert: (c, x) into keys/vals of `size` slots (power of two); returns
// whether c was new.
__device__ __forceinline__ bool tab_add(int32_t* keys, double* vals, uint32_t size, int32_t c, double x) {
  uint32_t h = hash_slot(static_cast<uint32_t>(c), size);
  while (true) {
    const int32_t old = atomicCAS(&keys[h], -1, c);
    if (old == -1 || old == c) {
      atomicAdd(&vals[h], x);
      return old == -1;
    }
    h = (h + 1) & (size - 1);
  }
}

// Every scan does nothing once the error slot is set (a membership outside
// [0, n), or a batch that names a vertex outside it).
__global__ void __launch_bounds__(kBlock) k_f_scan_wave(FMove M) {
  __shared__ int32_t s_keys[kFNW][kFWaveSlots];
  __shared__ double s_vals[kFNW][kFWaveSlots];
  constexpr int U = kFWaveMax / kWave;
  if (M.ctr[F_ERR]) return;
  const double m = *M.two_m / 2.0;
  const int lane = lane_id();
  const int wv = threadIdx.x / kWave;
  int32_t* keys = s_keys[wv];
  double* vals = s_vals[wv];
  const int64_t count = rows_in(M, FB_WAVE);
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kFNW;
  int64_t movers = 0, expand = 0;
  double dq_sum = 0.0;
  // (a lane owns the slots it inserts: it reads their sums and clears them)
  for (int t = lane; t < kFWaveSlots; t += kWave) {
    keys[t] = -1;
    vals[t] = 0.0;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int64_t idx = blockIdx.x * static_cast<int64_t>(kFNW) + wv; idx < count; idx += nw) {
    const int32_t i = M.list[FB_WAVE][idx];
    const int64_t s = M.g.row_start[i];
    const int32_t deg = M.g.row_len[i];
    const int32_t d = M.C[i];
    const double Ki = M.K[i];
    const uint32_t ts = max(64u, 1u << (32 - __clz(static_cast<uint32_t>(2 * max(deg, 1) - 1))));
    const int nu = __builtin_amdgcn_readfirstlane((deg + kWave - 1) / kWave);  // steps that hold arcs
    int32_t js[U], cs[U], own[U];
    float xs[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (q >= nu) continue;
      const int32_t k = lane + q * kWave;
      js[q] = k < deg ? M.g.col[s + k] : i;
      xs[q] = k < deg ? M.g.w[s + k] : 0.0f;
    }
    const double Sd = M.Sigma[d];
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (q < nu) cs[q] = js[q] != i ? M.C[js[q]] : d;
    double kid = 0.0;
#pragma unroll
    for (int q = 0; q < U; ++q) {
      own[q] = -1;
      if (q >= nu || js[q] == i) continue;
      const double x = static_cast<double>(xs[q]);
      if (cs[q] == d) {
        kid += x;
        continue;
      }
      uint32_t h = hash_slot(static_cast<uint32_t>(cs[q]), ts);
      while (true) {
        const int32_t old = atomicCAS(&keys[h], -1, cs[q]);
        if (old == -1 || old == cs[q]) {
          atomicAdd(&vals[h], x);
          if (old == -1) own[q] = static_cast<int32_t>(h);
          break;
        }
        h = (h + 1) & (ts - 1);
      }
    }
    kid = wave_sum_d(kid);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double bg = -DBL_MAX;
    int32_t bc = INT_MAX;
    double vv[U], sg[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (q >= nu) continue;
      vv[q] = own[q] >= 0 ? vals[own[q]] : 0.0;
      sg[q] = own[q] >= 0 ? M.Sigma[cs[q]] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (q >= nu || own[q] < 0) continue;
      keys[own[q]] = -1;
      vals[own[q]] = 0.0;
      const double g = dq_of(m, vv[q], kid, Ki, sg[q], Sd);
      if (better_f(g, cs[q], bg, bc)) {
        bg = g;
        bc = cs[q];
      }
    }
    wave_arg(bg, bc);
    bool mv = false;
    if (lane == 0) mv = commit(M, i, d, bc, bg, Ki);
    mv = __shfl(mv ? 1 : 0, 0) != 0;
    if (mv) {
      if (lane == 0) {
        movers += 1;
        expand += deg;
        dq_sum += bg;
      }
      for (int32_t k = lane; k < deg; k += kWave) {
        const int32_t j = M.g.col[s + k];
        if (j != i) set_bit(M.next, j);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (lane == 0) {
    stat_i(M.ctr, FS_MOVERS, movers);
    stat_i(M.ctr, FS_EXPAND, expand);
    stat_d(M.ctr, FS_DQ, dq_sum);
  }
}

// Rows past the wavefront bin: one workgroup each.  Up to 2048 arcs 256
// threads and a 4096-slot LDS table.  Longer (hub) rows 1024 threads and 8192
// slots, which hold the neighbour communities of any row that does not have
// over 6144 of them; one that does takes 2 x deg pool slots.
// (256 threads with the pool's table for every hub row: 51 us a launch over a
// few rows of up to 5000 arcs of a 250,001-vertex power-law graph, a chain of
// 20 arcs per thread and every insert an L2 atomic; this: 12.7 us.)
constexpr int kFWide = 1024;               // threads of the wide workgroups
constexpr int kFWideSlots = 8192;
constexpr int kFWideKeys = kFWideSlots - 2 * kFWide;  // (room for the inserts in flight)

struct FBest {
  double kid, g;
  int32_t c;
};
// The best move of row [s, s + deg) of vertex i (community d) by the
// workgroup's NT threads with the table keys/vals of ts slots.  LIMIT: gives
// up, with *over set, where the row has kFWideKeys communities.
template <int NT, bool GLOBAL, bool LIMIT>
__device__ __forceinline__ FBest group_best(const FMove& M, double m, int32_t i, int64_t s, int32_t deg, int32_t d,
                                            double Ki, int32_t* keys, double* vals, uint32_t ts, int32_t* s_n,
                                            int32_t* over, double* s_g, int32_t* s_c) {
  constexpr int NW = NT / kWave;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t t = threadIdx.x; t < ts; t += NT) {
    keys[t] = -1;
    vals[t] = 0.0;
  }
  if (LIMIT && threadIdx.x == 0) *s_n = *over = 0;
  __syncthreads();
  double kid = 0.0;
  for (int32_t k0 = threadIdx.x; k0 < deg; k0 += 4 * NT) {  // four arcs of a thread in flight
    int32_t js[4], cs[4];
    float xs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool in = k0 + q * NT < deg;
      js[q] = in ? M.g.col[s + k0 + q * NT] : i;
      xs[q] = in ? M.g.w[s + k0 + q * NT] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) cs[q] = js[q] != i ? M.C[js[q]] : d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (js[q] == i) continue;
      const double x = static_cast<double>(xs[q]);
      if (cs[q] == d) {
        kid += x;
        continue;
      }
      if (LIMIT && __hip_atomic_load(s_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= kFWideKeys) {
        *over = 1;
        continue;
      }
      const bool fresh = tab_add(keys, vals, ts, cs[q], x);
      if (LIMIT && fresh) atomicAdd(s_n, 1);
    }
  }
  kid = wave_sum_d(kid);
  if (lane == 0) s_g[wv] = kid;
  __syncthreads();
  FBest r{0.0, -DBL_MAX, INT_MAX};
  if (LIMIT && *over) return r;  // (uniform)
  for (int q = 0; q < NW; ++q) r.kid += s_g[q];
  const double Sd = M.Sigma[d];
  for (uint32_t t = threadIdx.x; t < ts; t += NT) {
    const int32_t c = GLOBAL ? ld_agent(&keys[t]) : keys[t];
    if (c < 0) continue;
    const double x = GLOBAL ? ld_agent(&vals[t]) : vals[t];
    const double g = dq_of(m, x, r.kid, Ki, M.Sigma[c], Sd);
    if (better_f(g, c, r.g, r.c)) {
      r.g = g;
      r.c = c;
    }
  }
  wave_arg(r.g, r.c);
  __syncthreads();
  if (lane == 0) {
    s_g[wv] = r.g;
    s_c[wv] = r.c;
  }
  __syncthreads();
  for (int q = 0; q < NW; ++q)
    if (better_f(s_g[q], s_c[q], r.g, r.c)) {
      r.g = s_g[q];
      r.c = s_c[q];
    }
  return r;
}

template <bool HUB>
__global__ void __launch_bounds__(HUB ? kFWide : kBlock) k_f_scan_group(FMove M) {
  constexpr int NT = HUB ? kFWide : kBlock;
  constexpr int kSlots = HUB ? kFWideSlots : kFBlockSlots;
  __shared__ int32_t s_keys[kSlots];
  __shared__ double s_vals[kSlots];
  __shared__ double s_g[NT / kWave];
  __shared__ int32_t s_c[NT / kWave];
  __shared__ int64_t s_off;
  __shared__ int32_t s_mv, s_n, s_over;
  if (M.ctr[F_ERR]) return;
  const double m = *M.two_m / 2.0;
  const int b = HUB ? FB_HUB : FB_BLOCK;
  const int64_t count = rows_in(M, b);
  int64_t movers = 0, expand = 0;
  double dq_sum = 0.0;
  for (int64_t idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int32_t i = M.list[b][idx];
    const int64_t s = M.g.row_start[i];
    const int32_t deg = M.g.row_len[i];
    const int32_t d = M.C[i];
    const double Ki = M.K[i];
    uint32_t ts = 64u;
    while (ts < static_cast<uint32_t>(kSlots) && ts < 2u * static_cast<uint32_t>(deg)) ts <<= 1;
    FBest r = group_best<NT, false, HUB>(M, m, i, s, deg, d, Ki, s_keys, s_vals, ts, &s_n, &s_over, s_g, s_c);
    if (HUB && s_over) {
      ts = 1u << (32 - __clz(static_cast<uint32_t>(2 * deg - 1)));
      if (threadIdx.x == 0) {
        const int64_t off = static_cast<int64_t>(atomicAdd(reinterpret_cast<unsigned long long*>(&M.ctr[F_POOL]),
                                                           static_cast<unsigned long long>(ts)));
        s_off = off + ts <= M.pool_slots ? off : -1;
        if (s_off < 0) flag(M.ctr, LV_EWORKSPACE);
      }
      __syncthreads();
      if (s_off < 0) return;  // (uniform) the error is flagged
      r = group_best<NT, true, false>(M, m, i, s, deg, d, Ki, M.pkeys + s_off, M.pvals + s_off, ts, nullptr, nullptr,
                                      s_g, s_c);
    }
    if (threadIdx.x == 0) s_mv = commit(M, i, d, r.c, r.g, Ki) ? 1 : 0;
    __syncthreads();
    if (s_mv) {
      if (threadIdx.x == 0) {
        movers += 1;
        expand += deg;
        dq_sum += r.g;
      }
      for (int32_t k = threadIdx.x; k < deg; k += NT) {
        const int32_t j = M.g.col[s + k];
        if (j != i) set_bit(M.next, j);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    stat_i(M.ctr, FS_MOVERS, movers);
    stat_i(M.ctr, FS_EXPAND, expand);
    stat_d(M.ctr, FS_DQ, dq_sum);
  }
}

// Frontier -> three bins (one thread per bitmask word) of an iteration that
// is one sub-round; the words read are cleared.  Workgroup counts per bin, one
// reservation.
__global__ void __launch_bounds__(kBlock) k_f_bin(uint32_t* __restrict__ cur, uint32_t* __restrict__ ever,
                                                const int32_t* __restrict__ row_len, int32_t n, int32_t* l0,
                                                int32_t* l1, int32_t* l2, int64_t* __restrict__ ctr) {
  __shared__ int32_t s_cnt[FB_N];
  __shared__ int64_t s_base[FB_N];
  int32_t* lists[FB_N] = {l0, l1, l2};
  const int64_t words = (static_cast<int64_t>(n) + 31) / 32;
  int64_t arcs = 0, processed = 0, affected = 0;
  for (int64_t w0 = blockIdx.x * static_cast<int64_t>(blockDim.x); w0 < words;
       w0 += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (threadIdx.x < FB_N) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t k = w0 + threadIdx.x;
    uint32_t bits = 0;
    if (k < words) {
      bits = cur[k];
      if (bits) cur[k] = 0;
      if (ever && bits) {
        const uint32_t old = ever[k];
        affected += __popc(bits & ~old);
        ever[k] = old | bits;
      }
    }
    int32_t cnt[FB_N] = {0, 0, 0};
    for (uint32_t r = bits; r; r &= r - 1) {
      const int32_t dg = row_len[k * 32 + (__ffs(r) - 1)];
      processed += 1;
      arcs += dg;
      cnt[dg <= kFWaveMax ? FB_WAVE : dg <= kFBlockMax ? FB_BLOCK : FB_HUB] += 1;
    }
    for (int q = 0; q < FB_N; ++q)
      if (cnt[q]) atomicAdd(&s_cnt[q], cnt[q]);
    __syncthreads();
    if (threadIdx.x < FB_N) {
      const int32_t c = s_cnt[threadIdx.x];
      s_base[threadIdx.x] = c ? static_cast<int64_t>(atomicAdd(
                                    reinterpret_cast<unsigned long long*>(&ctr[F_LIST0 + threadIdx.x * kCtrLine]),
                                    static_cast<unsigned long long>(c)))
                              : 0;
      s_cnt[threadIdx.x] = 0;
    }
    __syncthreads();
    for (uint32_t r = bits; r; r &= r - 1) {
      const int32_t i = static_cast<int32_t>(k * 32 + (__ffs(r) - 1));
      const int32_t dg = row_len[i];
      const int q = dg <= kFWaveMax ? FB_WAVE : dg <= kFBlockMax ? FB_BLOCK : FB_HUB;
      lists[q][s_base[q] + atomicAdd(&s_cnt[q], 1)] = i;
    }
    __syncthreads();
  }
  arcs = wave_sum_i64(arcs);
  processed = wave_sum_i64(processed);
  affected = wave_sum_i64(affected);
  if (lane_id() == 0) {
    stat_i(ctr, FS_ARCS, arcs);
    stat_i(ctr, FS_PROCESSED, processed);
    stat_i(ctr, FS_AFFECTED, affected);
  }
}

// bits [0, n) set, the rest of the `words` words cleared
__global__ void k_f_set_all(uint32_t* __restrict__ bm, int32_t n, int64_t words) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < words;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x)
    bm[k] = (k + 1) * 32 <= n ? 0xFFFFFFFFu : k * 32 >= n ? 0u : ((1u << (n - k * 32)) - 1u);
}

// ---------------------------------------------------------------------------
// Aggregation (Alg. 6)
// ---------------------------------------------------------------------------
// The row of super-vertex c by the workgroup's NT threads: a wavefront takes
// a member at a time, its arcs in lanes, the next member's row looked up
// meanwhile; arcs inside the community (its most frequent key) are summed in
// registers.  keys/vals: ts slots, ts >= 2 x the keys there can be.
template <int NT, bool GLOBAL>
__device__ __forceinline__ void aggregate_one(const FG& g, const int32_t* __restrict__ C,
                                              const int32_t* __restrict__ coff, const int32_t* __restrict__ cmem,
                                              int32_t c, int64_t v0, int32_t* __restrict__ out_len,
                                              int32_t* __restrict__ out_col, float* __restrict__ out_w,
                                              double* __restrict__ K2, double* __restrict__ S2, int32_t* keys,
                                              double* vals, uint32_t ts, double* s_r, int32_t* s_n) {
  constexpr int NW = NT / kWave;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t t = threadIdx.x; t < ts; t += NT) {
    keys[t] = -1;
    vals[t] = 0.0;
  }
  if (threadIdx.x == 0) *s_n = 0;
  __syncthreads();
  const int32_t m1 = coff[c + 1];
  int32_t q = coff[c] + wv;
  int64_t s = 0;
  int32_t len = 0;
  if (q < m1) {
    const int32_t i = cmem[q];
    s = g.row_start[i];
    len = g.row_len[i];
  }
  double self = 0.0;
  bool any = false;
  while (q < m1) {
    const int32_t nq = q + NW;
    int64_t ns = 0;
    int32_t nl = 0;
    if (nq < m1) {
      const int32_t i = cmem[nq];
      ns = g.row_start[i];
      nl = g.row_len[i];
    }
    for (int32_t k = lane; k < len; k += kWave) {
      const int32_t e = C[g.col[s + k]];
      const double x = static_cast<double>(g.w[s + k]);
      if (e == c) {
        self += x;
        any = true;
      } else {
        tab_add(keys, vals, ts, e, x);
      }
    }
    q = nq;
    s = ns;
    len = nl;
  }
  self = wave_sum_d(self);
  if (__any(any) && lane == 0) tab_add(keys, vals, ts, c, self);
  __syncthreads();
  double k2 = 0.0;
  for (uint32_t t = threadIdx.x; t < ts; t += NT) {
    const int32_t e = GLOBAL ? ld_agent(&keys[t]) : keys[t];
    if (e < 0) continue;
    const float x = static_cast<float>(GLOBAL ? ld_agent(&vals[t]) : vals[t]);
    const int32_t p = atomicAdd(s_n, 1);
    out_col[v0 + p] = e;
    out_w[v0 + p] = x;
    k2 += static_cast<double>(x);
  }
  k2 = wave_sum_d(k2);
  if (lane == 0) s_r[wv] = k2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < NW; ++k) t += s_r[k];
    out_len[c] = *s_n;
    K2[c] = t;
    S2[c] = t;
  }
  __syncthreads();
}

// One workgroup per community c: its members' arcs summed by neighbouring
// community (self-loops included) in FP64, written as the float32 row of
// super-vertex c at vstart[c] (capacity: the members' volume).  Communities
// of up to 2048 arcs take 256 threads and an LDS table of twice their volume;
// larger ones, which a workgroup finds among the communities of its residue
// class, 1024 threads and an LDS table where twice the level's communities fit
// it, else pool slots.
// (256 threads walking one member after another, 28 arcs at a time, and the
// pool's table past 2048 arcs: 986 us for 104 communities of 14,000 arcs;
// this: 45 us, the members' chains of dependent loads.)
struct FAgg {
  FG g;
  const int32_t *C, *coff, *cmem;
  const int64_t* vstart;
  int32_t nc;
  int32_t *out_len, *out_col;
  float* out_w;
  double *K2, *S2;
  int32_t* pkeys;
  double* pvals;
};
__device__ __forceinline__ uint32_t agg_slots(int64_t vol, int32_t nc) {
  const int64_t keys = min(vol, static_cast<int64_t>(nc));
  uint32_t ts = 64u;
  while (ts < 2 * keys) ts <<= 1;
  return ts;
}
__global__ void __launch_bounds__(kBlock) k_f_aggregate(FAgg A) {
  __shared__ int32_t s_keys[kFBlockSlots];
  __shared__ double s_vals[kFBlockSlots];
  __shared__ double s_r[kFNW];
  __shared__ int32_t s_n;
  for (int64_t c = blockIdx.x; c < A.nc; c += gridDim.x) {
    const int64_t v0 = A.vstart[c], vol = A.vstart[c + 1] - v0;
    if (vol > kFBlockMax) continue;
    aggregate_one<kBlock, false>(A.g, A.C, A.coff, A.cmem, static_cast<int32_t>(c), v0, A.out_len, A.out_col, A.out_w,
                                 A.K2, A.S2, s_keys, s_vals, agg_slots(vol, A.nc), s_r, &s_n);
  }
}
__global__ void __launch_bounds__(kFWide) k_f_aggregate_big(FAgg A) {
  __shared__ int32_t s_keys[kFWideSlots];
  __shared__ double s_vals[kFWideSlots];
  __shared__ double s_r[kFWide / kWave];
  __shared__ int32_t s_list[kFWide];
  __shared__ int32_t s_n, s_m;
  for (int64_t k0 = 0; k0 * gridDim.x + blockIdx.x < A.nc; k0 += kFWide) {
    if (threadIdx.x == 0) s_m = 0;
    __syncthreads();
    const int64_t mine = (k0 + threadIdx.x) * gridDim.x + blockIdx.x;
    if (mine < A.nc && A.vstart[mine + 1] - A.vstart[mine] > kFBlockMax)
      s_list[atomicAdd(&s_m, 1)] = static_cast<int32_t>(mine);
    __syncthreads();
    const int32_t found = s_m;
    for (int32_t q = 0; q < found; ++q) {
      const int32_t c = s_list[q];
      const int64_t v0 = A.vstart[c], vol = A.vstart[c + 1] - v0;
      const uint32_t ts = agg_slots(vol, A.nc);
      if (ts <= static_cast<uint32_t>(kFWideSlots))
        aggregate_one<kFWide, false>(A.g, A.C, A.coff, A.cmem, c, v0, A.out_len, A.out_col, A.out_w, A.K2, A.S2,
                                     s_keys, s_vals, ts, s_r, &s_n);
      else  // (ts <= 4 vol)
        aggregate_one<kFWide, true>(A.g, A.C, A.coff, A.cmem, c, v0, A.out_len, A.out_col, A.out_w, A.K2, A.S2,
                                    A.pkeys + 4 * v0, A.pvals + 4 * v0, ts, s_r, &s_n);
    }
    __syncthreads();
  }
}

// Sigma[C_i] += K_i, summed in LDS first (few communities take most of the
// vertices, and device atomics on one address queue).
constexpr int kFSumSlots = 2048;
__global__ void __launch_bounds__(kFWide) k_f_sigma(const int32_t* __restrict__ C, const double* __restrict__ K,
                                                        int32_t n, double* __restrict__ Sigma) {
  __shared__ int32_t s_keys[kFSumSlots];
  __shared__ double s_vals[kFSumSlots];
  for (int t = threadIdx.x; t < kFSumSlots; t += kFWide) {
    s_keys[t] = -1;
    s_vals[t] = 0.0;
  }
  __syncthreads();
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kFWide) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * kFWide) {
    const int32_t c = C[i];
    const double x = K[i];
    if (x == 0.0) continue;
    uint32_t h = hash_slot(static_cast<uint32_t>(c), kFSumSlots);
    bool done = false;
    for (int p = 0; p < 8 && !done; ++p) {
      const int32_t old = atomicCAS(&s_keys[h], -1, c);
      done = old == -1 || old == c;
      if (done) atomicAdd(&s_vals[h], x);
      h = (h + 1) & (kFSumSlots - 1);
    }
    if (!done) atomicAdd(&Sigma[c], x);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kFSumSlots; t += kFWide)
    if (s_keys[t] >= 0 && s_vals[t] != 0.0) atomicAdd(&Sigma[s_keys[t]], s_vals[t]);
}

// The error slot, 2m and the statistics summed over their replicas, to
// pinned host memory: one kernel and a wait (a copy of the counters to
// pageable memory: 5 KB, staged).
struct FRead {
  int64_t err, movers, arcs, processed, expand, affected;
  double dq, sum, sum2, two_m;
};
static_assert(FS_DQ == 5 && FS_SUM == 6 && FS_SUM2 == 7, "FRead lists the statistics in their order");
__global__ void __launch_bounds__(kBlock) k_f_publish(const int64_t* __restrict__ ctr,
                                                    const double* __restrict__ two_m, FRead* __restrict__ out) {
  static_assert(kFReps * 8 == kBlock, "a thread per replica and statistic");
  __shared__ int64_t s_v[kFReps * 8];
  s_v[threadIdx.x] = ctr[F_STATS + (threadIdx.x / 8) * kCtrLine + threadIdx.x % 8];
  __syncthreads();
  const int k = threadIdx.x;
  if (k < FS_DQ) {
    int64_t v = 0;
    for (int r = 0; r < kFReps; ++r) v += s_v[r * 8 + k];
    (&out->movers)[k] = v;
  } else if (k <= FS_SUM2) {
    double v = 0.0;
    for (int r = 0; r < kFReps; ++r) v += __longlong_as_double(s_v[r * 8 + k]);
    (&out->dq)[k - FS_DQ] = v;
  } else if (k == FS_SUM2 + 1) {
    out->err = ctr[F_ERR];
    out->two_m = *two_m;
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct FWs {
  int64_t words = 0;
  uint32_t *fa = nullptr, *fb = nullptr, *ever = nullptr;
  int32_t* list[FB_N] = {};
  int32_t* size = nullptr;
  int32_t* lC = nullptr;
  double *lK = nullptr, *lS = nullptr, *tot = nullptr;
  int32_t *flags = nullptr, *newid = nullptr, *ccount = nullptr, *coff = nullptr, *cmem = nullptr;
  int64_t *vol = nullptr, *vstart = nullptr;
  int64_t* lrs[2] = {};
  int32_t* llen[2] = {};
  int32_t* lcol[2] = {};
  float* lw[2] = {};
  int32_t* pkeys = nullptr;
  double* pvals = nullptr;
  int64_t pool_slots = 0;
  // batch edit tables
  unsigned long long* pkey = nullptr;
  int32_t* pzero = nullptr;
  int64_t psize = 0;
  int32_t *rkey = nullptr, *rapp = nullptr, *rzero = nullptr;
  int64_t rsize = 0;
  int32_t *dpos = nullptr, *imode = nullptr;
  Workspace scan;  // scan partials only
  int64_t* ctr = nullptr;
  const double* two_m = nullptr;  // the graph's
  size_t bytes = 0;
};

size_t carve_f(FWs& w, void* base, int32_t n, int64_t cap) {
  char* cur = static_cast<char*>(base);
  size_t total = 0;
  auto take = [&](size_t bytes) -> void* {
    void* p = base ? cur : nullptr;
    const size_t b = (std::max<size_t>(bytes, 1) + 255) & ~size_t(255);
    cur += b;
    total += b;
    return p;
  };
  const size_t un = static_cast<size_t>(n > 0 ? n : 1), ucap = static_cast<size_t>(cap > 0 ? cap : 1);
  w.words = (static_cast<int64_t>(un) + 31) / 32 + 1;
  w.fa = static_cast<uint32_t*>(take(4 * w.words));
  w.fb = static_cast<uint32_t*>(take(4 * w.words));
  w.ever = static_cast<uint32_t*>(take(4 * w.words));
  for (int b = 0; b < FB_N; ++b) w.list[b] = static_cast<int32_t*>(take(4 * un));
  w.size = static_cast<int32_t*>(take(4 * un));
  w.lC = static_cast<int32_t*>(take(4 * un));
  w.lK = static_cast<double*>(take(8 * un));
  w.lS = static_cast<double*>(take(8 * un));
  w.tot = static_cast<double*>(take(8 * un));
  w.flags = static_cast<int32_t*>(take(4 * (un + 1)));
  w.newid = static_cast<int32_t*>(take(4 * (un + 1)));
  w.ccount = static_cast<int32_t*>(take(4 * (un + 1)));
  w.coff = static_cast<int32_t*>(take(4 * (un + 1)));
  w.cmem = static_cast<int32_t*>(take(4 * un));
  w.vol = static_cast<int64_t*>(take(8 * (un + 1)));
  w.vstart = static_cast<int64_t*>(take(8 * (un + 1)));
  for (int k = 0; k < 2; ++k) {
    w.lrs[k] = static_cast<int64_t*>(take(8 * (un + 1)));
    w.llen[k] = static_cast<int32_t*>(take(4 * un));
    w.lcol[k] = static_cast<int32_t*>(take(4 * ucap));
    w.lw[k] = static_cast<float*>(take(4 * ucap));
  }
  w.pool_slots = 4 * static_cast<int64_t>(ucap) + 8192;
  w.pkeys = static_cast<int32_t*>(take(4 * static_cast<size_t>(w.pool_slots)));
  w.pvals = static_cast<double*>(take(8 * static_cast<size_t>(w.pool_slots)));
  w.scan.scan_part_len = scan_parts_needed(static_cast<int64_t>(un) + 2) + 8;
  w.scan.scan_part = static_cast<int64_t*>(take(8 * static_cast<size_t>(w.scan.scan_part_len)));
  w.ctr = static_cast<int64_t*>(take(8 * F_COUNT));
  w.bytes = total;
  return total;
}

// Carves the batch tables of the edit by pair (below) out of the pool.
bool carve_batch_tables(FWs& w, int64_t updates) {
  int64_t ps = 64;
  while (ps < 4 * updates) ps <<= 1;
  int64_t rs = 64;
  while (rs < 4 * updates) rs <<= 1;
  const size_t need = 8 * ps + 4 * ps + 12 * rs + 4 * 2 * updates + 4 * updates + 8 * 256;
  // the pool (keys, then values: 12 bytes a slot) is free during a batch edit
  if (need > static_cast<size_t>(w.pool_slots) * 12) return false;
  char* p = reinterpret_cast<char*>(w.pkeys);
  auto take = [&](size_t bytes) {
    char* q = p;
    p += (bytes + 255) & ~size_t(255);
    return q;
  };
  w.psize = ps;
  w.rsize = rs;
  w.pkey = reinterpret_cast<unsigned long long*>(take(8 * ps));
  w.pzero = reinterpret_cast<int32_t*>(take(4 * ps));
  w.rkey = reinterpret_cast<int32_t*>(take(4 * rs));
  w.rapp = reinterpret_cast<int32_t*>(take(4 * rs));
  w.rzero = reinterpret_cast<int32_t*>(take(4 * rs));
  w.dpos = reinterpret_cast<int32_t*>(take(8 * std::max<int64_t>(updates, 1)));
  w.imode = reinterpret_cast<int32_t*>(take(4 * std::max<int64_t>(updates, 1)));
  return true;
}

#define F_HIP(expr)                                                          \
  do {                                                                       \
    hipError_t e__ = (expr);                                                 \
    if (e__ != hipSuccess) return lv_fail(LV_EHIP, hipGetErrorString(e__));  \
  } while (0)

int blocks(int64_t items, int cap = 8192) {
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((items + kBlock - 1) / kBlock, cap)));
}

lv_status setup(FWs& w, const lv_graph_f* g, void* ws, size_t ws_bytes) {
  if (!g || g->n <= 0 || !g->row_start || !g->row_len || !g->col || !g->w || !g->two_m || g->cap < 0)
    return lv_fail(LV_EINVAL, "invalid graph");
  if (g->cap >= (int64_t(1) << 30)) return lv_fail(LV_EINVAL, "capacity of 2^30 arcs or more");
  if (!ws) return lv_fail(LV_EINVAL, "workspace pointer is null");
  if (ws_bytes < carve_f(w, nullptr, g->n, g->cap)) return lv_fail(LV_EWORKSPACE, "workspace too small");
  carve_f(w, ws, g->n, g->cap);
  w.two_m = g->two_m;
  return LV_OK;
}

// The error slot, 2m and the statistics, on the host.
lv_status read(const FWs& w, FRead& r, hipStream_t st) {
  int64_t* host;
  if (lv_status s = lv_pinned_host(&host)) return s;
  hipLaunchKernelGGL(k_f_publish, dim3(1), dim3(kBlock), 0, st, w.ctr, w.two_m, reinterpret_cast<FRead*>(host));
  F_HIP(hipGetLastError());
  F_HIP(hipStreamSynchronize(st));
  std::memcpy(&r, host, sizeof(FRead));
  return LV_OK;
}

lv_status zero_stats(const FWs& w, hipStream_t st) {
  F_HIP(hipMemsetAsync(w.ctr + F_LIST0, 0, sizeof(int64_t) * (F_COUNT - F_LIST0), st));
  return LV_OK;
}

lv_status dev_error(int64_t code) {
  if (code == LV_EEMPTY) return lv_fail(LV_EEMPTY, "graph has no edges (2m = 0)");
  if (code == LV_EINVAL) return lv_fail(LV_EINVAL, "the batch names a vertex outside [0, n), a self-loop or a "
                                                   "weight that is not finite and positive");
  if (code == kBadMember) return lv_fail(LV_EINVAL, "a membership lies outside [0, n)");
  if (code == LV_ENOEDGE) return lv_fail(LV_ENOEDGE, "a deletion names a missing edge or more weight than present");
  if (code == LV_ENOSLACK) return lv_fail(LV_ENOSLACK, "a row lacks free capacity; nothing was changed");
  if (code == LV_EWORKSPACE) return lv_fail(LV_EWORKSPACE, "workspace pool too small");
  return lv_fail(static_cast<lv_status>(code), "device error");
}

bool params_ok_f(const lv_params* p) {
  return p && p->mode == LV_ASYNC && p->max_iterations >= 1 && p->max_iterations <= LV_MAX_ITERS &&
         p->max_passes >= 1 && p->max_passes <= LV_MAX_PASSES && p->tolerance >= 0.0 && p->tolerance_drop > 0.0 &&
         p->aggregation_tolerance >= 0.0 && p->recompute_weights == 0 && p->reserved == 0;
}

// The batch edit by touched row (batch.hip) in the pool: counters, then the
// scratch.
int64_t* edit_counters(const FWs& w) { return reinterpret_cast<int64_t*>(w.pkeys); }
constexpr size_t kEditCtrBytes = (sizeof(int64_t) * CTR_COUNT + 255) & ~size_t(255);

// Each touched row is scanned once by the wavefronts of its chunks.  A batch
// whose scratch exceeds the pool (one of nearly as many updates as the graph
// has arcs) is edited by pair instead, one thread per update scanning its
// rows: on a 250,001-vertex power-law graph with hub rows 1000 updates take
// 2.1 ms that way.
bool edit_by_row(const FWs& w, int64_t nd, int64_t ni, int64_t cap) {
  BatchScratch b;
  return kEditCtrBytes + carve_batch(b, nullptr, nd, ni, cap) <= static_cast<size_t>(w.pool_slots) * 12;
}

lv_status enqueue_edit(const FWs& w, const lv_graph_f& g, const lv_edges_f& del, const lv_edges_f& ins,
                       hipStream_t st) {
  BatchScratch b;
  carve_batch(b, reinterpret_cast<char*>(w.pkeys) + kEditCtrBytes, del.count, ins.count, g.cap);
  b.tag = w.ever;
  b.row_slot = w.list[FB_WAVE];
  if (del.count + ins.count <= kSmallUpdates)
    launch_small_batch_f(g, del, ins, b, edit_counters(w), st);
  else
    launch_batch_f(g, del, ins, b, w.words, edit_counters(w), st);
  F_HIP(hipGetLastError());
  return LV_OK;
}

FBatch fbatch(const lv_edges_f* del, const lv_edges_f* ins) {
  FBatch b{};
  if (del && del->count > 0) {
    b.du = del->u;
    b.dv = del->v;
    b.dw = del->w;
    b.nd = del->count;
  }
  if (ins && ins->count > 0) {
    b.iu = ins->u;
    b.iv = ins->v;
    b.iw = ins->w;
    b.ni = ins->count;
  }
  return b;
}

bool edges_ok_f(const lv_edges_f* e) { return !e || e->count == 0 || (e->count > 0 && e->u && e->v && e->w); }

// The scans of one sub-round over the bins in `mask`, longest rows first;
// at most that many rows each.
void launch_scans_f(const FMove& M, uint32_t mask, int64_t hubs, int64_t big, int64_t rows, hipStream_t st) {
  if (mask & (1u << FB_HUB))
    hipLaunchKernelGGL(k_f_scan_group<true>, dim3(static_cast<int>(std::min<int64_t>(hubs, 256))), dim3(kFWide), 0,
                       st, M);
  if (mask & (1u << FB_BLOCK))
    hipLaunchKernelGGL(k_f_scan_group<false>, dim3(static_cast<int>(std::min<int64_t>(big, 768))), dim3(kBlock), 0,
                       st, M);
  if (mask & (1u << FB_WAVE))
    hipLaunchKernelGGL(k_f_scan_wave, dim3(blocks(rows * kWave, 4096)), dim3(kBlock), 0, st, M);
}

// The sub-rounds of one iteration from a plan of the frontier (plan.hip).
// The plan's bins up to the wavefront's lie next to each other in a
// sub-round's list and are one launch here.  (Binning per sub-round and
// launching every bin: 17.4-22 ms for a static run on a 50,003-vertex SBM
// graph, 4900 launches; planned: 3.4-4.4 ms.)
lv_status planned_rounds_f(FMove& M, const FWs& w, uint32_t* cur, uint32_t* ever, const std::vector<SubRound>& plan,
                           const lv_tuning& tu, lv_stats& S, hipStream_t st) {
  const PlanKeys pk = lv_plan_keys(plan, tu);
  PlanArgs a{};
  a.cur = cur;
  a.ever = ever;
  a.row_len = M.g.row_len;
  a.n = M.g.n;
  a.wave_max = kFWaveMax;
  for (int b = 0; b < NBINS; ++b) a.list[b] = w.list[FB_WAVE];
  a.mem = w.pkeys;  // (read back before the first scan uses the pool)
  launch_plan(a, pk, TimerPair(), st);
  int64_t* host;
  if (lv_status s = lv_pinned_host(&host)) return s;
  F_HIP(hipMemcpyAsync(host, w.pkeys, kPlanArcs + 8 * kPlanKeys, hipMemcpyDeviceToHost, st));
  F_HIP(hipStreamSynchronize(st));
  const int32_t* h = reinterpret_cast<const int32_t*>(host);
  const int64_t* arcs = host + kPlanArcs / 8;
  if (ever) S.vertices_affected += h[kPlanHost - kPlanTail + PT_AFFECTED];
  std::vector<int32_t> first(kPlanKeys);
  int32_t run = 0;
  for (int k = 0; k < pk.rounds * 8; ++k) {
    first[k] = run;
    if (k % 8 < NBINS) run += h[k];
  }
  for (const SubRound& r : plan) {
    const int32_t* c = h + r.key * 8;
    for (int b = 0; b < 8; ++b) S.arcs_scanned += arcs[r.key * 8 + b];
    int64_t rows = 0;
    for (int b = 0; b <= BIN_WAVE; ++b) rows += c[b];
    M.cnt[FB_WAVE] = rows;
    M.cnt[FB_BLOCK] = c[BIN_BLOCK];
    M.cnt[FB_HUB] = c[BIN_HUB];
    M.list[FB_WAVE] = w.list[FB_WAVE] + first[r.key * 8];
    M.list[FB_BLOCK] = w.list[FB_WAVE] + first[r.key * 8 + BIN_BLOCK];
    M.list[FB_HUB] = w.list[FB_WAVE] + first[r.key * 8 + BIN_HUB];
    const uint32_t mask = (rows ? 1u << FB_WAVE : 0u) | (c[BIN_BLOCK] ? 1u << FB_BLOCK : 0u) |
                          (c[BIN_HUB] ? 1u << FB_HUB : 0u);
    if (c[BIN_HUB])  // pool slots start over
      F_HIP(hipMemsetAsync(w.ctr + F_POOL, 0, sizeof(int64_t), st));
    launch_scans_f(M, mask, c[BIN_HUB], c[BIN_BLOCK], rows, st);
  }
  return LV_OK;
}

// Alg. 4 in the paper's precision, ASYNC; DF marking and updateWeights first
// for the dynamic call.
lv_status run_f(bool df, const lv_graph_f* g, const lv_edges_f* del, const lv_edges_f* ins, const lv_params* p,
                lv_state_f* state, void* wsp, size_t ws_bytes, lv_stats* stats, void* stream) {
  const auto t0 = std::chrono::steady_clock::now();
  if (!params_ok_f(p)) return lv_fail(LV_EINVAL, "invalid parameters (the paper-precision path runs LV_ASYNC)");
  if (!state || !state->C || !state->K || !state->Sigma) return lv_fail(LV_EINVAL, "invalid state");
  if (df && (!edges_ok_f(del) || !edges_ok_f(ins))) return lv_fail(LV_EINVAL, "invalid batch");
  FWs w;
  lv_status s = setup(w, g, wsp, ws_bytes);
  if (s) return s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  lv_stats local;
  lv_stats& S = stats ? *stats : local;
  std::memset(&S, 0, sizeof(lv_stats));
  const int32_t N = g->n;
  const lv_tuning tu = lv_effective_tuning();
  hipLaunchKernelGGL(k_f_begin, dim3(blocks(std::max<int64_t>(w.words, F_COUNT), 2048)), dim3(kBlock), 0, st, w.ctr,
                     w.fa, w.fb, w.ever, w.words, g->two_m);
  FG L0{N, g->row_start, g->row_len, g->col, g->w};
  int32_t* size0 = state->size ? state->size : w.size;
  if (!df) {
    hipLaunchKernelGGL(k_f_rows, dim3(blocks(static_cast<int64_t>(N) * kWave, 16384)), dim3(kBlock), 0,
                       st, L0, nullptr, state->K, state->Sigma, state->C, size0, w.ctr);
    hipLaunchKernelGGL(k_f_set_all, dim3(blocks(w.words)), dim3(kBlock), 0, st, w.fa, N, w.words);
  } else {
    const FBatch b = fbatch(del, ins);
    hipLaunchKernelGGL(k_f_check_c, dim3(blocks(N)), dim3(kBlock), 0, st, state->C, N, w.ctr);
    if (!state->size) {  // (the member counts index by C)
      FRead rc;
      if ((s = read(w, rc, st))) return s;
      if (rc.err) return dev_error(rc.err);
      launch_community_sizes(state->C, N, w.size, st);
    }
    if (b.nd + b.ni > 0)
      hipLaunchKernelGGL(k_f_update, dim3(blocks(b.nd + b.ni)), dim3(kBlock), 0, st, b, N, state->C, state->K,
                         state->Sigma, w.fa, w.ctr);
  }
  F_HIP(hipGetLastError());
  FRead rd{};

  FG L = L0;
  int32_t* Cl = state->C;
  const double* Kl = state->K;
  double* Sl = state->Sigma;
  int32_t* size = size0;
  uint32_t* cur = w.fa;
  uint32_t* next = w.fb;
  double tau = p->tolerance;
  bool aggregated = false;
  for (int32_t pass = 0; pass < p->max_passes; ++pass) {
    int32_t li = p->max_iterations;
    int64_t est = L.n;
    if (pass == 0 && df) est = 2 * (fbatch(del, ins).nd + fbatch(del, ins).ni);
    for (int32_t it = 0; it < p->max_iterations; ++it) {
      if (pass + it > 0 && (s = zero_stats(w, st))) return s;  // (k_f_begin cleared them)
      const std::vector<SubRound> plan = lv_sub_rounds(LV_ASYNC, pass, est, L.n, tu);
      FMove M{L, Cl, Kl, Sl, size, next, {w.list[FB_WAVE], w.list[FB_BLOCK], w.list[FB_HUB]}, {-1, -1, -1}, w.two_m,
              p->swap_guard, w.ctr, w.pool_slots, w.pkeys, w.pvals};
      if (plan.size() > 1) {
        if ((s = planned_rounds_f(M, w, cur, pass == 0 ? w.ever : nullptr, plan, tu, S, st))) return s;
      } else {
        hipLaunchKernelGGL(k_f_bin, dim3(blocks(w.words, 4096)), dim3(kBlock), 0, st, cur,
                           pass == 0 ? w.ever : nullptr, L.row_len, L.n, w.list[FB_WAVE], w.list[FB_BLOCK],
                           w.list[FB_HUB], w.ctr);
        const int64_t e = std::max<int64_t>(64, est);
        launch_scans_f(M, 7u, e, e, e, st);
      }
      F_HIP(hipGetLastError());
      std::swap(cur, next);
      if ((s = read(w, rd, st))) return s;
      if (rd.err) return dev_error(rd.err);
      est = rd.expand;
      S.moves += rd.movers;
      S.arcs_scanned += rd.arcs;
      if (pass == 0) S.vertices_affected += rd.affected;
      if (pass < LV_MAX_PASSES && it < LV_MAX_ITERS) S.iter_moves[pass][it] = rd.movers;
      if (rd.dq <= tau) {
        li = it + 1;
        break;
      }
    }
    S.passes = pass + 1;
    S.iterations[pass] = li;
    if (li <= 1) break;
    // renumber (ascending old id), then the aggregation stop
    F_HIP(hipMemsetAsync(w.flags, 0, sizeof(int32_t) * (static_cast<size_t>(L.n) + 1), st));
    launch_mark_exists(Cl, L.n, w.flags, st);
    exclusive_scan_i32(w.flags, w.newid, L.n, w.scan, st);
    int32_t nc = 0;
    F_HIP(hipMemcpyAsync(&nc, w.newid + L.n, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    F_HIP(hipStreamSynchronize(st));
    S.communities[pass] = nc;
    if (static_cast<double>(nc) / static_cast<double>(L.n) > p->aggregation_tolerance) break;
    launch_relabel(Cl, L.n, w.newid, st);
    if (pass > 0) launch_lookup(state->C, N, Cl, st);
    // members and volumes of the communities
    F_HIP(hipMemsetAsync(w.ccount, 0, sizeof(int32_t) * (static_cast<size_t>(nc) + 1), st));
    F_HIP(hipMemsetAsync(w.vol, 0, sizeof(int64_t) * (static_cast<size_t>(nc) + 1), st));
    launch_accumulate(Cl, L.n, L.row_len, nullptr, w.ccount, w.vol, st);  // member counts, volumes
    exclusive_scan_i32(w.ccount, w.coff, nc, w.scan, st);
    F_HIP(hipMemsetAsync(w.flags, 0, sizeof(int32_t) * (static_cast<size_t>(nc) + 1), st));
    launch_fill_members(Cl, L.n, w.coff, w.flags, w.cmem, st);
    const int k = pass & 1;
    exclusive_scan_i64(w.vol, w.lrs[k], nc, w.scan, st);
    const FAgg A{L, Cl, w.coff, w.cmem, w.lrs[k], nc, w.llen[k], w.lcol[k], w.lw[k], w.lK, w.lS, w.pkeys, w.pvals};
    hipLaunchKernelGGL(k_f_aggregate_big, dim3(std::min(nc, 256)), dim3(kFWide), 0, st, A);
    hipLaunchKernelGGL(k_f_aggregate, dim3(std::min(nc, 8192)), dim3(kBlock), 0, st, A);
    // the aggregate read the level's memberships (w.lC past the first pass)
    launch_iota_i32(w.lC, nc, st);
    launch_fill_i32(w.size, 1, nc, st);
    hipLaunchKernelGGL(k_f_set_all, dim3(blocks(w.words)), dim3(kBlock), 0, st, cur, nc, w.words);
    F_HIP(hipGetLastError());
    L = FG{nc, w.lrs[k], w.llen[k], w.lcol[k], w.lw[k]};
    Cl = w.lC;
    Kl = w.lK;
    Sl = w.lS;
    size = w.size;
    tau /= p->tolerance_drop;
    aggregated = true;
  }
  if (aggregated) {
    launch_lookup(state->C, N, Cl, st);
    hipLaunchKernelGGL(k_f_zero_d, dim3(blocks(N)), dim3(kBlock), 0, st, state->Sigma, static_cast<int64_t>(N));
    hipLaunchKernelGGL(k_f_sigma, dim3(std::min(256, N / 4096 + 1)), dim3(kFWide), 0, st, state->C, state->K, N,
                       state->Sigma);
    if (state->size) launch_community_sizes(state->C, N, state->size, st);
    F_HIP(hipGetLastError());
  }
  if (aggregated) F_HIP(hipStreamSynchronize(st));  // (else the last iteration's read waited)
  S.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return LV_OK;
}

}  // namespace
}  // namespace lv

using namespace lv;

extern "C" {

size_t lv_workspace_bytes_f(int32_t n, int64_t cap) {
  FWs w;
  return carve_f(w, nullptr, n, cap);
}

lv_status lv_graph_build_f(lv_graph_f* g, const lv_edges_f* e, float slack_frac, int32_t slack_min, void* wsp,
                           size_t ws_bytes, void* stream) {
  if (!e || !edges_ok_f(e) || slack_frac < 0.f || slack_min < 0) return lv_fail(LV_EINVAL, "invalid arguments");
  FWs w;
  lv_status s = setup(w, g, wsp, ws_bytes);
  if (s) return s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int32_t n = g->n;
  F_HIP(hipMemsetAsync(w.ctr, 0, sizeof(int64_t) * F_COUNT, st));
  F_HIP(hipMemsetAsync(g->row_len, 0, sizeof(int32_t) * static_cast<size_t>(n), st));
  if (e->count > 0)
    hipLaunchKernelGGL(k_f_count, dim3(blocks(e->count)), dim3(kBlock), 0, st, e->u, e->v, e->w, e->count, n,
                       g->row_len, w.ctr);
  // capacities: deg + max(slack_min, ceil(frac * deg)), then their scan
  launch_row_capacity(g->row_len, w.vol, n, slack_frac, slack_min, st);
  exclusive_scan_i64(w.vol, g->row_start, n, w.scan, st);
  FRead rd;
  if ((s = read(w, rd, st))) return s;
  if (rd.err) return dev_error(rd.err);
  int64_t need = 0;
  F_HIP(hipMemcpyAsync(&need, g->row_start + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
  F_HIP(hipStreamSynchronize(st));
  if (need > g->cap) return lv_fail(LV_ENOSLACK, "graph capacity too small (see lv_graph_capacity_bound)");
  F_HIP(hipMemsetAsync(g->row_len, 0, sizeof(int32_t) * static_cast<size_t>(n), st));
  if (e->count > 0)
    hipLaunchKernelGGL(k_f_scatter, dim3(blocks(e->count)), dim3(kBlock), 0, st, e->u, e->v, e->w, e->count,
                       g->row_start, g->row_len, g->col, g->w);
  FG G{n, g->row_start, g->row_len, g->col, g->w};
  hipLaunchKernelGGL(k_f_rows, dim3(blocks(static_cast<int64_t>(n) * kWave, 16384)), dim3(kBlock), 0, st,
                     G, nullptr, nullptr, nullptr, nullptr, nullptr, w.ctr);
  hipLaunchKernelGGL(k_f_set_two_m, dim3(1), dim3(1), 0, st, g->two_m, w.ctr, 0);
  F_HIP(hipGetLastError());
  F_HIP(hipStreamSynchronize(st));
  return LV_OK;
}

lv_status apply_batch_f(lv_graph_f* g, const lv_edges_f* del, const lv_edges_f* ins, void* wsp, size_t ws_bytes,
                        void* stream) {
  if (!edges_ok_f(del) || !edges_ok_f(ins)) return lv_fail(LV_EINVAL, "invalid batch");
  FWs w;
  lv_status s = setup(w, g, wsp, ws_bytes);
  if (s) return s;
  const FBatch b = fbatch(del, ins);
  if (b.nd + b.ni == 0) return LV_OK;
  if (edit_by_row(w, b.nd, b.ni, g->cap)) {
    const lv_edges_f none{};
    if ((s = enqueue_edit(w, *g, del ? *del : none, ins ? *ins : none, static_cast<hipStream_t>(stream)))) return s;
    int64_t err = 0;
    F_HIP(hipMemcpyAsync(&err, edit_counters(w), sizeof(int64_t), hipMemcpyDeviceToHost,
                         static_cast<hipStream_t>(stream)));
    F_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    return err ? dev_error(err) : LV_OK;
  }
  if (!carve_batch_tables(w, b.nd + b.ni)) return lv_fail(LV_EWORKSPACE, "batch too large for the workspace pool");
  hipStream_t st = static_cast<hipStream_t>(stream);
  F_HIP(hipMemsetAsync(w.ctr, 0, sizeof(int64_t) * F_COUNT, st));
  F_HIP(hipMemsetAsync(w.pkey, 0, 8 * static_cast<size_t>(w.psize), st));
  F_HIP(hipMemsetAsync(w.pzero, 0, 4 * static_cast<size_t>(w.psize), st));
  F_HIP(hipMemsetAsync(w.rkey, 0, 4 * static_cast<size_t>(w.rsize), st));
  F_HIP(hipMemsetAsync(w.rapp, 0, 4 * static_cast<size_t>(w.rsize), st));
  F_HIP(hipMemsetAsync(w.rzero, 0, 4 * static_cast<size_t>(w.rsize), st));
  FBTab t{w.pkey, w.pzero, w.psize, w.rkey, w.rapp, w.rzero, w.rsize, w.dpos, w.imode};
  lv_graph_f G = *g;
  if (b.nd) hipLaunchKernelGGL(k_f_val_del, dim3(blocks(b.nd)), dim3(kBlock), 0, st, b, G, t, w.ctr);
  if (b.ni) hipLaunchKernelGGL(k_f_val_ins, dim3(blocks(b.ni)), dim3(kBlock), 0, st, b, G, t, w.ctr);
  hipLaunchKernelGGL(k_f_val_cap, dim3(blocks(w.rsize)), dim3(kBlock), 0, st, G, t, w.ctr);
  F_HIP(hipGetLastError());
  FRead rd;
  if ((s = read(w, rd, st))) return s;
  if (rd.err) return dev_error(rd.err);
  if (b.nd) hipLaunchKernelGGL(k_f_del, dim3(blocks(b.nd)), dim3(kBlock), 0, st, b, G, t, w.ctr);
  hipLaunchKernelGGL(k_f_compact, dim3(blocks(w.rsize)), dim3(kBlock), 0, st, G, t, w.ctr);
  if (b.ni) hipLaunchKernelGGL(k_f_ins, dim3(blocks(b.ni)), dim3(kBlock), 0, st, b, G, t, w.ctr);
  hipLaunchKernelGGL(k_f_set_two_m, dim3(1), dim3(1), 0, st, g->two_m, w.ctr, 1);
  F_HIP(hipGetLastError());
  F_HIP(hipStreamSynchronize(st));
  return LV_OK;
}

lv_status louvain_static_f(const lv_graph_f* g, const lv_params* p, lv_state_f* out, void* ws, size_t ws_bytes,
                           lv_stats* stats, void* stream) {
  return run_f(false, g, nullptr, nullptr, p, out, ws, ws_bytes, stats, stream);
}

lv_status louvain_df_f(const lv_graph_f* g, const lv_edges_f* del, const lv_edges_f* ins, const lv_params* p,
                       lv_state_f* state, void* ws, size_t ws_bytes, lv_stats* stats, void* stream) {
  return run_f(true, g, del, ins, p, state, ws, ws_bytes, stats, stream);
}

lv_status modularity_f(const lv_graph_f* g, const int32_t* C, double* q_host, void* wsp, size_t ws_bytes,
                       void* stream) {
  if (!C || !q_host) return lv_fail(LV_EINVAL, "invalid arguments");
  FWs w;
  lv_status s = setup(w, g, wsp, ws_bytes);
  if (s) return s;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int32_t n = g->n;
  F_HIP(hipMemsetAsync(w.ctr, 0, sizeof(int64_t) * F_COUNT, st));
  FG G{n, g->row_start, g->row_len, g->col, g->w};
  hipLaunchKernelGGL(k_f_rows, dim3(blocks(static_cast<int64_t>(n) * kWave, 16384)), dim3(kBlock), 0, st,
                     G, C, w.lK, nullptr, nullptr, nullptr, w.ctr);
  FRead rd;
  if ((s = read(w, rd, st))) return s;
  const double intra = rd.sum2;
  F_HIP(hipMemsetAsync(w.ctr, 0, sizeof(int64_t) * F_COUNT, st));
  hipLaunchKernelGGL(k_f_zero_d, dim3(blocks(n)), dim3(kBlock), 0, st, w.tot, static_cast<int64_t>(n));
  hipLaunchKernelGGL(k_f_totals, dim3(blocks(n)), dim3(kBlock), 0, st, C, w.lK, n, w.tot, w.ctr);
  hipLaunchKernelGGL(k_f_sumsq, dim3(blocks(n, 4096)), dim3(kBlock), 0, st, w.tot, n, w.ctr);
  F_HIP(hipGetLastError());
  if ((s = read(w, rd, st))) return s;
  const double two_m = rd.two_m;
  if (rd.err) return lv_fail(LV_EINVAL, "a membership lies outside [0, n)");
  if (!(two_m > 0.0)) return lv_fail(LV_EEMPTY, "graph has no edges (2m = 0)");
  *q_host = intra / two_m - rd.sum / (two_m * two_m);
  return LV_OK;
}

}  // extern "C"
