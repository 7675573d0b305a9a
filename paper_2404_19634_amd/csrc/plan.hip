// Plan of one local-moving iteration: the frontier sorted by (sub-round,
// degree bin) in one pass over the bitmask.
//
// An ASYNC iteration visits the frontier in up to 128 sub-rounds (degree
// classes and hash rounds, lv_api.hip).  Picking each sub-round's vertices
// out of the bitmask again (k_bin_frontier, move.hip) walks the whole
// frontier once per sub-round, and without the counts on the host every bin
// of every sub-round is launched, empty or not: 5200 launches and 28 ms for a
// 10,000-vertex graph that holds two of the four degree classes, 19 us per
// binning on 300,000 vertices.  The plan counts the vertices and arcs of every
// (sub-round, bin) key, scans the counts, places the vertices, and prepares
// all hub rows' units; one readback then tells the host which launches
// remain and how large they are.  Moves of a sub-round never change the
// frontier being visited (they mark the next one), so planning them all
// before the first is the same schedule.
//
// Bound: one read of row_len per frontier vertex twice (count, place) and
// one 4-byte write: latency of four short kernels on small levels, HBM on
// large ones.  A workgroup takes tiles of 2048 vertices; counts are summed
// in LDS per key and reserved with one device atomic per key and tile.  (Count
// and place of 700,000 vertices 11 + 12 us with tiles of 4096, 9 + 10 of 2048,
// 10 + 11 of 1024; of 10,000 7 + 10, 5 + 7, 4 + 6.)
//
// Measured, picking per sub-round -> plan: static ASYNC on the 10,000-vertex
// SBM graph 29.8 -> 4.9 ms, on a 300,000-vertex power-law graph 24.0 -> 12.3
// ms; DS on 300,000 vertices 7.03 -> 0.99 ms; static SYNC (one round per
// iteration) on a 700,001-vertex R-MAT graph 24.0 -> 20.6 ms.
#include <algorithm>
#include <climits>

#include <hip/hip_ext.h>

#include "lv_internal.hpp"

namespace lv {
namespace {

constexpr int kPer = 8;                      // vertices per thread and tile
constexpr int kPlanTile = kBlock * kPer;
constexpr int kWordsPerTile = kPlanTile / 32;
constexpr int kKeySlots = 8;                 // bins of a sub-round (slot 7: rows without arcs)

// The sub-round of a vertex (see sub_rounds in lv_api.hip).
__device__ __forceinline__ int round_of(const PlanKeys& k, int32_t i, int32_t deg, int32_t n) {
  const int h = k.hash_bits > 0 ? static_cast<int>((static_cast<uint32_t>(i) * 0x9E3779B1u) >> (32 - k.hash_bits)) : 0;
  if (k.by_class) {
    const int c = deg >= 1025 ? 0 : deg >= 129 ? 1 : deg >= 17 ? 2 : 3;
    return (c << k.hash_bits) | h;
  }
  if (k.by_id)  // the range [n r / R, n (r + 1) / R) that holds i
    return static_cast<int>(((static_cast<int64_t>(i) + 1) * k.rounds + n - 1) / n - 1);
  return h;
}

struct Frontier {
  uint32_t* cur;
  const uint32_t* range;
  const int32_t* row_len;
  int32_t n;
  int32_t wave_max;
};

// The keys of this thread's vertices of tile t (-1: not in the frontier).
// Returns whether the tile holds any frontier vertex (workgroup-uniform).
__device__ __forceinline__ bool tile_keys(const Frontier& f, const PlanKeys& pk, int64_t t, int32_t (&key)[kPer],
                                          int32_t (&deg)[kPer], uint32_t* s_w) {
  const int64_t words = (static_cast<int64_t>(f.n) + 31) / 32;
  const int64_t w0 = t * kWordsPerTile;
  bool any = false;
  if (threadIdx.x < kWordsPerTile) {
    uint32_t w = 0;
    if (w0 + threadIdx.x < words) {
      w = f.cur[w0 + threadIdx.x];
      if (w && f.range) w &= f.range[w0 + threadIdx.x];
    }
    s_w[threadIdx.x] = w;
    any = w != 0;
  }
  if (!__syncthreads_or(any)) return false;
  const int64_t base = t * kPlanTile;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {  // (every bit below n: the frontier holds vertices only)
    const int v = q * kBlock + threadIdx.x;
    const bool on = (s_w[v >> 5] >> (v & 31)) & 1u;
    deg[q] = on ? f.row_len[base + v] : -1;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    key[q] = -1;
    if (deg[q] < 0) continue;
    const int32_t i = static_cast<int32_t>(base + q * kBlock + threadIdx.x);
    const int b = bin_of(deg[q], f.wave_max);
    key[q] = round_of(pk, i, deg[q], f.n) * kKeySlots + (b < 0 ? kKeySlots - 1 : b);
  }
  return true;
}

// Counters of the plan, the other sub-round and statistics sets, and the
// next frontier's list counts start from zero.
__global__ void k_plan_begin(PlanBuf p, int64_t* __restrict__ rc_next, int64_t* __restrict__ sc_next,
                             int64_t* __restrict__ next_cnt, int64_t* __restrict__ stamp) {
  if (stamp && threadIdx.x == 0) *stamp = static_cast<int64_t>(wall_clock64());
  for (int k = threadIdx.x; k < kPlanKeys; k += blockDim.x) {
    p.cnt[k] = 0;
    p.arcs[k] = 0;
  }
  for (int k = threadIdx.x; k < kPlanTail; k += blockDim.x) p.tail[k] = 0;
  if (rc_next)
    for (int k = threadIdx.x; k < kRoundSet; k += blockDim.x) rc_next[k] = 0;
  if (sc_next)
    for (int k = threadIdx.x; k < kStatSet; k += blockDim.x) sc_next[k] = 0;
  if (next_cnt)
    for (int r = threadIdx.x; r < kFlRegions; r += blockDim.x) next_cnt[r * kCtrLine] = 0;
}

__global__ void __launch_bounds__(kBlock) k_plan_count(Frontier f, PlanKeys pk, PlanBuf p) {
  __shared__ uint32_t s_w[kWordsPerTile];
  __shared__ int32_t s_cnt[kPlanKeys];
  __shared__ unsigned long long s_arc[kPlanKeys];
  __shared__ int32_t s_max;
  const int keys = pk.rounds * kKeySlots;
  for (int k = threadIdx.x; k < keys; k += kBlock) {
    s_cnt[k] = 0;
    s_arc[k] = 0;
  }
  if (threadIdx.x == 0) s_max = 0;
  const int64_t tiles = (static_cast<int64_t>(f.n) + kPlanTile - 1) / kPlanTile;
  int32_t top = 0;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    int32_t key[kPer], deg[kPer];
    __syncthreads();  // (the last tile's words are read; the counters are clear)
    if (!tile_keys(f, pk, t, key, deg, s_w)) continue;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (key[q] < 0) continue;
      atomicAdd(&s_cnt[key[q]], 1);
      if (deg[q]) atomicAdd(&s_arc[key[q]], static_cast<unsigned long long>(deg[q]));
      top = max(top, deg[q]);
    }
  }
  if (top > kBlockMaxDegree) atomicMax(&s_max, top);  // (only the longest hub row matters)
  __syncthreads();
  for (int k = threadIdx.x; k < keys; k += kBlock)
    if (s_cnt[k]) {
      atomicAdd(&p.cnt[k], s_cnt[k]);
      atomicAdd(reinterpret_cast<unsigned long long*>(&p.arcs[k]), s_arc[k]);
    }
  if (threadIdx.x == 0 && s_max) atomicMax(&p.tail[PT_MAXDEG], s_max);
}

// One workgroup: first list entry of every key, and the iteration's
// statistics (a sub-round visited twice counts twice).  With one sub-round
// each bin has a list of its own and its count goes to the round counters.
__global__ void __launch_bounds__(kBlock) k_plan_scan(PlanKeys pk, PlanBuf p, int64_t* __restrict__ rc,
                                                     int64_t* __restrict__ sc) {
  constexpr int kSpan = kPlanKeys / kBlock;
  __shared__ int32_t s_w[kBlock / kWave];
  __shared__ unsigned long long s_v[kKeySlots], s_a[kKeySlots];
  const int keys = pk.rounds * kKeySlots;
  const int lane = lane_id();
  if (threadIdx.x < kKeySlots) {
    s_v[threadIdx.x] = 0;
    s_a[threadIdx.x] = 0;
  }
  int32_t c[kSpan];
  int32_t sum = 0;
#pragma unroll
  for (int q = 0; q < kSpan; ++q) {
    const int k = threadIdx.x * kSpan + q;
    c[q] = (k < keys && k % kKeySlots != kKeySlots - 1) ? p.cnt[k] : 0;
    sum += c[q];
  }
  int32_t incl = sum;
  for (int s = 1; s < kWave; s <<= 1) {
    const int32_t o = __shfl_up(incl, s);
    if (lane >= s) incl += o;
  }
  if (lane == kWave - 1) s_w[threadIdx.x / kWave] = incl;
  __syncthreads();
  int32_t run = incl - sum;
  for (int w = 0; w < static_cast<int>(threadIdx.x) / kWave; ++w) run += s_w[w];
#pragma unroll
  for (int q = 0; q < kSpan; ++q) {
    const int k = threadIdx.x * kSpan + q;
    if (k < keys) p.cursor[k] = pk.rounds == 1 ? 0 : run;
    run += c[q];
  }
  if (!sc) return;
  // statistics: thread t sums the keys t, t + 256, ...: one bin
  int64_t v = 0, a = 0;
  for (int k = threadIdx.x; k < keys; k += kBlock) {
    const int r = k / kKeySlots;
    const int64_t visits = pk.by_class && (r >> pk.hash_bits) < pk.twice ? 2 : 1;
    v += visits * p.cnt[k];
    a += visits * p.arcs[k];
  }
  if (v) atomicAdd(&s_v[threadIdx.x % kKeySlots], static_cast<unsigned long long>(v));
  if (a) atomicAdd(&s_a[threadIdx.x % kKeySlots], static_cast<unsigned long long>(a));
  __syncthreads();
  if (threadIdx.x < kKeySlots) {
    const int b = threadIdx.x;
    v = static_cast<int64_t>(s_v[b]);
    a = static_cast<int64_t>(s_a[b]);
    if (v) {
      stat_add(sc, ST_PROCESSED, v);
      if (a) stat_add(sc, ST_ARCS, a);
      if (b < NBINS) {
        stat_add(sc, ST_BIN_V0 + b, v);
        stat_add(sc, ST_BIN_A0 + b, a);
      }
    }
    if (pk.rounds == 1 && b < NBINS) rc[rc_bin(b)] = p.cnt[b];
  }
}

struct PlanLists {
  int32_t* list[NBINS];  // one sub-round: per bin; else the same list
};

__global__ void __launch_bounds__(kBlock) k_plan_fill(Frontier f, PlanKeys pk, PlanBuf p, PlanLists L,
                                                     uint32_t* __restrict__ ever, int64_t* __restrict__ sc) {
  __shared__ uint32_t s_w[kWordsPerTile];
  __shared__ int32_t s_cnt[kPlanKeys];
  __shared__ int32_t s_base[kPlanKeys];
  const int keys = pk.rounds * kKeySlots;
  for (int k = threadIdx.x; k < keys; k += kBlock) s_cnt[k] = 0;
  const int64_t tiles = (static_cast<int64_t>(f.n) + kPlanTile - 1) / kPlanTile;
  const int64_t words = (static_cast<int64_t>(f.n) + 31) / 32;
  int64_t affected = 0;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    int32_t key[kPer], deg[kPer], pos[kPer];
    __syncthreads();
    const bool any = tile_keys(f, pk, t, key, deg, s_w);
    const int64_t w = t * kWordsPerTile + threadIdx.x;
    if (threadIdx.x < kWordsPerTile && w < words) {  // the frontier is consumed
      if (f.cur[w]) f.cur[w] = 0;
      if (any && ever && s_w[threadIdx.x]) {
        const uint32_t old = ever[w];
        affected += __popc(s_w[threadIdx.x] & ~old);
        ever[w] = old | s_w[threadIdx.x];
      }
    }
    if (!any) continue;
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      pos[q] = key[q] >= 0 && key[q] % kKeySlots != kKeySlots - 1 ? atomicAdd(&s_cnt[key[q]], 1) : -1;
    __syncthreads();
    for (int k = threadIdx.x; k < keys; k += kBlock) {
      const int32_t c = s_cnt[k];
      if (c) s_base[k] = atomicAdd(&p.cursor[k], c);
      s_cnt[k] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (pos[q] < 0) continue;
      L.list[key[q] % kKeySlots][s_base[key[q]] + pos[q]] =
          static_cast<int32_t>(t * kPlanTile + q * kBlock + threadIdx.x);
    }
  }
  affected = wave_sum_i64(affected);
  if (lane_id() == 0 && affected) {
    if (sc)
      stat_add(sc, ST_AFFECTED, affected);
    else
      atomicAdd(&p.tail[PT_AFFECTED], static_cast<int32_t>(affected));
  }
}

// Hub rows of sub-round blockIdx.x: table offsets (each sub-round uses the
// pool from its start), units, and zero sums.  Units of all sub-rounds lie
// one after another (reserved with one atomic each).  NT threads: 1024 where
// one workgroup has the whole frontier's hubs (some thousands on a
// 700,000-vertex R-MAT graph: 22 us with 256 threads and LDS scans, 11 so),
// 256 where there is a workgroup per sub-round.
template <int NT>
__global__ void __launch_bounds__(NT) k_plan_hubs(PlanBuf p, PlanLists L, int32_t rounds,
                                                 const int32_t* __restrict__ row_len, HubOut H,
                                                 int64_t* __restrict__ hub_kid, int64_t* __restrict__ rc) {
  constexpr int NW = NT / kWave;
  __shared__ int64_t s_wo[NW], s_wu[NW];  // the wavefronts' sums: slots; units | clear units << 32
  __shared__ int32_t s_u[NT], s_c[NT];    // inclusive sums of a chunk
  __shared__ int32_t s_before, s_ub, s_cb, s_ut, s_ct;
  const int r = blockIdx.x;
  const int key = r * kKeySlots + BIN_HUB;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int32_t count = p.cnt[key];
  if (count == 0) return;
  if (threadIdx.x == 0) s_before = s_ut = s_ct = 0;
  __syncthreads();
  for (int q = threadIdx.x; q < r; q += NT) {
    const int32_t c = p.cnt[q * kKeySlots + BIN_HUB];
    if (c) atomicAdd(&s_before, c);
  }
  // (the key's list range ends at the cursor that placed it)
  const int32_t* list = L.list[BIN_HUB] + (p.cursor[key] - count);
  if (rounds > 1) {  // the sub-round's share of the units (a single one's start at 0)
    int32_t ut = 0, ct = 0;
    for (int32_t k = threadIdx.x; k < count; k += NT) {
      const int32_t deg = row_len[list[k]];
      ut += static_cast<int32_t>(hub_units(deg));
      ct += static_cast<int32_t>(hub_cunits(deg));
    }
    ut = wave_sum_i32(ut);
    ct = wave_sum_i32(ct);
    if (lane == 0) {
      atomicAdd(&s_ut, ut);
      atomicAdd(&s_ct, ct);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      s_ub = atomicAdd(&p.tail[PT_UNITS], s_ut);
      s_cb = atomicAdd(&p.tail[PT_CUNITS], s_ct);
      p.hub_ubase[r] = s_ub;
      p.hub_units[r] = s_ut;
      p.hub_cbase[r] = s_cb;
      p.hub_cunits[r] = s_ct;
      p.hub_first[r] = s_before;
    }
  } else if (threadIdx.x == 0) {
    s_ub = s_cb = 0;
  }
  __syncthreads();
  const int64_t hb = s_before;
  int64_t off0 = 0;
  int32_t u0 = 0, c0 = 0;
  for (int32_t k0 = 0; k0 < count; k0 += NT) {
    const int32_t k = k0 + threadIdx.x;
    const int32_t m = min(NT, count - k0);
    const int32_t deg = k < count ? row_len[list[k]] : 0;
    const int64_t sl = k < count ? hub_slots(deg) : 0;
    const int32_t nu = k < count ? static_cast<int32_t>(hub_units(deg)) : 0;
    const int32_t nc = k < count ? static_cast<int32_t>(hub_cunits(deg)) : 0;
    int64_t io = sl, iu = (static_cast<int64_t>(nc) << 32) | nu;  // (sums stay under 2^31 each)
    for (int d = 1; d < kWave; d <<= 1) {
      const int64_t a = __shfl_up(io, d), b = __shfl_up(iu, d);
      if (lane >= d) {
        io += a;
        iu += b;
      }
    }
    if (lane == kWave - 1) {
      s_wo[wv] = io;
      s_wu[wv] = iu;
    }
    __syncthreads();
    int64_t to = 0, tu = 0;  // the chunk's sums
    for (int q = 0; q < NW; ++q) {
      if (q == wv) {
        io += to;
        iu += tu;
      }
      to += s_wo[q];
      tu += s_wu[q];
    }
    s_u[threadIdx.x] = static_cast<int32_t>(iu);
    s_c[threadIdx.x] = static_cast<int32_t>(iu >> 32);
    __syncthreads();
    if (k < count) {
      H.off[hb + k] = off0 + io - sl;
      H.cbase[hb + k] = c0 + static_cast<int32_t>(iu >> 32) - nc;
      H.cnum[hb + k] = nc;
      hub_kid[hb + k] = 0;
    }
    // unit x of the chunk belongs to the first hub whose inclusive sum exceeds x
    auto owner = [&](const int32_t* incl, int32_t x) {
      int lo = 0, hi = m - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (incl[mid] > x) hi = mid; else lo = mid + 1;
      }
      return lo;
    };
    const int32_t cu = static_cast<int32_t>(tu), cc = static_cast<int32_t>(tu >> 32);
    for (int32_t x = threadIdx.x; x < cu; x += NT) {
      const int q = owner(s_u, x);
      H.u_b[s_ub + u0 + x] = k0 + q;
      H.u_a[s_ub + u0 + x] = static_cast<int64_t>(x - (q ? s_u[q - 1] : 0)) * kHubUnitArcs;
    }
    for (int32_t x = threadIdx.x; x < cc; x += NT) {
      const int q = owner(s_c, x);
      H.c_b[s_cb + c0 + x] = k0 + q;
      H.c_s[s_cb + c0 + x] = static_cast<int64_t>(x - (q ? s_c[q - 1] : 0)) * kHubClearSlots;
    }
    off0 += to;
    u0 += cu;
    c0 += cc;
    __syncthreads();
  }
  if (rounds == 1 && threadIdx.x == 0) {
    rc[RC_HUB_UNITS] = u0;
    rc[RC_HUB_CUNITS] = c0;
  }
}

}  // namespace

PlanBuf plan_buf(void* mem) {
  PlanBuf p;
  p.cnt = static_cast<int32_t*>(mem);
  p.hub_ubase = p.cnt + kPlanKeys;
  p.hub_units = p.hub_ubase + kPlanRounds;
  p.hub_cbase = p.hub_units + kPlanRounds;
  p.hub_cunits = p.hub_cbase + kPlanRounds;
  p.hub_first = p.hub_cunits + kPlanRounds;
  p.tail = p.hub_first + kPlanRounds;
  p.arcs = reinterpret_cast<int64_t*>(static_cast<char*>(mem) + kPlanArcs);
  p.cursor = reinterpret_cast<int32_t*>(p.arcs + kPlanKeys);
  return p;
}

void launch_plan(const PlanArgs& a, const PlanKeys& pk, const TimerPair& t, hipStream_t st) {
  const PlanBuf p = plan_buf(a.mem);
  const Frontier f{a.cur, a.range, a.row_len, a.n, a.wave_max};
  PlanLists L;
  for (int b = 0; b < NBINS; ++b) L.list[b] = pk.rounds == 1 ? a.list[b] : a.list[0];
  const int64_t tiles = (static_cast<int64_t>(a.n) + kPlanTile - 1) / kPlanTile;
  const unsigned grid = static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(tiles, 2048)));
  // (timed from the first kernel's begin to the last one's end)
  const hipEvent_t none = nullptr;
  hipExtLaunchKernelGGL(k_plan_begin, dim3(1), dim3(1024), 0, st, t.start, none, 0, p, a.rc_next, a.sc_next,
                        a.next_cnt, a.stamp);
  hipLaunchKernelGGL(k_plan_count, dim3(grid), dim3(kBlock), 0, st, f, pk, p);
  hipLaunchKernelGGL(k_plan_scan, dim3(1), dim3(kBlock), 0, st, pk, p, a.rc, a.sc);
  hipExtLaunchKernelGGL(k_plan_fill, dim3(grid), dim3(kBlock), 0, st, none, a.hub_kid ? none : t.stop, 0, f, pk, p, L,
                        a.ever, a.sc);
  if (!a.hub_kid) return;
  if (pk.rounds == 1)
    hipExtLaunchKernelGGL(k_plan_hubs<1024>, dim3(1), dim3(1024), 0, st, none, t.stop, 0, p, L, pk.rounds, a.row_len,
                          a.hub, a.hub_kid, a.rc);
  else
    hipExtLaunchKernelGGL(k_plan_hubs<kBlock>, dim3(static_cast<unsigned>(pk.rounds)), dim3(kBlock), 0, st, none,
                          t.stop, 0, p, L, pk.rounds, a.row_len, a.hub, a.hub_kid, a.rc);
}

}  // namespace lv
