// Small batches: the edit, updateWeights, DF's marking and the first
// binning in three launches.
//
// A batch of a few hundred updates is bound by launches: eleven kernels of
// the edit (batch.hip) and four before the first scan, 2 to 11 us each for
// a few microseconds of dependent loads, 100 of 140 us.  Up to
// kSmallUpdates updates one workgroup of 1024 threads does everything but
// the row scans, one update per thread, with the tables and counts in LDS
// and barriers in place of launches:
//   k_small_head  validation, the pair table, the touched rows, their scan
//                 chunks (workgroup 0); the other workgroups clear the
//                 call's bitmasks meanwhile;
//   k_scan        (batch.hip) the touched rows, over the whole device;
//   k_small_tail  checks, the edit, Alg. 7, Alg. 1's marking, and the
//                 frontier's degree bins and hub units.
// The limit is one update per thread.  Update in one call, grid-wide kernels
// -> this, us (R-MAT of 2^20 vertices; power-law graph of 400,000): 20 updates
// 114 -> 66, 125 -> 67; 300 updates 136 -> 90, 130 -> 75; 1000 updates
// 173 -> 143, 144 -> 108.
#include <algorithm>
#include <climits>

#include "batch_device.hpp"
#include "lv_internal.hpp"

namespace lv {
namespace {

constexpr int kSB = 1024;                       // threads, and updates, of the workgroup
constexpr int kSW = kSB / kWave;
constexpr int kPairSlots = 4096;                // LDS pair table: at least 2 x updates + 2
constexpr int kRowSlots = 4096;                 // LDS table of touched rows: at most 2 x updates keys
static_assert(kSmallUpdates <= kSB && 2 * kSmallUpdates + 2 <= kPairSlots, "one update per thread");
constexpr int64_t kTwoMLimit = int64_t(1) << 31;

template <class T>
__device__ __forceinline__ T ld_agent(const T* p) {  // what other lanes changed with atomics
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix sum over the workgroup, with the total.
__device__ __forceinline__ int64_t scan_1024(int64_t v, int64_t* total, int64_t* lds) {
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  int64_t incl = v;
  for (int s = 1; s < kWave; s <<= 1) {
    const int64_t o = __shfl_up(incl, s);
    if (lane >= s) incl += o;
  }
  if (lane == kWave - 1) lds[wv] = incl;
  __syncthreads();
  int64_t before = 0, tot = 0;
  for (int w = 0; w < kSW; ++w) {
    if (w < wv) before += lds[w];
    tot += lds[w];
  }
  __syncthreads();
  *total = tot;
  return before + incl - v;
}

template <class T>
__device__ __forceinline__ T sum_1024(T v, T* lds) {
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  if (lane_id() == 0) lds[threadIdx.x / kWave] = v;
  __syncthreads();
  T t = 0;
  for (int w = 0; w < kSW; ++w) t += lds[w];
  __syncthreads();
  return t;
}

// The batch as the head and tail see it.  dw / iw of the pair table and the
// listing direction of each direction's row pass through the scratch:
// b.d_rank[e] is the direction that lists e's row.
template <class W>
__global__ void __launch_bounds__(kSB) k_small_head(Upd<W> U, int32_t edit, int32_t n,
                                                   const int64_t* __restrict__ row_start,
                                                   const int32_t* __restrict__ row_len, BatchScratch b,
                                                   int64_t* __restrict__ ctr, uint32_t* __restrict__ fr_a,
                                                   uint32_t* __restrict__ fr_b, uint32_t* __restrict__ ever,
                                                   uint32_t* __restrict__ moved, int64_t words) {
  if (blockIdx.x > 0) {  // the call's bitmasks
    const int64_t stride = static_cast<int64_t>(gridDim.x - 1) * kSB;
    for (int64_t k = (blockIdx.x - 1) * static_cast<int64_t>(kSB) + threadIdx.x; k < words; k += stride) {
      fr_a[k] = 0;
      fr_b[k] = 0;
      ever[k] = 0;
      moved[k] = 0;
    }
    return;
  }
  using T = decltype(as_total(W()));
  __shared__ uint64_t p_key[kPairSlots];
  __shared__ int32_t p_dw[kPairSlots];
  __shared__ int32_t p_iw[kPairSlots];
  __shared__ int32_t r_key[kRowSlots];   // row, or -1
  __shared__ int32_t r_list[kRowSlots];  // the direction that lists it
  __shared__ int32_t r_cnt[kRowSlots];   // its directions, then its first partner
  __shared__ int64_t s_scan[kSW];
  __shared__ T s_sum[kSW];
  __shared__ int32_t s_bad;
  for (int k = threadIdx.x; k < CTR_COUNT; k += kSB)
    ctr[k] = k == CTR_T_CALL ? static_cast<int64_t>(wall_clock64()) : 0;
  if (!edit) return;
  const int t = threadIdx.x;
  const uint32_t size = static_cast<uint32_t>(b.size);  // <= kPairSlots
  for (uint32_t s = t; s < size; s += kSB) {
    p_key[s] = kEmpty;
    p_dw[s] = 0;
    p_iw[s] = 0;
  }
  for (int s = t; s < kRowSlots; s += kSB) {
    r_key[s] = -1;
    r_cnt[s] = 0;
  }
  if (t == 0) s_bad = 0;
  __syncthreads();
  const int total = static_cast<int>(U.nd + U.ni);
  const bool on = t < total;
  const bool del = t < U.nd;
  int32_t end[2] = {0, 0};
  W x = 0;
  if (on) {
    end[0] = del ? U.du[t] : U.iu[t - U.nd];
    end[1] = del ? U.dv[t] : U.iv[t - U.nd];
    x = del ? U.dw[t] : U.iw[t - U.nd];
  }
  const int32_t a = end[0], c = end[1];
  bool ok = on && a >= 0 && c >= 0 && a < n && c < n && a != c && usable(x);
  int32_t h = -1;
  if (ok) {
    const uint64_t key = canon(a, c);
    uint32_t p = hash64(key, size - 1);
    while (true) {  // at most half full: ends
      const unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(&p_key[p]), kEmpty, key);
      if (old == kEmpty || old == key) break;
      p = (p + 1) & (size - 1);
    }
    h = static_cast<int32_t>(p);
    int32_t bits;
    __builtin_memcpy(&bits, &x, sizeof(bits));
    if (atomicCAS(del ? &p_dw[h] : &p_iw[h], 0, bits) != 0) ok = false;  // pair repeated on this side
  }
  if (on && !ok) s_bad = 1;
  // the touched rows: slot, listing direction, rank of the direction
  int32_t slot[2] = {-1, -1}, rank[2] = {0, 0};
  bool lists[2] = {false, false};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (!ok) continue;
    uint32_t p = mix32(static_cast<uint32_t>(end[q])) & (kRowSlots - 1);
    while (true) {  // at most half full: ends
      const int32_t old = atomicCAS(&r_key[p], -1, end[q]);
      if (old == -1 || old == end[q]) {
        lists[q] = old == -1;
        break;
      }
      p = (p + 1) & (kRowSlots - 1);
    }
    slot[q] = static_cast<int32_t>(p);
    if (lists[q]) r_list[p] = 2 * t + q;
    rank[q] = atomicAdd(&r_cnt[p], 1);
  }
  const T si = sum_1024(ok && !del ? as_total(x) : T(0), s_sum);  // (also the barrier behind the tables)
  const T sd = sum_1024(ok && del ? as_total(x) : T(0), s_sum);
  // chunks and partner ranges of the listed rows
  int32_t len[2] = {0, 0}, cnt[2] = {0, 0};
  int64_t start[2] = {0, 0};
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (lists[q]) {
      len[q] = row_len[end[q]];
      start[q] = row_start[end[q]];
      cnt[q] = r_cnt[slot[q]];
    }
  int64_t mine = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (lists[q]) mine += (static_cast<int64_t>((len[q] + kChunk - 1) / kChunk) << 32) | cnt[q];
  int64_t all = 0;
  int64_t at = scan_1024(mine, &all, s_scan);  // (barriers: every r_cnt is read before it is replaced)
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (!lists[q]) continue;
    const int32_t pbase = static_cast<int32_t>(at & 0xffffffffll);
    const int64_t cbase = at >> 32;
    const int32_t nch = (len[q] + kChunk - 1) / kChunk;
    r_cnt[slot[q]] = pbase;
    b.r_pbase[2 * t + q] = pbase;
    b.r_len[2 * t + q] = len[q];
    for (int32_t k = 0; k < nch; ++k) {
      BatchScratch::Chunk w;
      w.s = start[q];
      w.a = end[q];
      w.off = k * kChunk;
      w.end = min(len[q], (k + 1) * kChunk);
      w.cnt = cnt[q];
      w.pbase = pbase;
      w.pad = 0;
      b.chunk[cbase + k] = w;
    }
    at += (static_cast<int64_t>(nch) << 32) | cnt[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (on) b.row_of[2 * t + q] = lists[q] ? end[q] : -1;
    if (slot[q] < 0) continue;
    b.part[r_cnt[slot[q]] + rank[q]] = end[1 - q];
    b.d_rank[2 * t + q] = r_list[slot[q]];
  }
  if (on) b.slot[t] = ok ? h : -1;
  for (uint32_t s = t; s < size; s += kSB) {
    b.keys[s] = p_key[s];
    b.dw[s] = p_dw[s];
    b.iw[s] = p_iw[s];
    b.pos[2 * s] = -1;
    b.pos[2 * s + 1] = -1;
  }
  if (t == 0) {
    ctr[CTR_ERR] = s_bad ? LV_EINVAL : 0;
    ctr[CTR_B_RESV] = all;
    reinterpret_cast<T*>(ctr + CTR_STATS0)[ST_W_INS] = si;
    reinterpret_cast<T*>(ctr + CTR_STATS0)[ST_W_DEL] = sd;
  }
}

// Checks and phase 2 of the edit (batch.hip) by the workgroup; returns the
// error code.  Nothing of the graph is written on error.
template <class W, class T>
__device__ __forceinline__ int32_t small_edit(const Upd<W>& U, const int64_t* row_start, int32_t* row_len, int32_t* col,
                                              W* wt, T* two_m, bool bound, const BatchScratch& b, const int64_t* ctr,
                                              int32_t* r_zero, int32_t* r_app, int32_t* s_err) {
  const int t = threadIdx.x;
  const int total = static_cast<int>(U.nd + U.ni);
  const bool on = t < total;
  const bool del = t < U.nd;
  const W* dw = reinterpret_cast<const W*>(b.dw);
  const W* iw = reinterpret_cast<const W*>(b.iw);
  W* tw = reinterpret_cast<W*>(b.tw);
  for (int k = t; k < 2 * total; k += kSB) {
    r_zero[k] = 0;
    r_app[k] = 0;
  }
  if (t == 0) *s_err = static_cast<int32_t>(ctr[CTR_ERR]);
  __syncthreads();
  int32_t end[2] = {0, 0}, row[2] = {0, 0}, of[2] = {-1, -1}, len[2] = {0, 0};
  int64_t pos[2] = {-1, -1};
  bool merge[2] = {false, false}, zero[2] = {false, false};
  W cur[2] = {0, 0};
  W dwh = 0, iwh = 0;
  if (on && *s_err == 0) {
    const int32_t h = b.slot[t];
    end[0] = del ? U.du[t] : U.iu[t - U.nd];
    end[1] = del ? U.dv[t] : U.iv[t - U.nd];
    dwh = dw[h];
    iwh = iw[h];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      pos[q] = b.pos[2 * static_cast<int64_t>(h) + (end[q] > end[1 - q] ? 1 : 0)];
      row[q] = b.d_rank[2 * t + q];
      of[q] = b.row_of[2 * t + q];
      len[q] = of[q] >= 0 ? b.r_len[2 * t + q] : 0;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) cur[q] = pos[q] >= 0 ? wt[pos[q]] : W(0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool gone = dwh > 0 && !(cur[q] - dwh > 0);
      if (del) {
        if (pos[q] < 0 || cur[q] < dwh) {
          atomicCAS(s_err, 0, LV_ENOEDGE);
        } else if (gone) {
          zero[q] = true;
          atomicAdd(&r_zero[row[q]], 1);
        }
      } else {
        merge[q] = pos[q] >= 0 && !gone;
        if (!merge[q]) atomicAdd(&r_app[row[q]], 1);
      }
    }
  }
  __syncthreads();
  const T add = 2 * (reinterpret_cast<const T*>(ctr + CTR_STATS0)[ST_W_INS] -
                     reinterpret_cast<const T*>(ctr + CTR_STATS0)[ST_W_DEL]);
  const T nm = *two_m + add;
  if (bound && t == 0 && nm >= static_cast<T>(kTwoMLimit)) atomicCAS(s_err, 0, LV_EOVERFLOW);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (of[q] < 0) continue;
    const int64_t need = static_cast<int64_t>(len[q]) - r_zero[2 * t + q] + r_app[2 * t + q];
    if (need > row_start[of[q] + 1] - row_start[of[q]]) atomicCAS(s_err, 0, LV_ENOSLACK);
  }
  __syncthreads();
  if (*s_err) return *s_err;
  // weights: a pair deleted in part and merged back is written by its
  // deletion, in that order
  if (on) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (del)
        wt[pos[q]] = zero[q] ? W(0) : (cur[q] - dwh) + iwh;
      else if (merge[q] && dwh == 0)
        wt[pos[q]] = cur[q] + iwh;
    }
  }
  if (t == 0) *two_m = nm;
  __syncthreads();
  // rows that lost arcs: survivors of the cut tail (as k_tail)
  const int lane = lane_id();
  int64_t start[2] = {0, 0};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int32_t z = of[q] >= 0 ? r_zero[2 * t + q] : 0;
    if (of[q] >= 0) start[q] = row_start[of[q]];
    const int32_t pbase = z ? b.r_pbase[2 * t + q] : 0;
    if (z > 0 && z <= 16) {
      int64_t p = pbase;
      for (int32_t k = len[q] - z; k < len[q]; ++k) {
        const W x = wt[start[q] + k];
        if (x > 0) {
          b.tcol[p] = col[start[q] + k];
          tw[p] = x;
          ++p;
        }
      }
      row_len[of[q]] = len[q] - z;
    }
    for (uint64_t m = __ballot(z > 16); m; m &= m - 1) {
      const int src = __ffsll(static_cast<unsigned long long>(m)) - 1;
      const int32_t wz = __shfl(z, src), wl = __shfl(len[q], src), wr = __shfl(of[q], src);
      const int64_t ws = __shfl(start[q], src);
      const int32_t wp = __shfl(pbase, src);
      int32_t out = 0;
      for (int32_t k0 = wl - wz; k0 < wl; k0 += kWave) {
        const int32_t k = k0 + lane;
        const W x = k < wl ? wt[ws + k] : W(0);
        const bool keep = x > 0;
        const uint64_t km = __ballot(keep);
        if (keep) {
          const int64_t p = wp + out + __popcll(km & ((1ull << lane) - 1ull));
          b.tcol[p] = col[ws + k];
          tw[p] = x;
        }
        out += __popcll(km);
      }
      if (lane == 0) row_len[wr] = wl - wz;
    }
  }
  // the rows' state for every direction: start and length of the listed row
  __syncthreads();
  // (r_zero keeps the counts; r_app becomes the holes filled so far)
  int32_t lp[2] = {0, 0}, pb[2] = {0, 0};
  int64_t rs[2] = {0, 0};
  if (on) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      lp[q] = b.r_len[row[q]] - r_zero[row[q]];
      pb[q] = b.r_pbase[row[q]];
      rs[q] = row_start[end[q]];
    }
  }
  __syncthreads();
  for (int k = t; k < 2 * total; k += kSB) r_app[k] = 0;
  __syncthreads();
  if (on) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (del) {
        if (zero[q] && pos[q] - rs[q] < lp[q]) {
          const int32_t j = atomicAdd(&r_app[row[q]], 1);
          col[pos[q]] = b.tcol[pb[q] + j];
          wt[pos[q]] = tw[pb[q] + j];
        }
      } else if (!merge[q]) {
        const int64_t p = rs[q] + atomicAdd(&row_len[end[q]], 1);
        col[p] = end[1 - q];
        wt[p] = iwh;
      }
    }
  }
  __syncthreads();
  return 0;
}

template <class W, class T>
__global__ void __launch_bounds__(kSB) k_small_edit(Upd<W> U, const int64_t* __restrict__ row_start, int32_t* row_len,
                                                   int32_t* col, W* wt, T* two_m, int32_t bound, BatchScratch b,
                                                   int64_t* ctr) {
  __shared__ int32_t r_zero[2 * kSmallUpdates], r_app[2 * kSmallUpdates];
  __shared__ int32_t s_err;
  const int32_t err = small_edit(U, row_start, row_len, col, wt, two_m, bound != 0, b, ctr, r_zero, r_app, &s_err);
  if (threadIdx.x == 0 && err) ctr[CTR_ERR] = err;
}

struct SmallDf {
  const int32_t* C;
  int64_t* K;
  int64_t* Sigma;
  uint32_t* fr;    // frontier bitmask (clear on entry)
  FrontList fl;
  uint32_t* ever;
  int32_t bin;     // 1: the frontier goes to the degree bins; 0: to bitmask and list
  int32_t wave_max;
  int32_t* list[NBINS];
  HubOut hub;
  int64_t* hub_kid;
};

// The edit (if `edit`), then Alg. 7 and Alg. 1 for the batch, then (df.bin)
// the frontier in degree bins with its hub units and the iteration's
// statistics, as the first sub-round's binning leaves them.
__global__ void __launch_bounds__(kSB) k_small_tail(Upd<int32_t> U, int32_t edit, int32_t n,
                                                   const int64_t* __restrict__ row_start, int32_t* row_len,
                                                   int32_t* col, int32_t* wt, int64_t* two_m, BatchScratch b,
                                                   int64_t* ctr, SmallDf df) {
  constexpr int kSigSlots = 4096;  // at most 2 x updates communities: half full
  union Lds {
    struct {
      int32_t r_zero[2 * kSmallUpdates], r_app[2 * kSmallUpdates];
    } e;
    struct {
      int32_t key[kSigSlots];
      unsigned long long val[kSigSlots];
    } s;
    struct {
      int32_t pos[2 * kSmallUpdates], deg[2 * kSmallUpdates];
      int32_t u[2 * kSmallUpdates], c[2 * kSmallUpdates];  // inclusive sums of the hubs' units
    } h;
  };
  __shared__ Lds L;
  __shared__ int32_t s_err, s_nh;
  __shared__ int64_t s_scan[kSW];
  __shared__ int32_t s_bin[NBINS];
  __shared__ unsigned long long s_arc[NBINS];
  __shared__ int32_t s_proc;
  const int t = threadIdx.x;
  int32_t err = 0;
  if (edit) err = small_edit(U, row_start, row_len, col, wt, two_m, true, b, ctr, L.e.r_zero, L.e.r_app, &s_err);
  const int64_t tm = *two_m;
  if (t == 0) {
    if (!err) err = tm <= 0 ? LV_EEMPTY : (tm >= kTwoMLimit ? LV_EOVERFLOW : 0);
    s_err = err;
    ctr[CTR_TWO_M] = tm;
    ctr[CTR_T_CALL] = static_cast<int64_t>(wall_clock64());  // (DF's part begins after the edit)
    if (err) ctr[CTR_ERR] = err;
    s_nh = 0;
    s_proc = 0;
    // (the batch's weight totals sat in the statistics)
    ctr[CTR_STATS0 + ST_W_INS] = 0;
    ctr[CTR_STATS0 + ST_W_DEL] = 0;
  }
  if (t < NBINS) {
    s_bin[t] = 0;
    s_arc[t] = 0;
  }
  __syncthreads();
  if (s_err) return;
  for (int k = t; k < kSigSlots; k += kSB) {
    L.s.key[k] = -1;
    L.s.val[k] = 0;
  }
  __syncthreads();
  const int total = static_cast<int>(U.nd + U.ni);
  const bool del = t < U.nd;
  int32_t v[2] = {0, 0};
  int64_t x = 0;
  bool on = t < total;
  if (on) {
    v[0] = del ? U.du[t] : U.iu[t - U.nd];
    v[1] = del ? U.dv[t] : U.iv[t - U.nd];
    x = del ? -static_cast<int64_t>(U.dw[t]) : static_cast<int64_t>(U.iw[t - U.nd]);
    if (v[0] < 0 || v[1] < 0 || v[0] >= n || v[1] >= n || v[0] == v[1]) {
      set_error(ctr, LV_EINVAL);  // (not the batch the edit took: skipped, and reported)
      on = false;
    }
  }
  const int32_t c[2] = {on ? df.C[v[0]] : 0, on ? df.C[v[1]] : 0};
  const bool hit = on && (c[0] == c[1]) == del;
  bool fresh[2] = {false, false};
  if (df.bin) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t bit = 1u << (v[q] & 31);
      if (hit) fresh[q] = !(atomicOr(&df.fr[v[q] >> 5], bit) & bit);
    }
  } else {
    const bool both[2] = {hit, hit};
    front_mark_n(df.fr, df.fl, v, both);
  }
  if (on) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      atomic_add_i64(&df.K[v[q]], x);
      uint32_t p = hash_slot(static_cast<uint32_t>(c[q]), kSigSlots);
      while (true) {
        const int32_t old = atomicCAS(&L.s.key[p], -1, c[q]);
        if (old == -1 || old == c[q]) {
          atomicAdd(&L.s.val[p], static_cast<unsigned long long>(x));
          break;
        }
        p = (p + 1) & (kSigSlots - 1);
      }
    }
  }
  int32_t deg[2] = {0, 0}, at[2] = {-1, -1};
#pragma unroll
  for (int q = 0; q < 2; ++q)  // (appended rows: their lengths changed by atomics)
    if (fresh[q]) deg[q] = ld_agent(&row_len[v[q]]);
  __syncthreads();
  for (int k = t; k < kSigSlots; k += kSB)
    if (L.s.key[k] >= 0 && L.s.val[k]) atomic_add_i64(&df.Sigma[L.s.key[k]], static_cast<int64_t>(L.s.val[k]));
  if (!df.bin) {
    if (t == 0) ctr[CTR_T_MOVE] = static_cast<int64_t>(wall_clock64());
    return;
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (!fresh[q]) continue;
    const uint32_t bit = 1u << (v[q] & 31);
    atomicOr(&df.ever[v[q] >> 5], bit);
    atomicAnd(&df.fr[v[q] >> 5], ~bit);  // the frontier is consumed
    atomicAdd(&s_proc, 1);
    const int bin = bin_of(deg[q], df.wave_max);
    if (bin < 0) continue;
    at[q] = atomicAdd(&s_bin[bin], 1);
    atomicAdd(&s_arc[bin], static_cast<unsigned long long>(deg[q]));
    df.list[bin][at[q]] = v[q];
  }
  __syncthreads();  // (the Sigma table is read; its LDS serves the hubs)
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (fresh[q] && deg[q] > kBlockMaxDegree) {
      const int k = atomicAdd(&s_nh, 1);
      L.h.pos[k] = at[q];
      L.h.deg[k] = deg[q];
    }
  __syncthreads();
  int64_t* rc = ctr + CTR_ROUND0;
  const int nh = s_nh;
  int32_t u0 = 0, c0 = 0;
  if (nh > 0) {
    // Two hubs to a thread: prefix sums give each its pool slots and units,
    // and a unit finds its hub by a search of the sums.  (Hubs one after
    // another an update of 300 edges between 512 rows of 2600 arcs took 251 us,
    // of 1024 between 2048 rows 725; the grid-wide kernels 200 and 347; this
    // 118 and 240.)
    int64_t slots = 0, units = 0;  // units | clear units << 32 (each sum stays under 2^31)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (2 * t + q < nh) {
        const int32_t d = L.h.deg[2 * t + q];
        slots += hub_slots(d);
        units += (hub_cunits(d) << 32) | hub_units(d);
      }
    int64_t all_slots = 0, all_units = 0;
    int64_t off = scan_1024(slots, &all_slots, s_scan);
    int64_t at_unit = scan_1024(units, &all_units, s_scan);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (2 * t + q < nh) {
        const int32_t p = L.h.pos[2 * t + q], d = L.h.deg[2 * t + q];
        df.hub.off[p] = off;
        df.hub.cbase[p] = at_unit >> 32;
        df.hub.cnum[p] = static_cast<int32_t>(hub_cunits(d));
        df.hub_kid[p] = 0;
        off += hub_slots(d);
        at_unit += (hub_cunits(d) << 32) | hub_units(d);
        L.h.u[2 * t + q] = static_cast<int32_t>(at_unit);
        L.h.c[2 * t + q] = static_cast<int32_t>(at_unit >> 32);
      }
    __syncthreads();
    auto owner = [&](const int32_t* incl, int32_t x) {  // the first hub whose inclusive sum exceeds x
      int lo = 0, hi = nh - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (incl[mid] > x) hi = mid; else lo = mid + 1;
      }
      return lo;
    };
    u0 = static_cast<int32_t>(all_units);
    c0 = static_cast<int32_t>(all_units >> 32);
    for (int32_t x = t; x < u0; x += kSB) {
      const int k = owner(L.h.u, x);
      df.hub.u_b[x] = L.h.pos[k];
      df.hub.u_a[x] = static_cast<int64_t>(x - (k ? L.h.u[k - 1] : 0)) * kHubUnitArcs;
    }
    for (int32_t x = t; x < c0; x += kSB) {
      const int k = owner(L.h.c, x);
      df.hub.c_b[x] = L.h.pos[k];
      df.hub.c_s[x] = static_cast<int64_t>(x - (k ? L.h.c[k - 1] : 0)) * kHubClearSlots;
    }
  }
  int64_t* sc = ctr + CTR_STATS0;
  if (t < NBINS) {
    rc[rc_bin(t)] = s_bin[t];
    sc[ST_BIN_V0 + t] = s_bin[t];
    sc[ST_BIN_A0 + t] = static_cast<int64_t>(s_arc[t]);
  }
  if (t == 0) {
    rc[RC_HUB_UNITS] = u0;
    rc[RC_HUB_CUNITS] = c0;
    int64_t arcs = 0;
    for (int q = 0; q < NBINS; ++q) arcs += static_cast<int64_t>(s_arc[q]);
    sc[ST_PROCESSED] = s_proc;
    sc[ST_AFFECTED] = s_proc;
    sc[ST_ARCS] = arcs;
    ctr[CTR_T_MOVE] = static_cast<int64_t>(wall_clock64());
  }
}

template <class W, class E>
Upd<W> upd(const E& del, const E& ins) {
  return Upd<W>{del.u, del.v, del.w, del.count, ins.u, ins.v, ins.w, ins.count};
}

// Workgroups that clear the bitmasks beside the head.
unsigned clear_blocks(int64_t words) {
  return 1u + static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>((words + 4 * kSB - 1) / (4 * kSB), 512)));
}

}  // namespace

void launch_small_batch_f(const lv_graph_f& g, const lv_edges_f& del, const lv_edges_f& ins, const BatchScratch& b,
                          int64_t* ctr, hipStream_t st) {
  const Upd<float> U = upd<float>(del, ins);
  hipLaunchKernelGGL(k_small_head<float>, dim3(1), dim3(kSB), 0, st, U, 1, g.n, g.row_start, g.row_len, b, ctr, nullptr,
                     nullptr, nullptr, nullptr, 0);
  launch_batch_scan(g.row_start, g.col, del.count + ins.count, b, ctr, st);
  hipLaunchKernelGGL((k_small_edit<float, double>), dim3(1), dim3(kSB), 0, st, U, g.row_start, g.row_len, g.col, g.w,
                     g.two_m, 0, b, ctr);
}

void launch_small_batch(const lv_graph& g, const lv_edges& del, const lv_edges& ins, const BatchScratch& b,
                        int64_t* ctr, hipStream_t st) {
  const Upd<int32_t> U = upd<int32_t>(del, ins);
  hipLaunchKernelGGL(k_small_head<int32_t>, dim3(1), dim3(kSB), 0, st, U, 1, g.n, g.row_start, g.row_len, b, ctr,
                     nullptr, nullptr, nullptr, nullptr, 0);
  launch_batch_scan(g.row_start, g.col, del.count + ins.count, b, ctr, st);
  hipLaunchKernelGGL((k_small_edit<int32_t, int64_t>), dim3(1), dim3(kSB), 0, st, U, g.row_start, g.row_len, g.col,
                     g.w, g.two_m, 1, b, ctr);
}

void launch_small_df(const lv_graph& g, const lv_edges& del, const lv_edges& ins, const BatchScratch* b,
                     const lv_state& s, Workspace& ws, bool bin, int32_t wave_max, hipStream_t st) {
  const Upd<int32_t> U = upd<int32_t>(del, ins);
  const BatchScratch none{};
  const int32_t edit = b != nullptr && U.nd + U.ni > 0 ? 1 : 0;
  hipLaunchKernelGGL(k_small_head<int32_t>, dim3(clear_blocks(ws.words)), dim3(kSB), 0, st, U, edit, g.n, g.row_start,
                     g.row_len, edit ? *b : none, ws.ctr, ws.fr_a, ws.fr_b, ws.ever, ws.moved, ws.words);
  if (edit) launch_batch_scan(g.row_start, g.col, U.nd + U.ni, *b, ws.ctr, st);
  SmallDf df;
  df.C = s.C;
  df.K = s.K;
  df.Sigma = s.Sigma;
  df.fr = ws.fr_a;
  df.fl = front_list(ws, 0);
  df.ever = ws.ever;
  df.bin = bin ? 1 : 0;
  df.wave_max = wave_max;
  for (int k = 0; k < NBINS; ++k) df.list[k] = ws.bins[k];
  df.hub = HubOut{ws.hub_off, ws.hub_cbase, ws.hub_cnum, ws.u_ins_b, ws.u_ins_a, ws.u_emit_b, ws.u_emit_s};
  df.hub_kid = ws.hub_kid;
  hipLaunchKernelGGL(k_small_tail, dim3(1), dim3(kSB), 0, st, U, edit, g.n, g.row_start, g.row_len, g.col, g.w,
                     g.two_m, edit ? *b : none, ws.ctr, df);
}

}  // namespace lv
