// Device helpers of the batch edit, shared by its two forms: the grid-wide
// kernels of batch.hip and the one-workgroup kernels of small.hip.
#pragma once

#include "lv_internal.hpp"

namespace lv {
namespace {

constexpr uint64_t kEmpty = ~0ull;
constexpr int kChunk = 1024;        // arcs per scan unit (one wavefront)
constexpr int kFilterBits = 4096;   // per-wavefront partner filter
constexpr int kScanWaves = kBlock / kWave;

__device__ __forceinline__ uint64_t canon(int32_t a, int32_t b) {
  const uint32_t lo = static_cast<uint32_t>(min(a, b)), hi = static_cast<uint32_t>(max(a, b));
  return (static_cast<uint64_t>(lo) << 32) | hi;
}

__device__ __forceinline__ uint32_t hash64(uint64_t key, uint32_t mask) {
  key ^= key >> 33;
  key *= 0xff51afd7ed558ccdull;
  key ^= key >> 33;
  return static_cast<uint32_t>(key) & mask;
}

// Endpoints of direction e: directions 2k, 2k+1 belong to deletion k
// (k < nd), then 2(nd + k), 2(nd + k) + 1 to insertion k.  Direction
// 2k is the arc u -> v, 2k + 1 the arc v -> u.
// W: int32_t, or float (the paper's precision).
template <class W>
struct Upd {
  const int32_t *du, *dv;
  const W* dw;
  int64_t nd;
  const int32_t *iu, *iv;
  const W* iw;
  int64_t ni;
  __device__ __forceinline__ bool is_del(int64_t e) const { return e < 2 * nd; }
  __device__ __forceinline__ int64_t update(int64_t e) const { return e >> 1; }  // index into [del | ins]
  __device__ __forceinline__ void ends(int64_t e, int32_t& a, int32_t& c) const {
    const int64_t k = e >> 1;
    const int32_t x = k < nd ? du[k] : iu[k - nd];
    const int32_t y = k < nd ? dv[k] : iv[k - nd];
    a = (e & 1) ? y : x;
    c = (e & 1) ? x : y;
  }
  __device__ __forceinline__ W weight(int64_t e) const {
    const int64_t k = e >> 1;
    return k < nd ? dw[k] : iw[k - nd];
  }
};

__device__ __forceinline__ bool usable(int32_t x) { return x > 0; }
__device__ __forceinline__ bool usable(float x) { return isfinite(x) && x > 0.0f; }

// Weight totals: whole numbers, or FP64 sums in the same counter slots.
__device__ __forceinline__ int64_t as_total(int32_t x) { return x; }
__device__ __forceinline__ double as_total(float x) { return static_cast<double>(x); }
__device__ __forceinline__ double block_total(double v, double* lds) {
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  if (lane_id() == 0) lds[threadIdx.x / kWave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kBlock / kWave; ++w) t += lds[w];
  __syncthreads();
  return t;
}
__device__ __forceinline__ int64_t block_total(int64_t v, int64_t* lds) { return block_sum(v, lds); }
__device__ __forceinline__ void total_add(int64_t* sc, int st, int64_t v) { stat_add(sc, st, v); }
__device__ __forceinline__ void total_add(int64_t* sc, int st, double v) {
  atomicAdd(reinterpret_cast<double*>(&sc[(blockIdx.x % kStatReplicas) * kStatStride + st]), v);
}
template <class T>
__device__ __forceinline__ T total_of(const int64_t* sc, int st) {
  T v = 0;
  for (int r = 0; r < kStatReplicas; ++r) v += reinterpret_cast<const T*>(sc)[r * kStatStride + st];
  return v;
}

}  // namespace
}  // namespace lv
