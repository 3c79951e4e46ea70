// The miss fetch's device code: entries listed by the bookkeeping go from the pinned host pool to their slots, read by
// address.  Shared by the fetch kernel and by the attention kernels whose launch carries a fetch (ess_fetch).
#pragma once
#include "ess_internal.h"
#include "select_common.h"

namespace ess_fill {

// exclusive prefix sum of the per-sequence miss counts, pref[0 .. B] in LDS: by the first wave, ends with a barrier
__device__ __forceinline__ int prefix(const int32_t* __restrict__ miss_cnt, int fill_cap, int B, int32_t* pref) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid < 64) {
    int run = 0;
    for (int b0 = 0; b0 <= B; b0 += 64) {
      const int b = b0 + lane;
      const int cnt = b < B ? min(miss_cnt[b], fill_cap) : 0;
      const int inc = (int)ess_sel::wave_incl_scan((uint32_t)cnt, lane);
      if (b <= B) pref[b] = run + inc - cnt;
      run += __shfl(inc, 63, 64);
    }
  }
  __syncthreads();
  return pref[B];
}

// source and destination of the r-th entry of the flattened list
__device__ __forceinline__ void locate(const ess_fetch& f, const int32_t* pref, int r, const uint4*& src, uint4*& dst) {
  int lo = 0, hi = f.B;                                      // largest b with pref[b] <= r
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pref[mid] <= r) lo = mid; else hi = mid;
  }
  const int i = r - pref[lo];
  const int tok = f.fill_tok[(size_t)lo * f.fill_cap + i], slot = f.fill_slot[(size_t)lo * f.fill_cap + i];
  src = reinterpret_cast<const uint4*>(f.host_pool + ((size_t)lo * f.Lmax + tok) * f.row_stride);
  dst = reinterpret_cast<uint4*>(f.slot_pool + ((size_t)lo * f.S + slot) * f.row_stride);
}

// Every F entries of wave gw's share are in flight together (waves gw = 0 .. n_waves - 1 in all).  A whole workgroup calls.
template <int F>
__device__ __forceinline__ void entries(const ess_fetch& f, int32_t* pref, int gw, int n_waves) {
  const int M = prefix(f.miss_cnt, f.fill_cap, f.B, pref), lane = threadIdx.x & 63;
  const int chunks = f.row_stride >> 4;                      // <= 128 for the supported entry sizes
  const int c0 = lane, c1 = lane + 64;
  for (int r = gw; r < M; r += F * n_waves) {
    const uint4* src[F];
    uint4* dst[F];
    uint4 a[F], b[F];
#pragma unroll
    for (int u = 0; u < F; ++u) locate(f, pref, min(r + u * n_waves, M - 1), src[u], dst[u]);      // (past the end: the last entry once more, not stored)
#pragma unroll
    for (int u = 0; u < F; ++u) {
      if (c0 < chunks && r + u * n_waves < M) a[u] = src[u][c0];
      if (c1 < chunks && r + u * n_waves < M) b[u] = src[u][c1];
    }
#pragma unroll
    for (int u = 0; u < F; ++u) {
      if (c0 < chunks && r + u * n_waves < M) ess_store_nt(dst[u] + c0, a[u]);
      if (c1 < chunks && r + u * n_waves < M) ess_store_nt(dst[u] + c1, b[u]);
    }
  }
}

}  // namespace ess_fill
