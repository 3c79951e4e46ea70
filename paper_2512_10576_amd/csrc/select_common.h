// Pieces shared by the kernels of the selection (top-k, and the sampled lower bound of the fused selection).
#pragma once
#include "ess_internal.h"
#include <math.h>
#include <type_traits>

namespace ess_sel {

constexpr int CAND_CAP = 8192;             // candidate keys a row's list (and the LDS of the finishing kernel) holds
constexpr int HBITS = 11;                  // digits of a radix or of an even spread
constexpr int NBINS = 1 << HBITS;
// Keys of one digit that are counted at once; of more the digit is spread again: 200 equal scores counted / spread 10.2 / 11.0 us in a row of 8000, 12.7 /
// 14.7 in one of 12000; 900 34.8 / 11.1 and 38.6 / 17.4.
constexpr uint32_t FEW = 320;
constexpr uint32_t SMALL = 1024;           // keys of one digit that are counted at all
constexpr int NARROW = 3;                  // times a whole row's spread is narrowed to the digit that holds the k-th largest

// Scores between lo and hi spread evenly over the digits 1 .. 2046; below lo, -inf and what is no number: 0 or 1; above hi: up
// to 2047.  Monotone in the score, four instructions.  scale 0: the range gives no such digits.  (Ends past 1.6e38 are taken in,
// so that their distance is a number.)
// (Reciprocals and roots to the last bit but one, in an instruction where the exact ones take a dozen: a kernel that others have pushed out
// of the instruction cache waits for every line of its code.)
__host__ __device__ __forceinline__ float quick_rcp(float x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
__host__ __device__ __forceinline__ float quick_sqrt(float x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_sqrtf(x);
#else
  return sqrtf(x);
#endif
}
struct Spread {
  float lo, scale, step;                     // step: of a digit
  __host__ __device__ __forceinline__ Spread(float lo_, float hi_) : lo(fmaxf(lo_, -1.6e38f)) {
    const float span = fminf(hi_, 1.6e38f) - lo;
    step = span * (1.0f / (float)(NBINS - 3));
    scale = span > 1e-30f ? quick_rcp(step) : 0.f;
  }
  __host__ __device__ __forceinline__ uint32_t digit(float v) const {
#ifdef __HIP_DEVICE_COMPILE__
    return (uint32_t)__builtin_amdgcn_fmed3f(fmaf(v - lo, scale, 1.0f), 0.f, (float)(NBINS - 1));
#else
    return (uint32_t)fminf(fmaxf(fmaf(v - lo, scale, 1.0f), 0.f), (float)(NBINS - 1));
#endif
  }
  // a score that no score of digit d or above lies below (a hundredth of a digit covers the rounding of `digit`)
  __host__ __device__ __forceinline__ float edge(uint32_t d) const { return fmaf((float)d - 1.01f, step, lo); }
};

// Samples of a row above CAND_CAP positions: blocks of 16 scores, at most this many blocks; twice as many where more than 2048 are to be
// found beyond 262144 positions: with the fewer a list of 4096 at 300000 positions missed its size in one row of fifty.
constexpr int SAMPLE_TARGET = 4096;
__host__ __device__ inline int sample_blocks(int k, int vis) { return (k > 2048 && vis > 262144 ? 2 : 1) * SAMPLE_TARGET / 16; }
// A row's list takes the positions whose score reaches that of the t-th largest of its samples, `per` of them to a score; it must hold at least
// the k largest and at most CAND_CAP.  t: a quarter and about four standard deviations above the number of samples that are expected
// among the k largest (a sample of blocks is no random one, and a list that turns out too short costs the row a multiple of its time; the
// quarter makes the usual list 4 % more expensive), but not past the middle between that number and the one that a full list stands for:
// there both ends are more than three deviations away with k 4096 and 64 scores a sample.  (Without the middle every row of 4096 past 131072 positions
// asked for more than fits.)
__host__ __device__ inline uint32_t sample_target(int k, float per) {
  const float expct = (float)k * per;
  return (uint32_t)fmaxf(fminf(1.25f * expct + 4.0f * quick_sqrt(expct) + 8.0f, 0.47f * (expct + (float)CAND_CAP * per)), 1.0f);
}

// Inclusive prefix sum over the 64 lanes of a wave, by data-parallel-primitive moves inside the vector ALU (seven
// adds; the same through ds_bpermute is six dependent trips through the LDS crossbar): sums of 4 neighbours inside
// each row of 16 lanes (row_shr 1, 2, 3), of 8 and 16 (row_shr 4 and 8 on the banks that have such neighbours), then
// lane 15 of a row added to the next row (row_bcast 15, rows 1 and 3) and lane 31 to the upper half (row_bcast 31).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int /*lane*/) {
  const int x = (int)v;
  int r = x + __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, r, 0x114, 0xf, 0xe, true);
  r += __builtin_amdgcn_update_dpp(0, r, 0x118, 0xf, 0xc, true);
  r += __builtin_amdgcn_update_dpp(0, r, 0x142, 0xa, 0xf, false);
  r += __builtin_amdgcn_update_dpp(0, r, 0x143, 0xc, 0xf, false);
  return (uint32_t)r;
}

// Largest value of the wave's 64 lanes (STEPS 6), or of its last eight (STEPS 3), in all lanes, by the same moves.  A NaN is skipped.
template <int STEPS>
__device__ __forceinline__ float wave_max(float x) {
  constexpr int kLow = (int)0xff800000;
  auto with = [&](auto ctrl, auto rows) {
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(kLow, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
  };
  using std::integral_constant;
  with(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  if constexpr (STEPS > 3) {
    with(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    with(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    with(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
  }
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// The inclusive prefix sum inside each row of 16 lanes.
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v) {
  const int x = (int)v;
  int r = x + __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xf, 0xf, true);
  r += __builtin_amdgcn_update_dpp(0, r, 0x114, 0xf, 0xe, true);
  r += __builtin_amdgcn_update_dpp(0, r, 0x118, 0xf, 0xc, true);
  return (uint32_t)r;
}

// Sum of the first `wave` of NW (at most 16) words of LDS, the same in all lanes; *total the sum of all: each of the first
// lanes reads one and a row scan adds them up (a dozen instructions; a sum of NW broadcast reads, each with its select, is three times that, and a wave
// alone issues one in five cycles).
template <int NW>
__device__ __forceinline__ uint32_t waves_before(const uint32_t* wave_tot, int wave, int lane, uint32_t* total = nullptr) {
  static_assert(NW <= 16, "one row of lanes");
  const int upto = (int)row_incl_scan(lane < NW ? wave_tot[lane] : 0u);
  if (total) *total = (uint32_t)__builtin_amdgcn_readlane(upto, 15);
  return wave > 0 ? (uint32_t)__builtin_amdgcn_readlane(upto, wave - 1) : 0u;
}

// inclusive scan over the NTH threads of the workgroup in thread order; *total gets the sum
template <int NTH>
__device__ __forceinline__ uint32_t block_incl_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t inc = wave_incl_scan(v, lane);
  __syncthreads();                         // wave_tot may still be read from a previous call
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  const uint32_t off = waves_before<NTH / 64>(wave_tot, wave, lane, total);
  return inc + off;
}

}  // namespace ess_sel
