// Stage 2: per-query top-k over the indexer scores (ESS paper Sec. 3: the top
// 2,048 entries are selected).
//
// Selection order is (score descending, position ascending).  Every position
// gets a unique composite key  c = orderable_u32(score) << IB | (2^IB-1 - pos)
// (IB = bits needed for a position), so "the k largest composite keys" is a
// total order with no ties and any selection algorithm gives the same set.
//
// One workgroup per (b,t) row finds the threshold key T* = the k-th largest
// composite key, then emits every position whose key is >= T*:
//   A. long rows: a histogram of a sample of the scores gives a score that is
//      below the k-th largest with high probability yet keeps only a few
//      thousand positions at or above it; one pass over the row collects those
//      candidates in LDS.  If their number is not in
//      [k, buffer size] (an unlucky sample, massive ties) path B runs instead.
//   S. rows that fit the candidate buffer whole: all keys in registers, no list.
//   B. general: MSD radix narrowing on the composite key straight from memory,
//      11 bits a pass (histogram in 8 interleaved copies, copy = lane & 7, so
//      that lanes hitting one hot bin do not serialise), until the positions
//      matching the decided prefix fit the buffer; one pass collects them.
//   C. A and S: one histogram spread evenly over the candidates' scores, the
//      digit that holds the k-th spread again while it is too full, and
//      counting inside it; B: radix select inside LDS over the candidates.
//   D. positions leave in ascending order, each for its rank among the selected
//      (a counting sort), so the output is ordered and deterministic.
// Row passes keep several 16-byte loads per thread in flight; a workgroup that
// issued one load per thread and round would crawl at memory latency.
#include "index_tile.h"
#include "select_common.h"
#include <mutex>

namespace {

// Eight waves, two per SIMD: an instruction of sixteen takes 16 cycles, and the phases that do not depend on the row's length --
// scans, reductions, barriers -- are most of the kernel.  us a call, before (sixteen waves, a digit pass over 64-bit keys, positions read back
// from a bitmap word by word) / now, k 2048: 1 row of 8000 10.4 / 7.1, 32 rows of 4096 13.1 / 7.5, 13 of 16384 13.9 / 10.6, 32 of
// 32768 15.1 / 11.4, 46 of 40000 16.8 / 12.6, 20 of 65000 18.7 / 13.4, 4 of 131072 16.3 / 12.3, 64 of 115000 21.5 / 17.8.
constexpr int NT = 512;
constexpr int COPIES = 8;
using ess_sel::CAND_CAP;
using ess_sel::FEW;
using ess_sel::HBITS;
using ess_sel::NARROW;
using ess_sel::NBINS;
using ess_sel::SMALL;
using ess_sel::Spread;
constexpr int FAST_MIN_VIS = CAND_CAP + 1;   // rows above the candidate list's size are sampled (path A)
constexpr int PER = CAND_CAP / NT;           // keys per thread of a row or a list that is held in registers
constexpr int LIST_AHEAD = 3072 / NT;        // rounds of NT list entries that are asked for before their number is known
constexpr int ROUND = 8;                     // float4s per thread and round of a pass over a row
constexpr int DPT = NBINS / NT;              // digits per thread of a scan over a digit histogram
constexpr int RANK_WORDS = NBINS * 4;        // words of a row's bitmap up to which the words' ranks fit beside it (262144 positions)
static_assert(PER * (NT / 64) == 128 && DPT == 4, "two counts a lane; digits are read 16 bytes at a time");
constexpr uint32_t NONE = 0xffffffffu, ABOVE = NONE - 1u;     // in place of a digit: no key, or one that is not taken; one that is
constexpr uint32_t ROW_DONE = 0xffffffffu;   // in place of a candidate count: the candidate pass did the row itself

// what bounds_of needs (all that k_index_tau holds)
struct __align__(16) BoundsShared {
  uint32_t lhist[NBINS];                  // 8 KiB: digit histogram of the candidates, or of a sample
  uint32_t wave_tot[NT / 64];
  uint32_t sel_digit, sel_above, sel_count;
  uint32_t sbin[2];                       // bounds_of: the digits of its two bounds
  float red_lo[NT / 64], red_hi[NT / 64], probe[64];       // value_range: extremes of the waves' scores, and 64 of them
};

struct TopkShared : BoundsShared {
  union __align__(16) {
    uint32_t hist[NBINS * COPIES];        // 64 KiB
    unsigned long long cand[CAND_CAP];    // 64 KiB
  };
  union {
    int32_t out_list[ESS_MAX_TOPK];       // 16 KiB
    struct {
      unsigned long long few[SMALL + 8];  // the keys of one digit (read eight at a time)
      uint32_t few_rank[SMALL];           // how many of them are larger
    };
  };
  unsigned long long red_and[NT / 64], red_or[NT / 64];
  uint32_t out_n, cand_n;
  __align__(16) float stage[4 * ROUND * NT];               // 64 KiB: a round of a pass over a row
  uint32_t few_bits[CAND_CAP / 32];       // whole_row: positions taken of the crossing digit
  uint32_t taken[PER * (NT / 64)];        // whole_row: positions taken of every 64, in ascending order
};

__device__ __forceinline__ uint32_t orderable(float v) { return ess_orderable(v); }

using ess_sel::wave_incl_scan;
__device__ __forceinline__ uint32_t block_incl_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total) {
  return ess_sel::block_incl_scan<NT>(v, wave_tot, total);
}

// append `val` for lanes with pred, one LDS atomic per wave; entries past `cap` are counted, not stored
template <typename V>
__device__ __forceinline__ void wave_append(bool pred, V val, V* list, uint32_t* counter, uint32_t cap = 0xffffffffu) {
  const unsigned long long mask = __ballot(pred);
  if (mask == 0) return;
  const int lane = threadIdx.x & 63;
  uint32_t base = 0;
  const int leader = __ffsll((long long)mask) - 1;
  if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(mask));
  base = __shfl(base, leader, 64);
  const uint32_t pos = base + __popcll(mask & ((1ull << lane) - 1ull));
  if (pred && pos < cap) list[pos] = val;
}

// Calls f(position, score, valid) for every position of the row, by all threads the same number of
// times (f may hold wave-wide operations).  Each thread has four 16-byte loads in flight per round,
// which is what makes one workgroup able to pull a 512 KiB row at cache bandwidth, not at latency.
template <typename F>
__device__ __forceinline__ void scan_row(int tid, const float* srow, int vis, bool vec_ok, F&& f) {
  constexpr int U = 4;
  int done = 0;
  if (vec_ok) {
    const int nvec = vis >> 2;
    const float4* v4 = reinterpret_cast<const float4*>(srow);
    for (int base = 0; base < nvec; base += NT * U) {
      float4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = base + u * NT + tid;
        x[u] = j < nvec ? v4[j] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = base + u * NT + tid;
        const bool ok = j < nvec;
        f(4 * j + 0, x[u].x, ok);
        f(4 * j + 1, x[u].y, ok);
        f(4 * j + 2, x[u].z, ok);
        f(4 * j + 3, x[u].w, ok);
      }
    }
    done = nvec << 2;
  }
  for (int i0 = done; i0 < vis; i0 += NT) {
    const int i = i0 + tid;
    const bool ok = i < vis;
    f(i, ok ? srow[i] : 0.f, ok);
  }
}

// The positions of a row (or a slice of it) whose score reaches tau, as (position, score) pairs in LDS: `raw`, *n_raw of them,
// of which CAND_CAP have room.  Rounds of 32 positions a thread: the scores go to LDS as they are, and a bit per position says
// which reach tau (three instructions each); a lane then writes its few positions one after the other, and the wave fetches
// their scores densely.  (A predicated write per position, 32 of them with a tenth of the lanes each, took 5 k cycles per 16K
// positions; 3.3 k now.)  The loads of the first SETS rounds are issued by row_begin, before tau is known: one CU
// pulls a row at 33 GB/s, a 32K row in about the time the threshold takes.  Indices past the end are
// clamped, not predicated, so that every load is unconditional.  A row may start at any multiple of four bytes: its first
// positions up to a 16-byte boundary and its last ones, at most six, come by themselves.
__device__ __forceinline__ int to_boundary(const float* p) { return (int)((0u - (uint32_t)(reinterpret_cast<uintptr_t>(p) >> 2)) & 3u); }
typedef float float4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void row_load(int tid, const float* srow, int n, int base, float4v (&x)[ROUND]) {
  const float4v* v4 = reinterpret_cast<const float4v*>(srow);
#pragma unroll
  for (int g = 0; g < ROUND; ++g) x[g] = v4[max(min(base + g * NT + tid, (n >> 2) - 1), 0)];
}
template <int SETS>
__device__ __forceinline__ void row_begin(int tid, const float* srow, int n, float4v (&x)[SETS][ROUND]) {
#pragma unroll
  for (int s = 0; s < SETS; ++s) row_load(tid, srow, n, s * ROUND * NT, x[s]);
}
template <int SETS>
__device__ __forceinline__ void collect(int tid, const float* srow, int first, int n, float4v (&x)[SETS][ROUND], float tau,
                                        uint2* raw, uint32_t* n_raw, float* stage) {
  const int lane = tid & 63, head = to_boundary(srow), nvec = (n - head) >> 2;      // (n is at least 1021)
  auto round = [&](int base, float4v (&y)[ROUND]) {
    float4v* const st4 = reinterpret_cast<float4v*>(stage);
    uint32_t hits = 0;                       // position 4 g + e of the thread's 32: bit 31 - (4 g + e)
#pragma unroll
    for (int g = 0; g < ROUND; ++g) {
      st4[g * NT + tid] = y[g];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hits = (hits << 1) | (y[g][e] >= tau ? 1u : 0u);
        asm volatile("" : "+v"(hits));       // (one at a time: left alone, the bits are packed in a tree)
      }
    }
    // groups past the end hold the last one's scores again
    const int groups = min(max((nvec - base - tid + NT - 1) / NT, 0), ROUND);
    hits &= groups == ROUND ? 0xffffffffu : ~(0xffffffffu >> (4 * groups));
    if (base + SETS * ROUND * NT < nvec) row_load(tid, srow + head, n - head, base + SETS * ROUND * NT, y);
    const uint32_t cnt = __popc(hits), inc = wave_incl_scan(cnt, lane), sum = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    if (sum == 0) return;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(n_raw, sum);
    const uint32_t from = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (from + sum > (uint32_t)CAND_CAP) return;              // too many: the list is not used
    at = from + inc - cnt;
    while (hits) {
      const uint32_t i = (uint32_t)__builtin_clz(hits);
      hits &= ~(0x80000000u >> i);
      raw[at++].x = 4u * ((i >> 2) * NT + (uint32_t)tid) + (i & 3u);
    }
    // (a wave reads what its own lanes wrote: nothing may be moved across)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t j = from + lane; j < from + sum; j += 64) {
      const uint32_t i = raw[j].x;
      raw[j] = make_uint2((uint32_t)(first + head + 4 * base) + i, __float_as_uint(stage[i]));
    }
    __builtin_amdgcn_wave_barrier();
  };
  for (int base = 0; base < nvec; base += SETS * ROUND * NT) {
    round(base, x[0]);
    if constexpr (SETS == 2)
      if (base + ROUND * NT < nvec) round(base + ROUND * NT, x[SETS - 1]);
  }
  if (tid < 64) {
    const int i = tid < head ? tid : 4 * nvec + tid;         // (behind the head come the vectors)
    const float s = i < n ? srow[i] : 0.f;
    wave_append<uint2>(i < n && s >= tau, make_uint2((uint32_t)(first + i), __float_as_uint(s)), raw, n_raw, CAND_CAP);
  }
}

// D, second half: the positions marked in the bitmap bmp[0..W), in ascending order, to orow[0..k)
__device__ __forceinline__ void emit_bitmap(TopkShared& sm, int tid, const uint32_t* bmp, int W, int k, int32_t* __restrict__ orow) {
  const int wpt = (W + NT - 1) / NT;
  const int w0 = min(tid * wpt, W), w1 = min(w0 + wpt, W);
  uint32_t mine = 0;
  for (int wd = w0; wd < w1; ++wd) mine += __popc(bmp[wd]);
  uint32_t total;
  uint32_t outp = block_incl_scan(mine, sm.wave_tot, &total) - mine;
  for (int wd = w0; wd < w1; ++wd) {
    uint32_t bits = bmp[wd];
    while (bits) {
      const int bit = __ffs(bits) - 1;
      bits &= bits - 1;
      if (outp < (uint32_t)k) orow[outp] = wd * 32 + bit;
      ++outp;
    }
  }
}

// A running sum over four counts starts at `above`, below need: the index of the count that takes it to need or beyond, with the sum in front of it
// in `above` and with it in `upto`.  (Selects: with a branch a count this was three times the code.)
__device__ __forceinline__ uint32_t crossing_of(const uint32_t (&cnt)[DPT], uint32_t need, uint32_t& above, uint32_t& upto) {
  static_assert(DPT == 4, "written for four");
  const uint32_t s0 = above + cnt[0], s1 = s0 + cnt[1], s2 = s1 + cnt[2], s3 = s2 + cnt[3];
  const bool p0 = s0 < need, p1 = s1 < need, p2 = s2 < need;
  above = p2 ? s2 : (p1 ? s1 : (p0 ? s0 : above));
  upto = p2 ? s3 : (p1 ? s2 : (p0 ? s1 : s0));
  return (p0 ? 1u : 0u) + (p1 ? 1u : 0u) + (p2 ? 1u : 0u);
}

// Which of the 2048 digits of the histogram sm.lhist contains the need-th largest key, counted
// from the top: sm.sel_digit, with sm.sel_above keys above it and sm.sel_count in it.  Ends with a barrier.
// all: the number of keys, those of digit 0 need not be in the histogram then.
__device__ __forceinline__ void crossing_digit(TopkShared& sm, int tid, uint32_t need, uint32_t all = 0u) {
  const int d0 = NBINS - DPT - DPT * tid;      // thread tid owns four digits, descending
  const uint4 h = *reinterpret_cast<const uint4*>(&sm.lhist[d0]);
  const uint32_t cnt[DPT] = {h.w, h.z, h.y, h.x};
  const uint32_t mine = h.x + h.y + h.z + h.w;
  uint32_t total;
  uint32_t above = block_incl_scan(mine, sm.wave_tot, &total) - mine;
  if (above < need && above + mine >= need) {
    uint32_t upto;
    const uint32_t i = crossing_of(cnt, need, above, upto);
    sm.sel_digit = (uint32_t)(d0 + DPT - 1) - i; sm.sel_above = above; sm.sel_count = upto - above;
  }
  if (all != 0u && total < need && tid == 0) { sm.sel_digit = 0u; sm.sel_above = total; sm.sel_count = all - total; }
  __syncthreads();
}

// Extremes of the workgroup's values (+inf and -inf where a thread has none), the same in all threads.  One barrier.
__device__ __forceinline__ void value_range(BoundsShared& sm, int tid, float& lo, float& hi) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lo = -ess_sel::wave_max<6>(-lo);
  hi = ess_sel::wave_max<6>(hi);
  if (lane == 0) { sm.red_lo[wave] = lo; sm.red_hi[wave] = hi; }
  __syncthreads();
  lo = -ess_sel::wave_max<3>(-sm.red_lo[lane & (NT / 64 - 1)]);
  hi = ess_sel::wave_max<3>(sm.red_hi[lane & (NT / 64 - 1)]);
}

// The spread of a set of scores of which the one with `share` of the set at or above it is looked for; lo, hi: a thread's
// extremes of the finite ones; probe: one of them, or NaN (64 are looked at).  Between their extremes, unless of 64 pairs of probes four
// share a digit then -- an outlier far away, a mask of the lowest number, magnitudes apart --: between two probes in whose middle, by
// rank, the one looked for is expected; what lies outside is in the end digits.  All threads find the same.  One barrier.
__device__ __forceinline__ Spread spread_of(BoundsShared& sm, int tid, float lo, float hi, float probe, float share) {
  constexpr float kInf = __builtin_inff();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (lane < 64 / (NT / 64)) sm.probe[wave * (64 / (NT / 64)) + lane] = probe;         // eight lanes' worth of each wave's, one to a lane
  value_range(sm, tid, lo, hi);
  probe = sm.probe[lane];
  const Spread sp(lo, hi);
  const uint32_t d = sp.digit(probe);
  const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d, 0x121, 0xf, 0xf, true);      // (the lane beside, in a ring of 16)
  if (__builtin_expect(__popcll(__ballot(d == next)) < 4, 1)) return sp;
  uint32_t larger = 0;                       // of 32 probes, how many are larger than the lane's
#pragma unroll
  for (int j = 0; j < 32; ++j)
    larger += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(probe), 4 * (j >> 1) + (j & 1))) > probe ? 1u : 0u;
  const float rank = share * 0.5f * (float)__popcll(__ballot(probe == probe)), at = (float)larger;
  const bool fin = fabsf(probe) < kInf;
  const float below = ess_sel::wave_max<6>(fin && at >= rank + 6.0f ? probe : -kInf), over = -ess_sel::wave_max<6>(fin && at <= rank - 6.0f ? -probe : -kInf);
  const Spread finer(below > -kInf ? below : lo, over < kInf ? over : hi);
  return finer.scale == 0.f ? sp : finer;
}

__device__ __forceinline__ float score_of(uint32_t o) {      // the score of an ess_orderable image
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Two bounds of a row's selection from a sample of its scores (ns in all, N a thread, the u-th of a thread valid where
// u * NT + tid < ns): *tau, a score at or above which very probably lie the k largest and not many more (see sample_target), and
// *tau_hi, one at or above which lie about an eighth of those: a list spread between the two has few keys a digit near tau, and
// its last digit is not crowded either (adds to one address pass one after the other: with the fewest that are surely taken, half of all, in the last
// digit that pass took 3.3 k cycles instead of 1.6).
// The sample is spread evenly over the digits from the smallest of the threads' largest finite samples (with k below a third of the row the bound lies above it; what
// lies below, half of the sample or a mask of the lowest number, need not be counted) to the second largest of the waves' (one outlier is not among them).  Where the
// digit of the bound is still too full for the list, its samples alone are spread again, like the keys of a whole row.
// us, k 2048, of a form with the top 14 bits of the float as digits and sixteen waves, of an even spread between the extremes with those bits behind it, and of this.
// 1 x 12000: as they come 12.8 / 10.4 / 10.3, one score 1e30 12.8 / 16.3 / 9.8, a fifth masked 12.2 / 15.7 / 10.3, 70 % masked 13.6 / 19.6 / 17.1;
// 64 x 115000: 21.3 / 17.7 / 17.5, 21.4 / 24.7 / 17.8, 21.4 / 23.9 / 17.7, 22.9 / 25.4 / 20.4.
// False: no bounds: nothing finite to go by, or (*tau == *tau_hi then) more equal scores than a list holds.
// sm.lhist must be clear and sm.sbin 0xffffffff once a barrier has passed.
template <int N>
__device__ __forceinline__ bool bounds_of(BoundsShared& sm, int tid, const float (&sv)[N], int ns, int k, int vis, float* tau, float* tau_hi) {
  constexpr float kInf = __builtin_inff(), kMost = 3.4028235e38f;
  float lo = kInf, hi = -kInf;               // of a thread's finite samples
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const bool fin = u * NT + tid < ns && fabsf(sv[u]) < kInf;
    lo = fminf(lo, fin ? sv[u] : kInf);
    hi = fmaxf(hi, fin ? sv[u] : -kInf);
  }
  if (3 * k < vis && hi > -kInf) lo = hi;
  value_range(sm, tid, lo, hi);
  const float x = sm.red_hi[tid & (NT / 64 - 1)], second = ess_sel::wave_max<3>(x == hi ? -kInf : x);
  auto beyond = [](float v) { return v + fmaxf(fabsf(v) * 1e-6f, 1e-29f); };
  Spread sp(lo, fmaxf(second > -kInf ? second : hi, beyond(lo)));
  if (sp.scale == 0.f) return false;         // nothing finite, or scores past 1.6e38 alone
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t du = sp.digit(sv[u]);
    if (u * NT + tid < ns && du != 0u) atomicAdd(&sm.lhist[du], 1u);
  }
  const float per = (float)ns * ess_sel::quick_rcp((float)vis), room = (float)CAND_CAP * per;         // room: the samples that a full list stands for
  uint32_t need[2] = {ess_sel::sample_target(k, per), max((uint32_t)(0.125f * (float)k * per), 1u)};
  __syncthreads();
  // the digits of the need[0]-th and the need[1]-th largest of `all`: sm.sbin; of the first also how many lie above and in it
  auto search = [&](uint32_t all) {
    const int d0 = NBINS - DPT - DPT * tid;
    const uint4 h = *reinterpret_cast<const uint4*>(&sm.lhist[d0]);
    const uint32_t cnt[DPT] = {h.w, h.z, h.y, h.x};
    const uint32_t mine = h.x + h.y + h.z + h.w;
    uint32_t total;
    const uint32_t inc = block_incl_scan(mine, sm.wave_tot, &total);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      uint32_t above = inc - mine;
      if (above < need[w] && inc >= need[w]) {
        uint32_t upto;
        sm.sbin[w] = (uint32_t)(d0 + DPT - 1) - crossing_of(cnt, need[w], above, upto);
        if (w == 0) { sm.sel_above = above; sm.sel_count = upto - above; }
      }
      if (tid == 0 && total < need[w] && all >= need[w]) {   // (those of digit 0 need not be in the histogram)
        sm.sbin[w] = 0u;
        if (w == 0) { sm.sel_above = total; sm.sel_count = all - total; }
      }
    }
    __syncthreads();
  };
  search((uint32_t)ns);
  uint32_t b0 = sm.sbin[0], b1 = sm.sbin[1], above = sm.sel_above;
  uint32_t reach = above + sm.sel_count;     // samples that reach digit b0
  if (__builtin_expect(b0 - 1u < NONE - 1u && (float)reach < 0.9f * room, 1)) {
    *tau = sp.edge(b0);
    *tau_hi = sp.edge(b1 + 1);
    return *tau_hi > *tau;
  }
  if (b0 == NONE) return false;              // fewer samples than the bound asks for
  // (rare) the digit's own samples, spread again
  uint32_t d[N];
#pragma unroll
  for (int u = 0; u < N; ++u) d[u] = u * NT + tid < ns ? sp.digit(sv[u]) : NONE;
#pragma unroll 1
  for (int round = 0; round < NARROW; ++round) {
    lo = kInf;
    hi = -kInf;
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (d[u] == b0) {
        const float x = sv[u] == sv[u] ? sv[u] : -kInf;      // (as a key has it)
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
      }
    *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
    value_range(sm, tid, lo, hi);
    sp = Spread(lo, hi);
    if (sp.scale == 0.f) {                   // equal, or as good as equal
      *tau = fminf(lo, kMost);
      *tau_hi = (float)reach < room ? beyond(*tau) : *tau;
      return *tau >= -kMost && *tau_hi > *tau;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      d[u] = d[u] == b0 ? sp.digit(sv[u]) : NONE;
      if (d[u] != NONE) atomicAdd(&sm.lhist[d[u]], 1u);
    }
    __syncthreads();
    need[0] -= above;
    need[1] = b1 == b0 ? need[1] - above : 1u;               // (or the upper bound is that of this digit)
    const uint32_t in = sm.sel_count, before = reach - in;
    search(in);
    b0 = sm.sbin[0];
    b1 = sm.sbin[1];
    above = sm.sel_above;
    reach = before + above + sm.sel_count;
    if (b0 >= 1u && ((float)reach < 0.9f * room || (round == NARROW - 1 && (float)reach < room))) {
      *tau = fmaxf(sp.edge(b0), -kMost);
      *tau_hi = fminf(sp.edge(b1 + 1), kMost);
      return *tau_hi > *tau;
    }
  }
  return false;
}

// Inside the digit that holds the k-th largest key -- a handful of keys, sm.few[0..cnt): f(key) for the `take` largest, found by
// counting.  Keys are distinct.  Up to sixteen are counted by one thread each; of more (equal scores) each key's rivals are shared
// by the threads that there are (145 keys: 15 k cycles by one thread each and one at a time, 2.5 k now).  Begins with a
// barrier; sm.few_rank must be clear once it has passed.
template <typename F>
__device__ __forceinline__ void take_few(TopkShared& sm, int tid, uint32_t cnt, uint32_t take, F&& f) {
  if (tid < 8) sm.few[cnt + tid] = 0ull;                     // (keys are read eight at a time; none is smaller than this one)
  __syncthreads();
  auto count = [&](unsigned long long my, uint32_t from, uint32_t step) {
    uint32_t above = 0;
    for (uint32_t i = from; i < cnt; i += step) {
      unsigned long long x[8];
#pragma unroll
      for (uint32_t e = 0; e < 8; ++e) x[e] = sm.few[i + e];
#pragma unroll
      for (uint32_t e = 0; e < 8; ++e) {
        above += x[e] > my ? 1u : 0u;
        asm volatile("" : "+v"(above));      // (a compare and an add with carry; left alone, bits are packed and counted)
      }
    }
    return above;
  };
  if (cnt <= 16) {
    if ((uint32_t)tid < cnt && count(sm.few[tid], 0, 8) < take) f(sm.few[tid]);
    return;
  }
  const uint32_t shares = max(NT / cnt, 1u), share = shares > 1 ? (uint32_t)tid / cnt : 0u;
  if (share < shares)
    for (uint32_t j = (uint32_t)tid - share * cnt; j < cnt; j += NT) {
      const uint32_t above = count(sm.few[j], 8 * share, 8 * shares);
      if (above) atomicAdd(&sm.few_rank[j], above);
    }
  __syncthreads();
  for (uint32_t j = tid; j < cnt; j += NT)
    if (sm.few_rank[j] < take) f(sm.few[j]);
}

// What bounds the two finishing forms below: the keys are few and everything waits for everything in front of it, so time is the
// instructions of all waves and the barriers.  A key is worth as few instructions as can be: its digit is computed once
// and kept, 64-bit keys are built for the one digit that has to be resolved, and positions leave by rank.

// A row finished from its candidate list (`listed` scores v and positions p, k <= listed <= CAND_CAP) when the k-th largest score very probably lies in [tau, tau_hi) (see bounds_of).  One
// histogram spreads that range over 2046 digits (what lies above goes into the last), the digit that holds the k-th largest
// key is found, and inside it the key by counting.  The positions taken are marked in a bitmap of the row, and each leaves
// for its rank: the positions taken in the words before, and in its word before it.
// Where that digit holds more keys than counting takes (ties, a k-th largest score outside the range), its keys alone are spread between
// their own extremes, and equal scores by their positions.  us, a row of 12000, counted or by the general selection / now: 900 equal
// scores at the k-th 38.6 / 17.4, 3000 28.7 / 25.3; 64 rows of 115000: 45.7 / 26.7, 36.1 / 32.0.
// Returns false, with the keys in sm.cand, when that did not help (or the range gives no digits): the caller goes on with the general selection.
template <int N>
__device__ __forceinline__ bool finish_rounds(TopkShared& sm, int tid, const float (&v)[PER], const uint32_t (&p)[PER], uint32_t listed,
                                            float tau, float tau_hi, int vis, int k, int IB, int32_t* __restrict__ orow) {
  const unsigned long long imask = (1ull << IB) - 1ull;
  auto key = [&](int u) {
    uint32_t low = (uint32_t)imask - p[u];
    asm volatile("" : "+v"(low));            // (where it is asked for, not by every list)
    return ((unsigned long long)orderable(v[u]) << IB) | low;
  };
  // (keys of a list may still be on their way:) clear the histogram and the row's bitmap
  uint32_t* const bmp = sm.hist;
  const int W = (vis + 31) >> 5;             // at most 16384 words
  for (int j = 4 * tid; j < W; j += 4 * NT) *reinterpret_cast<uint4*>(&bmp[j]) = make_uint4(0, 0, 0, 0);
  *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
  if (tid == 0) sm.cand_n = 0;
  const Spread sp(tau, tau_hi);
  uint32_t d[N];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < N; ++u) {
    d[u] = (uint32_t)(u * NT + tid) < listed ? sp.digit(v[u]) : NONE;
    if (d[u] != NONE) atomicAdd(&sm.lhist[d[u]], 1u);
  }
  __syncthreads();
  crossing_digit(sm, tid, (uint32_t)k);
  uint32_t dsel = sm.sel_digit, take = (uint32_t)k - sm.sel_above, cnt = sm.sel_count;
  // (rare) that digit's keys alone, spread again; equal ones by their positions (below 2^19: exact).  Through LDS, in loops that need not be
  // unrolled: a step's other kernels push this code out of the instruction cache.  Unrolled over registers it made rare rows faster (15.5 us for 900 equal
  // scores, now 18) and the finish of every list slower (32 rows of 128K 10.3 us, now 9.7; 40 of 100K in the fused selection 8.75, now 8.45).
  if (__builtin_expect(cnt > FEW && cnt != take && sp.scale != 0.f, 0)) {
    float* const value = sm.stage;
    uint32_t* const digit = reinterpret_cast<uint32_t*>(sm.stage) + CAND_CAP;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      value[u * NT + tid] = v[u];
      digit[u * NT + tid] = d[u];
    }
    bool by_position = false;
#pragma unroll 1
    for (int round = 0; round < NARROW + 2 && cnt > FEW && cnt != take; ++round) {
      constexpr float kInf = __builtin_inff();
      float lo = kInf, hi = -kInf;
#pragma unroll 1
      for (int j = tid; j < (int)listed; j += NT)
        if (digit[j] == dsel) {
          lo = fminf(lo, value[j]);
          hi = fmaxf(hi, value[j]);
        }
      *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
      value_range(sm, tid, lo, hi);
      const Spread finer(lo, hi);
      if (lo == hi && !by_position) {
        by_position = true;
#pragma unroll
        for (int u = 0; u < N; ++u) value[u * NT + tid] = -(float)p[u];
        __syncthreads();                     // (every wave has its extremes)
        continue;
      }
      if (finer.scale == 0.f) break;
#pragma unroll 1
      for (int j = tid; j < (int)listed; j += NT) {
        const uint32_t was = digit[j];
        uint32_t now = was < dsel || was == NONE ? NONE : ABOVE;
        if (was == dsel) {
          now = finer.digit(value[j]);
          atomicAdd(&sm.lhist[now], 1u);
        }
        digit[j] = now;
      }
      __syncthreads();
      crossing_digit(sm, tid, take);
      dsel = sm.sel_digit; take -= sm.sel_above; cnt = sm.sel_count;
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (d[u] != NONE) d[u] = digit[u * NT + tid];
  }
  if (cnt != take || sp.scale == 0.f) {
    if (cnt > SMALL || sp.scale == 0.f) {
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if ((uint32_t)(u * NT + tid) < listed) sm.cand[u * NT + tid] = key(u);
      if (tid == 0) sm.cand_n = listed;
      __syncthreads();
      return false;
    }
    for (int j = tid; j < (int)SMALL; j += NT) sm.few_rank[j] = 0;
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (d[u] == dsel) sm.few[atomicAdd(&sm.cand_n, 1u)] = key(u);
  }
  const uint32_t above = cnt == take ? dsel : dsel + 1;      // digits from here on are taken whole
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (d[u] >= above && d[u] != NONE) atomicOr(&bmp[p[u] >> 5], 1u << (p[u] & 31));
  if (cnt != take)
    take_few(sm, tid, cnt, take, [&](unsigned long long c) {
      const uint32_t pos = (uint32_t)(imask - (c & imask));
      atomicOr(&bmp[pos >> 5], 1u << (pos & 31));
    });
  __syncthreads();
  if (W > RANK_WORDS) {
    emit_bitmap(sm, tid, bmp, W, k, orow);
    return true;
  }
  uint32_t* const rank0 = sm.hist + RANK_WORDS;            // behind the bitmap: the positions taken in front of each word
  auto ranks = [&](auto quads) {                           // a thread's words: 4 * Q in a row
    constexpr int Q = decltype(quads)::value;
    uint4 w[Q];
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int j = 4 * (Q * tid + i);
      w[i] = j < W ? *reinterpret_cast<const uint4*>(&bmp[j]) : make_uint4(0, 0, 0, 0);
      w[i] = make_uint4(__popc(w[i].x), __popc(w[i].y), __popc(w[i].z), __popc(w[i].w));
      n += w[i].x + w[i].y + w[i].z + w[i].w;
    }
    uint32_t total;
    uint32_t at = block_incl_scan(n, sm.wave_tot, &total) - n;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int j = 4 * (Q * tid + i);
      if (j < W) *reinterpret_cast<uint4*>(&rank0[j]) = make_uint4(at, at + w[i].x, at + w[i].x + w[i].y, at + w[i].x + w[i].y + w[i].z);
      at += w[i].x + w[i].y + w[i].z + w[i].w;
    }
  };
  if (W <= 4 * NT) ranks(std::integral_constant<int, 1>{});
  else if (W <= 8 * NT) ranks(std::integral_constant<int, 2>{});
  else ranks(std::integral_constant<int, 4>{});
  __syncthreads();
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t wd = (uint32_t)(u * NT + tid) < listed ? p[u] >> 5 : 0u, bits = bmp[wd], bit = 1u << (p[u] & 31u);
    const uint32_t at = rank0[wd] + __popc(bits & (bit - 1u));
    if ((uint32_t)(u * NT + tid) < listed && (bits & bit)) orow[at] = (int32_t)p[u];
  }
  return true;
}
__device__ __forceinline__ bool finish_list(TopkShared& sm, int tid, const float (&v)[PER], const uint32_t (&p)[PER], uint32_t listed,
                                            float tau, float tau_hi, int vis, int k, int IB, int32_t* __restrict__ orow) {
  if (listed <= 8u * NT) return finish_rounds<8>(sm, tid, v, p, listed, tau, tau_hi, vis, k, IB, orow);
  return finish_rounds<PER>(sm, tid, v, p, listed, tau, tau_hi, vis, k, IB, orow);
}

// Path S: a row that fits the candidate list whole needs no sample and no list: its scores in registers.  They are spread evenly
// over 2046 digits (spread_of); the digit that holds the k-th
// largest is found, and inside it the key by counting.  A wave holds 64 consecutive positions at a time, so a position's rank
// is the number taken in the 64s before, plus a bit count: no bitmap.  Even digits hold a dozen keys near the threshold where
// scores are as they come.  Where one holds more than counting takes, its keys alone are spread between their own extremes; equal scores are
// taken by position, like the ranks.  us, 1 row / 32 rows of 8000, k 2048, of a form with 14 bits of the float as first digit and sixteen waves, of an even spread
// between the extremes with the general selection behind it, and of this: as they come 10.4, 11.1 / 7.3, 7.9 / 7.1, 7.6; one score a thousand spreads away
// 10.4, 11.2 / 20.7, 20.9 / 7.8, 9.5; 1e30 10.3, 11.0 / 25.7, 26.2 / 7.8, 8.1; a fifth masked with -3.4e38 10.5, 11.3 / 23.4, 24.0 / 7.1, 10.9; exponentials of
// twice a normal value 10.1, 10.5 / 25.7, 38.8 / 7.1, 8.5; 900 equal at the threshold 30.0, 30.4 / 34.8, 35.5 / 11.1, 12.0; three values 28.7, 30.5 / 26.4, 28.2 / 11.1, 11.4.
// Where rows are shared it is part 0 of the candidate pass (MODE 1) that takes such a row, not the finishing kernel:
// inlined there beside its other paths it cost every longer row 0.4 to 0.6 us.
// Returns false, with the keys in sm.cand, when more than SMALL keys share that digit all the same (magnitudes apart in several steps).
__device__ __forceinline__ bool whole_row(TopkShared& sm, int tid, const float (&v)[PER], int vis, int k, int IB,
                                          int32_t* __restrict__ orow) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned long long imask = (1ull << IB) - 1ull;
  auto key = [&](int u) {
    uint32_t low = (uint32_t)imask - (uint32_t)(u * NT + tid);
    asm volatile("" : "+v"(low));            // (where it is asked for: left alone, all sixteen are computed by every row, 0.3 us)
    return ((unsigned long long)orderable(v[u]) << IB) | low;
  };
  *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
  if (tid == 0) sm.cand_n = 0;
  constexpr float kInf = __builtin_inff();
  float lo = kInf, hi = -kInf;               // of the finite scores
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const bool fin = u * NT + tid < vis && fabsf(v[u]) < kInf;
    lo = fminf(lo, fin ? v[u] : kInf);
    hi = fmaxf(hi, fin ? v[u] : -kInf);
  }
  // (probes from two places of the row)
  const float probe = (lane & 1) ? (PER / 2 * NT + tid < vis ? v[PER / 2] : __builtin_nanf("")) : (tid < vis ? v[0] : __builtin_nanf(""));
  const Spread sp = spread_of(sm, tid, lo, hi, probe, (float)k / (float)vis);
  uint32_t d[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    d[u] = sp.digit(v[u]);
    if (sp.scale == 0.f) d[u] = v[u] == kInf ? NBINS - 1 : (v[u] > -kInf ? 1u : 0u);      // (one value)
    if (u * NT + tid >= vis) d[u] = NONE;
    if (d[u] - 1u < (uint32_t)(NBINS - 1)) atomicAdd(&sm.lhist[d[u]], 1u);
  }
  __syncthreads();
  crossing_digit(sm, tid, (uint32_t)k, (uint32_t)vis);
  uint32_t dsel = sm.sel_digit, take = (uint32_t)k - sm.sel_above, cnt = sm.sel_count;
  bool equal = false;                        // all keys of that digit have one score
  // (rare)
  if (__builtin_expect(cnt > FEW && cnt != take, 0)) {
#pragma unroll 1
    for (int round = 0; round < NARROW && cnt > FEW && cnt != take; ++round) {      // the keys of that digit alone
      lo = kInf;
      hi = -kInf;
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (d[u] == dsel) {
          const float x = v[u] == v[u] ? v[u] : -kInf;         // (as a key has it)
          lo = fminf(lo, x);
          hi = fmaxf(hi, x);
        }
      *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
      value_range(sm, tid, lo, hi);
      equal = lo == hi;
      const Spread finer(lo, hi);
      if (equal || finer.scale == 0.f) break;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (d[u] == dsel) {
          d[u] = finer.digit(v[u]);
          atomicAdd(&sm.lhist[d[u]], 1u);
        } else {
          d[u] = d[u] == NONE || d[u] < dsel ? NONE : ABOVE;
        }
      }
      __syncthreads();
      crossing_digit(sm, tid, take);
      dsel = sm.sel_digit; take -= sm.sel_above; cnt = sm.sel_count;
    }
  }
  if (cnt > SMALL && cnt != take && !equal) {
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (u * NT + tid < vis) sm.cand[u * NT + tid] = key(u);
    __syncthreads();
    return false;
  }
  // n in lane u of a wave: a count of its u-th 64 positions; in lane (8 u + wave) / 2 afterwards: that of all positions before.  One barrier
  auto counts_before = [&](uint32_t n) {
    if (lane < PER) sm.taken[lane * (NT / 64) + wave] = n;
    __syncthreads();
    const uint2 two = *reinterpret_cast<const uint2*>(&sm.taken[2 * lane]);
    return wave_incl_scan(two.x + two.y, lane) - (two.x + two.y) + ((wave & 1) ? two.x : 0u);
  };
  auto before_of = [&](uint32_t before, int u) { return (uint32_t)__builtin_amdgcn_readlane((int)before, (u * (NT / 64) + wave) >> 1); };
  auto rank_in = [](unsigned long long m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
  // the few that are taken of the crossing digit: a bit per position
  const uint32_t above = cnt == take ? dsel : dsel + 1;      // digits from here on are taken whole
  uint2 bits = make_uint2(0u, 0u);           // lane u: those of the wave's u-th 64
  if (__builtin_expect(equal, 0)) {          // of equal scores the first positions
    uint32_t n = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const unsigned long long t = __ballot(d[u] == dsel);
      n = lane == u ? (uint32_t)__popcll(t) : n;
    }
    const uint32_t before = counts_before(n);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const unsigned long long t = __ballot(d[u] == dsel);
      const uint32_t rank = before_of(before, u) + rank_in(t);
      const unsigned long long first = t & __ballot(rank < take);
      if (lane == u) bits = make_uint2((uint32_t)first, (uint32_t)(first >> 32));
    }
    __syncthreads();                         // (sm.taken has been read)
  } else if (cnt != take) {
    if (tid < (int)(sizeof(sm.few_bits) / 4)) sm.few_bits[tid] = 0;
    for (int j = tid; j < (int)SMALL; j += NT) sm.few_rank[j] = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (d[u] == dsel) sm.few[atomicAdd(&sm.cand_n, 1u)] = key(u);
    take_few(sm, tid, cnt, take, [&](unsigned long long c) {
      const uint32_t pos = (uint32_t)(imask - (c & imask));
      atomicOr(&sm.few_bits[pos >> 5], 1u << (pos & 31));
    });
    __syncthreads();
    if (lane < PER) bits = *reinterpret_cast<const uint2*>(&sm.few_bits[2 * (lane * (NT / 64) + wave)]);
  }
  unsigned long long m[PER];                 // taken positions of the wave's u-th 64
  uint32_t n = 0;                            // lane u: how many
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    m[u] = __ballot(d[u] >= above && d[u] != NONE) |
           ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)bits.y, u) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)bits.x, u));
    n = lane == u ? (uint32_t)__popcll(m[u]) : n;
  }
  const uint32_t before = counts_before(n);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const uint32_t at = before_of(before, u);                // (by all lanes: a lane that is off need not hold its value)
    if ((m[u] >> lane) & 1ull) orow[at + rank_in(m[u])] = u * NT + tid;
  }
  return true;
}

// MODE 0: one workgroup does the whole row (grid: rows).
// MODE 1 + MODE 2, for small batches of long rows: the candidate pass of path A, the only part that
// scales with the row, is spread over `parts` workgroups per row in a kernel of its own (MODE 1, grid
// parts x rows: every workgroup finds the same threshold from the same samples, scans its slice and
// appends its candidates to the row's list in global memory, g_cnt[row] counting them), and the
// finishing kernel (MODE 2, grid rows) takes the list when its size is in [k, buffer] -- else it does
// the row by itself like MODE 0.  The hand-over is the kernel boundary: workgroups of one kernel
// never exchange data (an agent-scope fence inside a kernel costs tens of microseconds on this
// multi-die part, where it writes the L2 back).  g_cnt is zero between steps: MODE 2 clears it.
// MODE 4: as MODE 0 where max_ctx allows only rows that fit the candidate list (path S): the scores are asked for before the
// row's length is known.
// MODE 3: the finishing kernel of the fused selection (grid rows).  The row's list was written by the emitting
// index-score pass (index_kernel.h), for rows of any length; `score` is scratch memory, not scores: a row whose list
// cannot be used (fewer than k or more than the buffer holds: a misleading sample, massive ties) has its scores
// computed here, by this workgroup, into its row of `score`, and is then done like MODE 0.
// one work item = (part, row) of k_topk<MODE>; every field of `sm` is set before it is read, so items may follow each other
struct TopkRecompute {                     // MODE 3: what it takes to compute a row's scores
  const uint8_t* q; const float* w; const uint8_t* key; const int32_t* block_table;
  int n_pages, Hi, Di;
};
template <int MODE, bool DYN>
__device__ __forceinline__ void topk_item(TopkShared& sm, int item, int parts, float* score,
                                          const int32_t* __restrict__ ctx_len, int T, int Lmax, int k, int IB,
                                          int32_t* __restrict__ idx_out, unsigned long long* __restrict__ g_cand,
                                          uint32_t* __restrict__ g_cnt, uint32_t* __restrict__ g_tau, const TopkRecompute& rc) {
  const int row = item / parts;
  const int part = item % parts;
  const int b = row / T, t = row % T;
  // (looping form: the thread index passes through an empty asm statement, so that what is derived from it is computed
  // per work item instead of being carried in registers across the loop, where it led to spills)
  int tid_ = threadIdx.x;
  if constexpr (DYN) asm volatile("" : "+v"(tid_));
  const int tid = tid_, lane = tid & 63;
  float* srow = score + (size_t)row * Lmax;
  int32_t* orow = idx_out + (size_t)row * k;
  float v[MODE == 2 || MODE == 3 ? 1 : PER];
  if constexpr (MODE == 4) {               // no row is longer than the list: asked for beside the row's length
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = srow[min(u * NT + tid, Lmax - 1)];
  }
  int vis = ctx_len[b] - (T - 1 - t);
  vis = max(0, min(vis, Lmax));
  auto load_whole = [&](float (&v)[PER], int n) {
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = srow[min(u * NT + tid, n - 1)];      // (clamped, not predicated; what lies past the end is not looked at)
  };
  if constexpr (MODE == 1) if (vis <= k || vis < FAST_MIN_VIS) {  // nothing to prepare: a short row is done here, or later
    if (part == 0 && vis > k) {
      load_whole(v, vis);
      if (whole_row(sm, tid, v, vis, k, IB, orow) && tid == 0) g_cnt[row] = ROW_DONE;
    }
    return;
  }
  uint32_t listed = 0;
  unsigned long long c[MODE == 2 || MODE == 3 ? PER : 1];
  float list_lo = 0.f, list_hi = 0.f;
  if constexpr (MODE == 2 || MODE == 3) {  // candidates prepared by the kernel in front (0 if none)
    // (the first entries, usually all, are asked for beside their number: a place behind the list's end holds anything)
    const unsigned long long* grow = g_cand + (size_t)row * CAND_CAP;
#pragma unroll
    for (int u = 0; u < LIST_AHEAD; ++u) c[u] = grow[u * NT + tid];
    const uint2 bounds = *reinterpret_cast<const uint2*>(g_tau + 2 * row);      // left by the kernel that made the list
    list_lo = score_of(bounds.x);
    list_hi = bounds.x != 0u && bounds.y > bounds.x ? score_of(bounds.y) : list_lo;
    listed = g_cnt[row];
    __syncthreads();
    if (tid == 0) g_cnt[row] = 0;
    if (MODE == 2 && listed == ROW_DONE) return;
  }
  if (vis <= k) {                          // everything visible is selected
    for (int j = tid; j < k; j += NT) orow[j] = j < vis ? j : -1;
    return;
  }

  const unsigned long long imask = (1ull << IB) - 1ull;
  const bool vec_ok = ((Lmax & 3) == 0) && ((reinterpret_cast<uintptr_t>(score) & 15) == 0);
  auto comp_of = [&](int i, float v) -> unsigned long long {
    return ((unsigned long long)orderable(v) << IB) | (imask - (unsigned long long)i);
  };

  // decided high bits of T* (`prefix`), number of undecided low bits (`rem`), and how many of the
  // keys matching the prefix are still to be taken (`need`); candidates matching it sit in sm.cand
  int rem = 32 + IB;
  unsigned long long prefix = 0;
  uint32_t need = (uint32_t)k;
  bool have_cand = false;                   // sm.cand[0..nc) holds every key matching the prefix
  bool all_in_cand = false;                 // ... and every key above it as well (path A)
  int nc = 0;

  // ---- S: rows that fit the candidate list whole
  if constexpr (MODE == 0 || MODE == 4) if (vis <= CAND_CAP) {
    if constexpr (MODE == 0) load_whole(v, vis);
    if (whole_row(sm, tid, v, vis, k, IB, orow)) return;
    nc = vis;                              // the keys are in sm.cand now, the general selection takes them
    have_cand = true;
    all_in_cand = true;
  }

  // ---- A: sampled one-pass collection for long rows
  const bool use_list = (MODE == 2 || MODE == 3) && listed >= (uint32_t)k && listed <= (uint32_t)CAND_CAP;
  if (MODE == 3 && !use_list) {
    const uint8_t* q_row = rc.q + (size_t)row * rc.Hi * rc.Di;
    const float* w_row = rc.w + (size_t)row * rc.Hi;
    const int32_t* table_row = rc.block_table ? rc.block_table + (size_t)b * (Lmax / ESS_PAGE_TOKENS) : nullptr;
    const uint8_t* keys = rc.block_table ? rc.key : rc.key + (size_t)b * Lmax * rc.Di;
    if (rc.Di == 128) ess_idx::row_scores_slow<128>(q_row, w_row, rc.Hi, keys, Lmax, table_row, rc.n_pages, vis, srow);
    else if (rc.Di == 64) ess_idx::row_scores_slow<64>(q_row, w_row, rc.Hi, keys, Lmax, table_row, rc.n_pages, vis, srow);
    else ess_idx::row_scores_slow<32>(q_row, w_row, rc.Hi, keys, Lmax, table_row, rc.n_pages, vis, srow);
    __syncthreads();                       // the scores are read back by other threads of this workgroup
  }
  if constexpr (MODE == 2 || MODE == 3) if (use_list) {
    const unsigned long long* grow = g_cand + (size_t)row * CAND_CAP;
    float lv[PER];
    uint32_t lp[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (u >= LIST_AHEAD) c[u] = (uint32_t)(u * NT) < listed && (uint32_t)(u * NT + tid) < listed ? grow[u * NT + tid] : 0ull;
      lv[u] = score_of((uint32_t)(c[u] >> IB));
      lp[u] = (uint32_t)(imask - (c[u] & imask));
    }
    if (!(list_hi > list_lo)) {              // a list without bounds: its own extremes
      constexpr float kInf = __builtin_inff();
      list_lo = kInf;
      list_hi = -kInf;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const bool fin = (uint32_t)(u * NT + tid) < listed && fabsf(lv[u]) < kInf;
        list_lo = fminf(list_lo, fin ? lv[u] : kInf);
        list_hi = fmaxf(list_hi, fin ? lv[u] : -kInf);
      }
      value_range(sm, tid, list_lo, list_hi);
    }
    if (finish_list(sm, tid, lv, lp, listed, list_lo, list_hi, vis, k, IB, orow)) return;
  }
  float tau = 0.f, tau_hi = 1.f;
  if (MODE != 4 && (vis >= FAST_MIN_VIS || use_list)) {
    bool found = use_list;
    if (!use_list) {
      // samples: blocks of 16 consecutive scores (one 64-byte piece of a cache line), one of every 1, 2, 4 .. blocks at a
      // place that changes from one to the next (scores that repeat with the stride would else be counted all or not at all),
      // SAMPLE_TARGET scores in all at most, or twice that (sample_blocks).  (One score out of every 16th..32nd touches every cache line of the
      // row: in cache-line traffic the sample then costs as much as the pass that follows.)
      const int nblk_all = vis >> 4, blocks = ess_sel::sample_blocks(k, vis);
      int every = 0;                         // (a power of two as its exponent)
      while ((nblk_all >> every) > blocks) ++every;
      const int ns = (nblk_all >> every) << 4;
      // this workgroup's slice of the row (boundaries on 16-byte pieces); its first round is asked for behind the samples
      const int s_lo = parts > 1 ? (int)(((long)vis * part / parts) & ~3L) : 0;
      const int s_hi = (parts > 1 && part + 1 < parts) ? (int)(((long)vis * (part + 1) / parts) & ~3L) : vis;
      // (a shared row's slice is one round up to 128K: with two sets a step of 4 x 128K takes 42.3 us instead of 41.9)
      constexpr int SETS = MODE == 1 ? 1 : 2;
      float4v x[SETS][ROUND];
      const float* const slice = srow + s_lo;
      const int head = to_boundary(slice);
      auto sampled = [&](auto per_thread) {
        constexpr int N = decltype(per_thread)::value;
        float sv[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int j = min(u * NT + tid, ns - 1);
          const int blk = ((j >> 4) << every) + (int)(((uint32_t)(j >> 4) * 0x9e3779b1u >> 16) & ((1u << every) - 1u));
          sv[u] = srow[(size_t)blk * 16 + (j & 15)];
        }
        *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
        if (tid == 0) { sm.cand_n = 0; sm.sbin[0] = sm.sbin[1] = NONE; }
        row_begin<SETS>(tid, slice + head, s_hi - s_lo - head, x);
        __builtin_amdgcn_sched_barrier(0);
        return bounds_of(sm, tid, sv, ns, k, vis, &tau, &tau_hi);
      };
      found = __builtin_expect(blocks * 16 == ess_sel::SAMPLE_TARGET, 1) ? sampled(std::integral_constant<int, ess_sel::SAMPLE_TARGET / NT>{})
                                                                         : sampled(std::integral_constant<int, 2 * ess_sel::SAMPLE_TARGET / NT>{});
      if (MODE == 1 && !found) return;       // no usable threshold: the finishing kernel takes path B
      // The pass only compares floats and stores (position, score) of the few positions at or above
      // the threshold (NaN is below, -0 == +0: the order of the keys),
      // and the composite keys are computed afterwards, densely, for the candidates alone.
      if (found) collect(tid, slice, s_lo, s_hi - s_lo, x, tau, reinterpret_cast<uint2*>(sm.cand), &sm.cand_n, sm.stage);
      __syncthreads();
    }
    if (found) {
      nc = (int)sm.cand_n;
      if (MODE == 1) {
        // append this slice's candidates to the row's list; the true count is added even when it overflows,
        // so that the finishing kernel sees the overflow
        unsigned long long* grow = g_cand + (size_t)row * CAND_CAP;
        if (tid == 0) {
          sm.sel_above = atomicAdd(&g_cnt[row], (uint32_t)nc);
          if (part == 0) { g_tau[2 * row] = orderable(tau); g_tau[2 * row + 1] = orderable(tau_hi); }      // (every part finds the same two)
        }
        __syncthreads();
        const uint32_t gbase = sm.sel_above;
        if (nc <= CAND_CAP)
          for (int j = tid; j < nc; j += NT)
            if (gbase + (uint32_t)j < (uint32_t)CAND_CAP) {
              const uint2 pv = reinterpret_cast<const uint2*>(sm.cand)[j];
              grow[gbase + j] = comp_of((int)pv.x, __uint_as_float(pv.y));
            }
        return;
      }
      if (!use_list && nc >= k && nc <= CAND_CAP) {
        float lv[PER];
        uint32_t lp[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          uint2 pv = make_uint2(0u, 0u);
          if (u * NT < nc && u * NT + tid < nc) pv = reinterpret_cast<const uint2*>(sm.cand)[u * NT + tid];
          lp[u] = pv.x;
          lv[u] = __uint_as_float(pv.y);
        }
        __syncthreads();                   // the bitmap shares its memory with the list: every thread holds its keys first
        if (finish_list(sm, tid, lv, lp, (uint32_t)nc, tau, tau_hi, vis, k, IB, orow)) return;
      }
      if (nc >= k && nc <= CAND_CAP) {
        // bits on which the candidates differ: everything above is common and decided
        unsigned long long a = ~0ull, o = 0ull;
        for (int j = tid; j < nc; j += NT) { a &= sm.cand[j]; o |= sm.cand[j]; }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) { a &= __shfl_xor(a, d, 64); o |= __shfl_xor(o, d, 64); }
        if (lane == 0) { sm.red_and[tid >> 6] = a; sm.red_or[tid >> 6] = o; }
        __syncthreads();
        a = ~0ull; o = 0ull;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) { a &= sm.red_and[i]; o |= sm.red_or[i]; }
        const unsigned long long diff = a ^ o;
        rem = diff ? 64 - __clzll((long long)diff) : 0;
        prefix = rem < 64 ? (o >> rem) : 0;
        have_cand = true;
        all_in_cand = true;
      }
      __syncthreads();
    }
  }

  // ---- B: general narrowing from memory
  uint32_t cnt_match = (uint32_t)vis;
  if (!have_cand) {
    // A sample with more equal scores than a list holds (bounds_of): is the k-th largest one of them?  One pass instead of three.
    // If not, those above them may be a list.  us, k 2048, of a row of 12000 with 800 scores above zero 36.6 / 25.4, of 40000 with 2700 36.9 / 34.1.
    if (tau == tau_hi) {
      uint32_t above = 0, equal = 0;
      scan_row(tid, srow, vis, vec_ok, [&](int, float v, bool ok) {
        above += ok && v > tau ? 1u : 0u;
        equal += ok && v == tau ? 1u : 0u;
      });
      uint32_t all_above, all_equal;
      block_incl_scan(above, sm.wave_tot, &all_above);
      block_incl_scan(equal, sm.wave_tot, &all_equal);
      if (all_above < need && all_above + all_equal >= need) {
        prefix = orderable(tau);
        rem = IB;
        need -= all_above;
        cnt_match = all_equal;
      } else if (all_above >= need && all_above <= (uint32_t)CAND_CAP) {
        if (tid == 0) sm.cand_n = 0;
        __syncthreads();
        scan_row(tid, srow, vis, vec_ok, [&](int i, float v, bool ok) {
          wave_append<unsigned long long>(ok && v > tau, comp_of(i, v), sm.cand, &sm.cand_n, CAND_CAP);
        });
        __syncthreads();
        nc = (int)sm.cand_n;
        have_cand = all_in_cand = true;
      }
    }
  }
  if (!have_cand) {
    while (cnt_match > (uint32_t)CAND_CAP && rem > 0) {
      const int bits = min(HBITS, rem);
      const int shift = rem - bits;
      const uint32_t dmask = (1u << bits) - 1u;
      for (int j = tid; j < NBINS * COPIES; j += NT) sm.hist[j] = 0;
      __syncthreads();
      scan_row(tid, srow, vis, vec_ok, [&](int i, float v, bool ok) {
        const unsigned long long c = comp_of(i, v);
        if (ok && (c >> rem) == prefix)
          atomicAdd(&sm.hist[(((uint32_t)(c >> shift)) & dmask) * COPIES + (lane & 7)], 1u);
      });
      __syncthreads();
      for (int j = tid; j < NBINS; j += NT) {              // the copies of a digit are added up
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < COPIES; ++r) sum += sm.hist[j * COPIES + r];
        sm.lhist[j] = sum;
      }
      __syncthreads();
      crossing_digit(sm, tid, need);
      need -= sm.sel_above;
      prefix = (prefix << bits) | sm.sel_digit;
      cnt_match = sm.sel_count;
      rem = shift;
      __syncthreads();
    }
    if (tid == 0) sm.cand_n = 0;
    __syncthreads();
    scan_row(tid, srow, vis, vec_ok, [&](int i, float v, bool ok) {
      const unsigned long long c = comp_of(i, v);
      wave_append<unsigned long long>(ok && (c >> rem) == prefix, c, sm.cand, &sm.cand_n, CAND_CAP);
    });
    __syncthreads();
    nc = (int)sm.cand_n;
  }

  // ---- C: radix select inside LDS: the need-th largest candidate among those matching the prefix
  while (rem > 0) {
    const int bits = min(HBITS, rem);
    const int shift = rem - bits;
    const uint32_t dmask = (1u << bits) - 1u;
    for (int j = tid; j < NBINS; j += NT) sm.lhist[j] = 0;
    __syncthreads();
    for (int j = tid; j < nc; j += NT) {
      const unsigned long long c = sm.cand[j];
      if ((c >> rem) == prefix) atomicAdd(&sm.lhist[((uint32_t)(c >> shift)) & dmask], 1u);
    }
    __syncthreads();
    crossing_digit(sm, tid, need);
    need -= sm.sel_above;
    prefix = (prefix << bits) | sm.sel_digit;
    const uint32_t cnt = sm.sel_count;
    rem = shift;
    __syncthreads();
    if (cnt == need) break;                  // every key with this prefix is taken
  }
  const unsigned long long t_star = rem < 64 ? (prefix << rem) : 0ull;

  // ---- D: mark the selected positions in a bitmap of the row, read them back in ascending order
  uint32_t* bmp = sm.hist;                   // aliases cand: the keys are moved out first
  const int W = (vis + 31) >> 5;             // <= 16384 words
  if (all_in_cand) {
    if (tid == 0) sm.out_n = 0;
    __syncthreads();
    for (int j0 = 0; j0 < nc; j0 += NT) {
      const int j = j0 + tid;
      const unsigned long long c = j < nc ? sm.cand[j] : 0ull;
      wave_append<int32_t>(j < nc && c >= t_star, (int32_t)(imask - (c & imask)), sm.out_list, &sm.out_n, ESS_MAX_TOPK);
    }
    __syncthreads();
    for (int j = tid; j < W; j += NT) bmp[j] = 0;
    __syncthreads();
    for (int j = tid; j < k; j += NT) {
      const int pos = sm.out_list[j];
      atomicOr(&bmp[pos >> 5], 1u << (pos & 31));
    }
  } else {
    __syncthreads();
    for (int j = tid; j < W; j += NT) bmp[j] = 0;
    __syncthreads();
    scan_row(tid, srow, vis, vec_ok, [&](int i, float v, bool ok) {
      if (ok && comp_of(i, v) >= t_star) atomicOr(&bmp[i >> 5], 1u << (i & 31));
    });
  }
  __syncthreads();
  emit_bitmap(sm, tid, bmp, W, k, orow);
}

template <int MODE, bool DYN>
__global__ __launch_bounds__(NT) void k_topk(float* score, const int32_t* __restrict__ ctx_len,
                                             int T, int Lmax, int k, int IB, int32_t* __restrict__ idx_out,
                                             unsigned long long* __restrict__ g_cand, uint32_t* __restrict__ g_cnt,
                                             uint32_t* __restrict__ g_tau, ess_xcd xcd, int rows, int parts_arg,
                                             const TopkRecompute rc) {
  __shared__ TopkShared sm;
  __shared__ int s_item;
  const int parts = MODE == 1 ? parts_arg : 1;
  // work item = (part, row): by workgroup index, or drawn from the launch's counter off the XCDs to be avoided
  ESS_WORK_LOOP(DYN, xcd, MODE == 1 ? blockIdx.y * parts + blockIdx.x : blockIdx.x, rows * parts, &s_item, item) {
    topk_item<MODE, DYN>(sm, item, parts, score, ctx_len, T, Lmax, k, IB, idx_out, g_cand, g_cnt, g_tau, rc);
  }
}

// The bounds of every row's selection, from the scores of the sequence's sample blocks (one workgroup per row), as
// ess_orderable images of scores:
// tau[row][0] = a score that very probably has at least k and at most a few thousand of the row's scores at or above
// it; 0 (everything is a candidate) for rows that fit the candidate buffer whole or whose sample gives no bound;
// 0xffffffff (nothing) for rows with at most k visible positions, which need no list;
// tau[row][1] = a score with about an eighth of k of the row's scores at or above it (see bounds_of; 0 without a bound): the k-th
// largest score very probably lies between the two, which lets the finishing kernel resolve that range in one pass.
// Also clears the row's candidate counter for the pass that follows.
template <bool DYN>
__global__ __launch_bounds__(NT) void k_index_tau(const float* __restrict__ sample, const int32_t* __restrict__ ctx_len,
                                                  int T, int Lmax, int k, int period, int nsamp,
                                                  uint32_t* __restrict__ tau, uint32_t* __restrict__ g_cnt, ess_xcd xcd,
                                                  int rows) {
  __shared__ BoundsShared sm;
  __shared__ int s_item;
  ESS_WORK_LOOP(DYN, xcd, blockIdx.x, rows, &s_item, row) {
    const int tid = threadIdx.x;
    const int b = row / T, t = row % T;
    const int len = min(ctx_len[b], Lmax);
    const int vis = max(0, len - (T - 1 - t));
    if (tid == 0) g_cnt[row] = 0;
    if (vis <= k || vis <= CAND_CAP) {
      if (tid == 0) {
        tau[2 * row] = vis <= k ? 0xffffffffu : 0u;
        tau[2 * row + 1] = 0u;
      }
      continue;
    }
    // the blocks that count are the first nv: starts grow with the block number
    const int lim = len - (T - 1);
    int nv = lim / period;
    if (nv < nsamp && ess_sample_start(nv, period) + 64 <= lim) ++nv;
    nv = min(nv, nsamp);
    const int ns = nv * 64;
    // the samples are requested before the histogram is cleared: one round trip to memory, not two
    const float* srow = sample + (size_t)row * nsamp * 64;
    constexpr int N = ESS_SAMPLE_BLOCKS * 64 / NT;
    float sv[N];
#pragma unroll
    for (int u = 0; u < N; ++u) sv[u] = u * NT + tid < ns ? srow[u * NT + tid] : 0.f;
    *reinterpret_cast<uint4*>(&sm.lhist[DPT * tid]) = make_uint4(0, 0, 0, 0);
    if (tid == 0) sm.sbin[0] = sm.sbin[1] = 0xffffffffu;
    float lo = 0.f, hi = 1.f;
    const bool found = ns > 0 && bounds_of(sm, tid, sv, ns, k, vis, &lo, &hi);
    if (tid == 0) {
      tau[2 * row] = found || lo == hi ? orderable(lo) : 0u;   // (lo == hi: more equal scores than a list holds; those below need not be listed either)
      tau[2 * row + 1] = found ? orderable(hi) : 0u;
    }
  }
}

}  // namespace

namespace {
// Launches of one top-k call.  cand / cnt: candidate lists [ESS_TOPK_SHARED_ROWS][CAND_CAP] and their counters
// (zero at launch, zero again afterwards), only used when rows are shared by several workgroups.
int launch_topk(int max_ctx, int k, const float* score_in, const int32_t* ctx_len, int B, int T, int32_t* idx,
                unsigned long long* cand, uint32_t* cnt, uint32_t* tau, hipStream_t st, ess_xcd xcd) {
  float* score = const_cast<float*>(score_in);          // read only in these modes
  const TopkRecompute rc{};
  int IB = 1;
  while ((1 << IB) < max_ctx) ++IB;
  // small batches of long rows: the candidate pass goes to a kernel of its own that puts several
  // workgroups on every row (as many as fill the chip, at most 8)
  const int rows = B * T;
  int parts = 1;
  if (max_ctx >= 65536 && rows <= ESS_TOPK_SHARED_ROWS) {
    parts = 256 / rows;
    if (parts > 8) parts = 8;
  }
  const ess_xcd x0 = xcd, x1 = ess_xcd{xcd.ticket ? xcd.ticket + ESS_TICKET_WORDS : nullptr, xcd.avoid,
                                       xcd.host_need ? xcd.host_need + 1 : nullptr, xcd.grid_override};
  const bool dyn = xcd.ticket != nullptr;
#define ESS_TOPK_LAUNCH(MODE, grid, x, np)                                                                           \
  do {                                                                                                               \
    if (dyn) hipLaunchKernelGGL((k_topk<MODE, true>), grid, dim3(NT), 0, st, score, ctx_len, T, max_ctx, k, IB, idx, \
                                cand, cnt, tau, x, rows, np, rc);                                                    \
    else hipLaunchKernelGGL((k_topk<MODE, false>), grid, dim3(NT), 0, st, score, ctx_len, T, max_ctx, k, IB, idx,    \
                            cand, cnt, tau, x, rows, np, rc);                                                        \
  } while (0)
  if (parts > 1) {
    const dim3 g1 = dyn ? dim3(ess_xcd_grid(parts * rows, x0)) : dim3(parts, rows);
    ESS_TOPK_LAUNCH(1, g1, x0, parts);
    ESS_TOPK_LAUNCH(2, dim3(ess_xcd_grid(rows, x1)), x1, 1);
  } else if (max_ctx <= CAND_CAP) {
    ESS_TOPK_LAUNCH(4, dim3(ess_xcd_grid(rows, x1)), x1, 1);
  } else {
    ESS_TOPK_LAUNCH(0, dim3(ess_xcd_grid(rows, x1)), x1, 1);
  }
#undef ESS_TOPK_LAUNCH
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}
}  // namespace

int ess_launch_topk(ess_ctx* ctx, const float* score, const int32_t* ctx_len, int B, int T, int32_t* idx,
                    hipStream_t st, ess_xcd xcd) {
  return launch_topk(ctx->cfg.max_ctx, ctx->cfg.topk, score, ctx_len, B, T, idx, ctx->topk_cand, ctx->topk_cnt, ctx->topk_tau, st, xcd);
}

// The two small kernels of the fused selection that live here (see ess_internal.h).
int ess_launch_index_tau(ess_ctx* ctx, const int32_t* ctx_len, int B, int T, int b0, hipStream_t st, ess_xcd xcd) {
  const ess_config& c = ctx->cfg;
  const int rows = B * T, nsamp = ess_sample_count(c.max_ctx);
  const size_t r0 = (size_t)b0 * T;
  const dim3 grid(ess_xcd_grid(rows, xcd));
  if (xcd.ticket)
    hipLaunchKernelGGL((k_index_tau<true>), grid, dim3(NT), 0, st, ctx->sel_sample + r0 * nsamp * 64, ctx_len, T, c.max_ctx,
                       c.topk, ess_sample_period(c.max_ctx), nsamp, ctx->sel_tau + 2 * r0, ctx->sel_cnt + r0, xcd, rows);
  else
    hipLaunchKernelGGL((k_index_tau<false>), grid, dim3(NT), 0, st, ctx->sel_sample + r0 * nsamp * 64, ctx_len, T, c.max_ctx,
                       c.topk, ess_sample_period(c.max_ctx), nsamp, ctx->sel_tau + 2 * r0, ctx->sel_cnt + r0, xcd, rows);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_topk_finish(ess_ctx* ctx, const uint8_t* q, const float* w, const uint8_t* key, const int32_t* block_table,
                           int n_pages, const int32_t* ctx_len, int B, int T, int b0, int32_t* idx, hipStream_t st,
                           ess_xcd xcd) {
  const ess_config& c = ctx->cfg;
  int IB = 1;
  while ((1 << IB) < c.max_ctx) ++IB;
  const int rows = B * T;
  const size_t r0 = (size_t)b0 * T;
  const TopkRecompute rc{q, w, key, block_table, n_pages, c.idx_heads, c.idx_dim};
  const dim3 grid(ess_xcd_grid(rows, xcd));
  if (xcd.ticket)
    hipLaunchKernelGGL((k_topk<3, true>), grid, dim3(NT), 0, st, ctx->score_ws + r0 * c.max_ctx, ctx_len, T, c.max_ctx, c.topk,
                       IB, idx, ctx->sel_cand + r0 * CAND_CAP, ctx->sel_cnt + r0, ctx->sel_tau + 2 * r0, xcd, rows, 1, rc);
  else
    hipLaunchKernelGGL((k_topk<3, false>), grid, dim3(NT), 0, st, ctx->score_ws + r0 * c.max_ctx, ctx_len, T, c.max_ctx, c.topk,
                       IB, idx, ctx->sel_cand + r0 * CAND_CAP, ctx->sel_cnt + r0, ctx->sel_tau + 2 * r0, xcd, rows, 1, rc);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_sel_cand_cap() { return CAND_CAP; }

size_t ess_topk_cand_bytes() { return (size_t)ESS_TOPK_SHARED_ROWS * CAND_CAP * sizeof(unsigned long long); }

// ---------------------------------------------------------------------------------------------
// ess_topk_static: the top-k for callers that cannot allocate.  Its scratch memory -- the candidate lists of rows
// shared by several workgroups, and their counters -- is this array, part of the library's image on every
// GPU it is loaded on (8 MiB + 1536 bytes).  In host code the array's name is not a device address: the address
// on the current device is asked for once per device and kept.
namespace {
constexpr size_t kStaticCand = (size_t)ESS_TOPK_SHARED_ROWS * CAND_CAP;          // candidate keys
constexpr size_t kStaticWords = kStaticCand + ESS_TOPK_SHARED_ROWS / 2 + ESS_TOPK_SHARED_ROWS;   // + the rows' counters (uint32 each) + their bounds (2 x uint32)
constexpr int kMaxDevices = 64;
static_assert(ESS_TOPK_STATIC_MAX_ROWS == ESS_TOPK_SHARED_ROWS, "the static scratch holds one candidate list per shared row");
}  // namespace
static __device__ __align__(256) unsigned long long ess_topk_scratch[kStaticWords];
namespace {
unsigned long long* g_static_ptr[kMaxDevices];                                   // per device: address of its copy of the array
std::mutex g_static_mu;
}  // namespace

extern "C" int ess_topk_static(const float* score, const int32_t* ctx_len, int32_t B, int32_t T, int32_t max_ctx,
                               int32_t k, int32_t* idx, void* stream) {
  if (!score || !ctx_len || !idx) return ess_fail(ESS_ERR_INVALID_ARG, "NULL argument");
  if (B < 1 || T < 1 || T > 4) return ess_fail(ESS_ERR_INVALID_ARG, "B %d, T %d (T: 1 to 4)", B, T);
  if ((long)B * T > ESS_TOPK_STATIC_MAX_ROWS)
    return ess_fail(ESS_ERR_CAPACITY, "ess_topk_static: B*T = %ld rows exceed the %d its static scratch memory holds",
                    (long)B * T, ESS_TOPK_STATIC_MAX_ROWS);
  if (max_ctx < 1 || max_ctx > ESS_MAX_CTX)
    return ess_fail(ESS_ERR_CAPACITY, "ess_topk_static: max_ctx %d outside [1, %d]", max_ctx, ESS_MAX_CTX);
  if (k < 1 || k > ESS_MAX_TOPK) return ess_fail(ESS_ERR_CAPACITY, "ess_topk_static: k %d outside [1, %d]", k, ESS_MAX_TOPK);
  int dev = 0;
  ESS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return ess_fail(ESS_ERR_UNSUPPORTED, "ess_topk_static: device %d", dev);
  unsigned long long* base;
  {
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {                 // first call on this device: where does its copy of the array live?
      void* p = nullptr;
      ESS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(ess_topk_scratch)));
      if (!p) return ess_fail(ESS_ERR_HIP, "ess_topk_static: the scratch array has no address on device %d", dev);
      g_static_ptr[dev] = static_cast<unsigned long long*>(p);
    }
    base = g_static_ptr[dev];
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(base + kStaticCand);
  // the array keeps what the last call left: the counters must start at zero (a fill kernel, not a memset node,
  // so that the call may be captured in a graph)
  int rc = ess_launch_fill_u32(cnt, ESS_TOPK_SHARED_ROWS, 0u, st);
  if (rc != ESS_OK) return rc;
  return launch_topk(max_ctx, k, score, ctx_len, B, T, idx, base, cnt, cnt + ESS_TOPK_SHARED_ROWS, st, ess_xcd{nullptr, 0, nullptr, 0});
}
