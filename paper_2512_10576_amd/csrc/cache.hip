// Stages 3 + 5: Sparse Memory Pool look-up, LRU update, miss fetch and row
// gather (ESS paper Sec. 3.1 FlashTrans, Sec. 3.2 LRU-based eviction and
// admission).  The swap unit is one Latent-Cache entry (Sec. 3.1).
//
// Reading of "LRU-based" implemented here (step-granular, order-free):
//   R = distinct valid selected positions of a sequence; resident members are
//   hits and get stamp := step; the others, in ascending position, take the
//   slots smallest in (stamp, slot) among slots with stamp < step; the former
//   token of a taken slot becomes non-resident.
//
// One workgroup per sequence does the whole update without any serial list:
//   - the selection is turned into a bitmap in LDS (dedups the T query
//     tokens and yields misses in ascending position by a prefix sum);
//   - the threshold stamp of the victims comes from one histogram pass over
//     the stamps' ages (conflict-free: 32 interleaved copies, copy =
//     lane & 31); only where it is older than 254 steps does a radix select
//     on the 32-bit stamps follow.  Ties on the threshold stamp are broken by
//     slot order with one block scan.  Up to 1024 victims are ordered by a
//     stable counting sort over their ages (by comparing all pairs where
//     some are older than that), more by a bitonic sort in LDS;
//   - the i-th miss is paired with the i-th victim and a fetch list is
//     written for the fill kernel;
//   - per (b,t), slots of hits and of fetched entries are compacted into two
//     lists, which drive Attn0 and Attn1 (Sec. 3.3).
// The fetch itself is a separate kernel so that it can run on a side stream:
// GPU threads read the pinned host pool by address (the paper's UVA idea),
// one wave per 1152- or 656-byte entry, many entries in flight.
#include "ess_internal.h"
#include "select_common.h"
#include "fetch.h"

namespace {

constexpr int BT = 1024;

struct BookShared {
  uint32_t wave_tot[BT / 64], wave_tot2[BT / 64];
  uint32_t sel_digit, sel_below, sel_upto;
};
// The large arrays of the bookkeeping kernel live in dynamic LDS, sized by the configuration:
//   bm [W]  bitmap of the missed positions (W = max_ctx / 32 words, rounded up to an even number)
//   un      histogram of the stamps (256 x 32 counters, 32 KiB), later the victims' (stamp, slot) keys
//           (vict_cap = sel_cap rounded up to a power of two, 8 bytes each)
//   mt [sel_cap]  missed positions in ascending order (sel_cap = max_q_tokens * topk)
constexpr int BOOK_HIST_BYTES = 256 * 32 * 4;
// Inside `un`, in words, while the victims' list takes no more than its first 2048 (up to 1024 victims):
constexpr int BOOK_CNT = 2048;       // [256 digits][16 waves] bytes: the list's slots of a digit in a wave's part of it
constexpr int BOOK_LISTS = 6144;     // [4][16] totals of the hit / miss lists (a longer list of victims is done with by then)
constexpr int BOOK_BELOW = 7168;     // [256] victims of smaller digits
constexpr int BOOK_PRE = 7424;       // [1024] 16 bits each: misses in front of a thread's bitmap words
static_assert(BOOK_PRE + BT / 2 <= BOOK_HIST_BYTES / 4, "book layout");
inline int book_pow2(int n) { int p = 1; while (p < n) p <<= 1; return p; }
inline size_t book_words(int max_ctx) { return (size_t)(((max_ctx + 31) / 32 + 1) & ~1); }
inline size_t book_union_bytes(int sel_cap) {
  const size_t v = (size_t)book_pow2(sel_cap) * 8;
  return v > (size_t)BOOK_HIST_BYTES ? v : (size_t)BOOK_HIST_BYTES;
}
inline size_t book_lds_bytes(int max_ctx, int sel_cap) {
  return book_words(max_ctx) * 4 + book_union_bytes(sel_cap) + (size_t)sel_cap * 4;
}

using ess_sel::wave_incl_scan;
__device__ __forceinline__ uint32_t block_incl_scan(uint32_t v, uint32_t* wave_tot, uint32_t* total) {
  return ess_sel::block_incl_scan<BT>(v, wave_tot, total);
}

__device__ void bitonic_sort_u64(unsigned long long* a, int n) {
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int t = threadIdx.x; t < (n >> 1); t += BT) {
        const int lo = 2 * t - (t & (stride - 1));
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;
        const unsigned long long x = a[lo], y = a[hi];
        if ((x > y) == up) { a[lo] = y; a[hi] = x; }
      }
    }
  }
  __syncthreads();
}

// set bits of the wave's mask in front of this lane's
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// idx: [B, T, kk] selected positions (-1 = none).  Dynamic LDS: bitmap of Lmax bits.
// REG: pools up to 16384 slots.  A wave owns a contiguous range of slots, 64 of them (one a lane) at a time, at most
// 16 times: the stamps are read once, whole lines at a time, and held in registers.  (Sixteen consecutive slots a thread make a
// load of a wave touch some 30 lines.)  What bounds the kernel: two dependent trips to memory (5 us) and the instructions of
// 16 waves on one CU (four to a SIMD: each costs all of them 16 cycles), hence the counts by ballot and the sums over waves by
// one row of lanes.  One sequence, cycles at 2.4 GHz, threads owning consecutive slots / this: 8192 slots, 190 misses
// 40500 / 32500; 6554 slots, 360 misses 34300 / 31800; 9001 slots, two tokens, 110 misses 39600 / 35000; 13108 slots,
// two tokens, 420 misses 66300 / 56000.  (Reading the stamps at the start, beside the look-up, with an LDS bitmap of the
// hit slots instead of a store each: the same with misses, 3 us longer where there are none.)
template <bool REG, bool DYN>
__global__ __launch_bounds__(BT) void k_bookkeeping(
    const int32_t* __restrict__ idx, int T, int kk, int Lmax, int S, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ token_of, uint32_t* __restrict__ stamp, uint32_t step, int32_t* __restrict__ slot_idx_out,
    int32_t* __restrict__ fresh_idx, int32_t* __restrict__ hit_list, int32_t* __restrict__ miss_list, int32_t* __restrict__ n_hit,
    int32_t* __restrict__ n_miss, int32_t* __restrict__ fill_tok, int32_t* __restrict__ fill_slot, int fill_cap,
    int32_t* __restrict__ miss_cnt, int32_t* __restrict__ miss_count_out, unsigned long long* __restrict__ stats,
    unsigned long long* __restrict__ seq_stats,
    int row_stride, int count_step, int32_t* __restrict__ host_miss, ess_xcd xcd, int n_seq,
    uint32_t* __restrict__ zero_tickets, int n_zero_tickets, int bm_words, int union_bytes) {
  extern __shared__ __align__(16) uint32_t bm[];              // see the layout above
  uint32_t* const s_hist = bm + bm_words;
  unsigned long long* const s_vict = reinterpret_cast<unsigned long long*>(bm + bm_words);
  int32_t* const s_miss_tok = reinterpret_cast<int32_t*>(bm + bm_words + union_bytes / 4);
  const int vict_cap = union_bytes / 8;                       // >= the misses of one step, rounded up to a power of two
  __shared__ BookShared sm;
  __shared__ int s_item;
  constexpr int RS = 16;                       // register-held stamps per thread
  // work counters of the kernels that follow this one beside the fetch it feeds: cleared here, by the first
  // workgroup, so that no launch has to do it (this kernel itself never uses the counters it clears)
  if (zero_tickets && blockIdx.x == 0)            // n_zero_tickets launches' counters: the words in use
    for (int i = threadIdx.x; i < n_zero_tickets * ESS_TICKET_USED; i += BT)
      zero_tickets[(i / ESS_TICKET_USED) * ESS_TICKET_WORDS + (i % ESS_TICKET_USED) * ESS_TK_STRIDE] = 0;
  // work item = sequence: by workgroup index, or drawn from the launch's counter off the XCDs to be avoided
  ESS_WORK_LOOP(DYN, xcd, blockIdx.x, n_seq, &s_item, b) {
  // (looping form: the thread index passes through an empty asm statement, so that what is derived from it is
  // computed per work item instead of being carried in registers across the loop, where it led to spills)
  int tid_ = threadIdx.x;
  if constexpr (DYN) asm volatile("" : "+v"(tid_));
  const int tid = tid_, lane = tid & 63;
  const int W = (Lmax + 31) >> 5;
  const int nsel = T * kk;
  const int32_t* sel = idx + (size_t)b * nsel;
  int32_t* so = slot_of + (size_t)b * Lmax;
  int32_t* to = token_of + (size_t)b * S;
  uint32_t* stp = stamp + (size_t)b * S;

  // this wave's slots in the register form: [ws, ws + 64 * nj), nj <= 16
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nj_reg = (S + BT - 1) / BT;
  const int ws = wave * nj_reg * 64;
  uint32_t sr[RS];
  for (int j = tid; j < W; j += BT) bm[j] = 0;
  {
    uint2* const h2 = reinterpret_cast<uint2*>(s_hist);          // the counters of the age pass
    for (int j = tid; j < BOOK_HIST_BYTES / 8; j += BT) h2[j] = make_uint2(0, 0);
  }
  // look-up straight from the selection list (all gathers of a thread in flight together): hits get
  // their stamp, misses set their bit; duplicates across the T query tokens do the same thing twice
  // (kept: when one round covers the selection and a query token's list is whole rounds of the workgroup, the
  // lists at the end are built from these registers instead of a second look-up)
  const bool keep = nsel <= 4 * BT && kk % BT == 0;
  if (tid == 0) sm.sel_upto = 0xffffffffu;       // (stays so where a step has too few slots that it may evict)
  uint32_t my_valid = 0;
  int sv[4] = {-1, -1, -1, -1}, slv[4] = {-1, -1, -1, -1};
  auto select = [&](int e0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * BT + tid;
      sv[u] = e < nsel ? sel[e] : -1;
    }
  };
  auto look_up = [&]() {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (sv[u] >= Lmax) sv[u] = -1;
      slv[u] = sv[u] >= 0 ? so[sv[u]] : -1;
    }
  };
  auto mark = [&]() {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (sv[u] < 0) continue;
      ++my_valid;
      if (slv[u] < 0) atomicOr(&bm[sv[u] >> 5], 1u << (sv[u] & 31));
      else stp[slv[u]] = step;
    }
  };
  select(0);
  look_up();
  __syncthreads();                               // the bitmap is clear
  mark();
  for (int e0 = 4 * BT; e0 < nsel; e0 += 4 * BT) {
    select(e0);
    look_up();
    mark();
  }
  __syncthreads();
  // misses in ascending position: prefix sum over the bitmap words (a thread's words: a power of two of them)
  int wsh = 0;
  while ((BT << wsh) < W) ++wsh;
  const int w0 = min(tid << wsh, W), w1 = min(w0 + (1 << wsh), W);
  uint32_t my_miss = 0;
  for (int wd = w0; wd < w1; ++wd) my_miss += __popc(bm[wd]);
  // one scan for both counts (each at most T * k <= 8192: 16 bits apiece)
  uint32_t both;
  const uint32_t miss_inc = block_incl_scan(my_miss | (my_valid << 16), sm.wave_tot, &both) & 0xffffu;
  const uint32_t m = both & 0xffffu, nvalid = both >> 16;
  const uint32_t miss_before = miss_inc - my_miss;
  {
    uint32_t pos = miss_before;
    for (int wd = w0; wd < w1; ++wd) {
      uint32_t bits = bm[wd];
      while (bits) {
        const int bit = __ffs(bits) - 1;
        bits &= bits - 1;
        if (pos < (uint32_t)fill_cap) s_miss_tok[pos] = wd * 32 + bit;
        ++pos;
      }
    }
  }
  __syncthreads();                               // the stamps of the hits are visible

  // the counts leave here, so that their way to memory (and to the host) passes beside the work below
  if (tid == 0) {
    miss_cnt[b] = (int32_t)m;
    if (miss_count_out) miss_count_out[b] = (int32_t)m;
    if (host_miss) host_miss[b] = (int32_t)m;       // pinned host memory: the host's view for the overlap switch
  }
  if (tid < 8) {
    // counters of the context (steps, valid entries, misses, bytes) and the same of the sequence, a lane each (adds that
    // return nothing: a read of the counters would be waited for)
    const int which = tid & 3;
    const bool whole = tid < 4;
    const unsigned long long add = which == 0 ? (whole && !(b == 0 && count_step) ? 0ull : 1ull)
                                 : which == 1 ? nvalid
                                 : which == 2 ? m : (unsigned long long)m * (unsigned long long)row_stride;
    atomicAdd(whole ? &stats[which] : &seq_stats[4 * (size_t)b + which], add);
  }

  // pair the i-th miss with victim v, whose former token is `old`
  auto pair = [&](uint32_t i, int v, int old) {
    const int s = s_miss_tok[i];
    if (old >= 0) so[old] = -1;
    to[v] = s;
    so[s] = v;
    stp[v] = step;
    fill_tok[(size_t)b * fill_cap + i] = s;
    fill_slot[(size_t)b * fill_cap + i] = v;
  };
  const bool by_rank = m <= (uint32_t)BT;
  uint16_t* const s_pre = reinterpret_cast<uint16_t*>(s_hist + BOOK_PRE);
  if (m > 0) {
    if constexpr (REG) {
      const int left = min(S - ws, 64 * nj_reg);
#pragma unroll
      for (int j = 0; j < RS; ++j) {
        sr[j] = 0xffffffffu;                       // never evictable
        if (64 * j + 64 <= left) sr[j] = stp[ws + 64 * j + lane];
        else if (64 * j < left && 64 * j + lane < left) sr[j] = stp[ws + 64 * j + lane];
      }
    }
    // (larger pools) this thread's slots: [v0, v1), contiguous so that slot order is thread order
    const int v0 = min(tid * nj_reg, S), v1 = min(v0 + nj_reg, S);
    // f(stamp) of every slot this thread owns
    auto each_stamp = [&](auto&& f) {
      if constexpr (REG) {
#pragma unroll
        for (int j = 0; j < RS; ++j) {
          if (j < nj_reg) f(sr[j]);
        }
      } else {
        for (int j = v0; j < v1; ++j) f(stp[j]);
      }
    };
    // ---- m-th smallest stamp among evictable slots (stamp < step).  One pass by age: the stamps of the last 254 steps
    // have a digit each, everything older shares digit 0.  In a pool in its steady state the victims are some 50 steps
    // old, so the threshold stamp is known after this pass whatever the step number; only when it falls among the older
    // ones (base > 0) do 8-bit MSD radix passes over these follow.  32 sequences, 16384 slots, 280 misses each, with this
    // pass against radix passes alone: steady state 21.6 us against 25.8; a new pool first used at step 300 26.4 against
    // 27.3, at step 70000 29.4 against 28.5; victims 6000 steps old 28.1 against 27.2: there it is one pass too many.
    uint32_t prefix = 0, need = m;
    const uint32_t base = step > 255u ? step - 255u : 0u;
    auto age_digit = [&](uint32_t st) -> uint32_t { return __builtin_elementwise_sub_sat(st, base); };     // <= 254 for st < step
    // counters (cleared here) and the prefix sum over the 256 digits; the digit that holds the need-th smallest
    auto clear_hist = [&]() {
      uint2* h2 = reinterpret_cast<uint2*>(s_hist);
      for (int j = tid; j < 256 * 16; j += BT) h2[j] = make_uint2(0, 0);
      __syncthreads();
    };
    auto find_digit = [&](uint32_t* below_out) {
      __syncthreads();
      uint32_t c = 0, inc = 0;
      if (wave < 4) {                                  // (the other waves only meet the barriers)
        // a thread's 32 copies are consecutive words, so consecutive threads start 32 words apart: the 16-byte
        // pieces are taken in an order rotated by the thread index, which spreads a read over the banks
        const uint4* h4 = reinterpret_cast<const uint4*>(s_hist + tid * 32);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
          const uint4 x = h4[(g + tid) & 7];
          c += x.x + x.y + x.z + x.w;
        }
        inc = wave_incl_scan(c, lane);
        if (lane == 63) sm.wave_tot[wave] = inc;
      }
      __syncthreads();
      if (wave < 4) {
        inc += ess_sel::waves_before<4>(sm.wave_tot, wave, lane);
        const uint32_t below = inc - c;
        if (below < need && inc >= need) { sm.sel_digit = tid; sm.sel_below = below; sm.sel_upto = inc; }
        if (below_out) below_out[tid] = below;
      }
      __syncthreads();
      need -= sm.sel_below;
    };
    uint32_t* const s_below = s_hist + BOOK_BELOW;
    // (the counters were cleared with the bitmap; the barriers of the scan above lie between)
    each_stamp([&](uint32_t st) {
      if (st < step) atomicAdd(&s_hist[age_digit(st) * 32 + (lane & 31)], 1u);
    });
    find_digit(s_below);
    const bool by_age = sm.sel_digit > 0 || base == 0;
    // whether a digit is one stamp for every victim: not if some are older than the digits tell apart (read here, as
    // a long list of victims takes this place)
    const bool one_stamp = base == 0 || s_below[1] == 0;
    if (by_age) {
      prefix = base + sm.sel_digit;
      __syncthreads();
    } else {
      // evictable stamps are < step, so digits above step's top byte are zero for all of them: skip those passes
      // (looking at the older ones alone, stamp <= base, saves a pass up to step 510, but its comparison is not shared with
      // the other loops and makes the kernel 0.25 us longer for everyone)
      need = m;
      const int first_pass = step < (1u << 16) ? 2 : (step < (1u << 24) ? 1 : 0);
      for (int pass = first_pass; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        __syncthreads();
        clear_hist();
        each_stamp([&](uint32_t st) {
          if (st < step && (pass == first_pass || (st >> (shift + 8)) == prefix))
            atomicAdd(&s_hist[((st >> shift) & 255u) * 32 + (lane & 31)], 1u);
        });
        find_digit(nullptr);
        prefix = (prefix << 8) | sm.sel_digit;
        __syncthreads();
      }
    }
    const uint32_t tau = prefix;               // threshold stamp; `need` slots with stamp == tau are taken, lowest slots first
    // ---- collect victims: stamp < tau, plus the first `need` slots (in slot order) with stamp == tau.  The list is in
    // slot order.  Where it is ordered by counting below (one stamp a digit) and there is room, every slot up to tau goes in: the
    // order alone then tells the victims, its first m.  (A pool in its steady state has about as many slots at tau as it needs victims.)
    const uint32_t upto = sm.sel_upto;
    const bool counted = by_rank && by_age && one_stamp;
    const bool all = REG && counted && upto <= (uint32_t)BT;
    const int n_list = all ? (int)upto : (int)m;
    uint32_t* const s_cnt = s_hist + BOOK_CNT;
    s_cnt[tid] = 0;
    if (all) {
      uint32_t n = 0;
#pragma unroll
      for (int j = 0; j < RS; ++j)
        if (j < nj_reg) n += (uint32_t)__popcll(__ballot(sr[j] <= tau));
      if (lane == 0) sm.wave_tot2[wave] = n;
      __syncthreads();
      uint32_t at = ess_sel::waves_before<BT / 64>(sm.wave_tot2, wave, lane);
#pragma unroll
      for (int j = 0; j < RS; ++j) {
        if (j >= nj_reg) continue;
        const uint64_t take = __ballot(sr[j] <= tau);
        if (sr[j] <= tau) s_vict[at + lanes_below(take)] = ((unsigned long long)sr[j] << 32) | (uint32_t)(ws + 64 * j + lane);
        at += (uint32_t)__popcll(take);
      }
    } else
    if constexpr (REG) {
      // counts of the wave by ballot, 16 bits each (at most 16384 slots)
      uint32_t n_eq = 0, n_lt = 0;
#pragma unroll
      for (int j = 0; j < RS; ++j)
        if (j < nj_reg) {
          n_eq += (uint32_t)__popcll(__ballot(sr[j] == tau));
          n_lt += (uint32_t)__popcll(__ballot(sr[j] < tau));
        }
      if (lane == 0) sm.wave_tot2[wave] = n_eq | (n_lt << 16);
      __syncthreads();
      const uint32_t before = ess_sel::waves_before<BT / 64>(sm.wave_tot2, wave, lane);
      uint32_t left = need - min(before & 0xffffu, need);            // slots at the threshold stamp still to be taken
      uint32_t at = (before >> 16) + need - left;                    // victims in front of the next 64 slots
#pragma unroll
      for (int j = 0; j < RS; ++j) {
        if (j >= nj_reg) continue;
        asm volatile("" : "+v"(sr[j]));                              // (the masks of the counts are not worth keeping)
        uint64_t take = __ballot(sr[j] < tau);
        if (left > 0) {
          uint64_t eq = __ballot(sr[j] == tau);
          if ((uint32_t)__popcll(eq) > left) eq = __ballot(sr[j] == tau && lanes_below(eq) < left);
          left -= (uint32_t)__popcll(eq);
          take |= eq;
        }
        if (take) {
          const uint32_t i = at + lanes_below(take);
          if (__builtin_amdgcn_inverse_ballot_w64(take) && i < (uint32_t)vict_cap)
            s_vict[i] = ((unsigned long long)sr[j] << 32) | (uint32_t)(ws + 64 * j + lane);
          at += (uint32_t)__popcll(take);
        }
      }
    } else {
      uint32_t my_eq = 0, my_lt = 0;
      each_stamp([&](uint32_t st) {
        my_eq += (st == tau) ? 1u : 0u;
        my_lt += (st < tau) ? 1u : 0u;
      });
      uint32_t tot_eq, tot_lt;
      uint32_t rank = block_incl_scan(my_eq, sm.wave_tot, &tot_eq) - my_eq;      // slots at the threshold stamp in front of this thread's
      // where this thread's victims go: those of the threads before it come first
      uint32_t at = block_incl_scan(my_lt, sm.wave_tot, &tot_lt) - my_lt + min(rank, need);
      for (int j = v0; j < v1; ++j) {
        const uint32_t st = stp[j];
        bool take = st < tau;
        if (st == tau) { take = rank < need; ++rank; }
        if (take) {
          if (at < (uint32_t)vict_cap) s_vict[at] = ((unsigned long long)st << 32) | (uint32_t)j;
          ++at;
        }
      }
    }
    if (by_rank) s_pre[tid] = (uint16_t)miss_before;       // (read where the lists are built)
    // ---- order the victims by (stamp, slot)
    if (counted) {
      // A digit is one stamp here.  The list is in slot order, so a stable counting sort by age is the order: a victim's place is the number of
      // slots of smaller digits (all of them victims) plus the number of victims with its digit in front of it -- inside its
      // wave by matching the eight digit bits, and the counts of the waves before.  (Was: every key compared with
      // every other, 4.5 us for 280 victims; this takes 1.5.)
      // The former token is asked for as soon as the slot is known, and the pairing follows from the registers.
      uint8_t* const cnt8 = reinterpret_cast<uint8_t*>(s_cnt);         // [256 digits][16 waves]: at most 64 each
      __syncthreads();
      const bool in = tid < n_list;
      unsigned long long my_key = 0;
      uint32_t dg = 0, ahead = 0;
      int my_old = -1;
      if (wave * 64 < n_list) {                        // whole waves
        if (in) {
          my_key = s_vict[tid];
          my_old = to[(uint32_t)my_key];
          dg = age_digit((uint32_t)(my_key >> 32));
        }
        unsigned long long same = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const unsigned long long bal = __ballot((dg >> bit) & 1u);
          same &= ((dg >> bit) & 1u) ? bal : ~bal;
        }
        ahead = lanes_below(same);
        if (in && ahead == 0) cnt8[dg * 16 + wave] = (uint8_t)__popcll(same);
      }
      __syncthreads();
      if (in) {
        ahead += s_below[dg];
        const uint4 c = reinterpret_cast<const uint4*>(s_cnt)[dg];     // the waves in front: their bytes, summed
        const uint32_t cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int n = wave - 4 * x;
          const uint32_t mask = n >= 4 ? 0xffffffffu : (n > 0 ? (1u << (8 * n)) - 1u : 0u);
          ahead = __builtin_amdgcn_sad_u8(cw[x] & mask, 0u, ahead);
        }
        if (ahead < m) {
          s_vict[ahead] = my_key;                      // (every key of the list is in its thread's registers)
          pair(ahead, (int)(uint32_t)my_key, my_old);
        }
      }
    } else if (by_rank) {
      __syncthreads();
      // every victim's rank = the number of smaller keys, counted by BT / m threads per victim, each over its share
      // of the list (LDS broadcast reads), and added up in LDS
      uint32_t* s_rank = reinterpret_cast<uint32_t*>(s_vict + vict_cap / 2);        // the list takes the lower half at most
      const int mr = ((int)m + 63) & ~63;            // threads of one share: whole waves
      const int shares = BT / mr;
      for (int j = tid; j < (int)m; j += BT) s_rank[j] = 0;
      __syncthreads();
      const int i = tid % mr, p = tid / mr;
      unsigned long long my_key = 0;
      if (i < (int)m && p < shares) {
        my_key = s_vict[i];
        const int j0 = (int)((long)m * p / shares), j1 = (int)((long)m * (p + 1) / shares);
        int rk = 0;
        int j = j0;
        for (; j + 8 <= j1; j += 8) {            // eight independent LDS reads in flight (the plain loop waits for each: 280 victims 2.2 us longer)
          unsigned long long x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = s_vict[j + u];
#pragma unroll
          for (int u = 0; u < 8; ++u) rk += x[u] < my_key ? 1 : 0;
        }
        for (; j < j1; ++j) rk += s_vict[j] < my_key ? 1 : 0;
        atomicAdd(&s_rank[i], (uint32_t)rk);
      }
      __syncthreads();
      const int my_rank = (tid < (int)m) ? (int)s_rank[tid] : -1;
      if (tid < (int)m) my_key = s_vict[tid];
      __syncthreads();
      if (my_rank >= 0) s_vict[my_rank] = my_key;
      __syncthreads();
    } else {
      __syncthreads();
      int np = 1;
      while (np < (int)m) np <<= 1;
      for (int j = (int)m + tid; j < np; j += BT) s_vict[j] = ~0ull;
      bitonic_sort_u64(s_vict, np);
    }
    // ---- pair the i-th miss with the i-th victim
    if (!counted)
      for (uint32_t i = tid; i < m; i += BT) {
        const int v = (int)(uint32_t)s_vict[i];
        pair(i, v, to[v]);
      }
  }
  // a miss's place among the misses: the bits before its own in the bitmap
  auto miss_place = [&](int pos) -> uint32_t {
    const int wd = pos >> 5;
    uint32_t i = s_pre[wd >> wsh] + (uint32_t)__popc(bm[wd] & ((1u << (pos & 31)) - 1u));
    for (int x = wd & (int)(~0u << wsh); x < wd; ++x) i += (uint32_t)__popc(bm[x]);
    return i;
  };
  // A miss finds its slot in the victims' list; in a longer list, or where the selection is read again, the table itself tells, once it is written.
  const bool by_list = keep && by_rank;
  __syncthreads();                               // table updates visible to the whole workgroup

  // ---- per (b,t): slot of every selected entry, and the compacted hit / fetched lists
  if (slot_idx_out == nullptr && hit_list == nullptr) continue;
  if (keep) {
    // Entry u * BT + tid of the sequence was looked up by this thread in round u: a hit keeps the slot it had, a miss got
    // its slot in the pairing above (all reads of a thread in flight together).  A query token's list is whole rounds,
    // so one exchange of the waves' counts serves all of them.
    const int rounds = nsel / BT, per_t = kk / BT;
    uint32_t* const lists_tot = s_hist + BOOK_LISTS;
    uint32_t ex[4];
    int sl[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool fresh = u < rounds && sv[u] >= 0 && slv[u] < 0;
      sl[u] = u < rounds && sv[u] >= 0 ? slv[u] : -1;
      if (fresh) sl[u] = by_list ? (int)(uint32_t)s_vict[miss_place(sv[u])] : so[sv[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= rounds) break;
      const size_t at = (size_t)b * nsel + u * BT + tid;
      const bool fresh = sv[u] >= 0 && slv[u] < 0;
      if (slot_idx_out) slot_idx_out[at] = sl[u];
      if (fresh_idx) fresh_idx[at] = fresh ? sl[u] | ESS_FRESH_BIT : sl[u];
      const uint64_t hits = __ballot(sl[u] >= 0 && !fresh), misses = __ballot(sl[u] >= 0 && fresh);
      ex[u] = lanes_below(fresh ? misses : hits);
      if (lane == 0) lists_tot[u * (BT / 64) + wave] = (uint32_t)__popcll(hits) | ((uint32_t)__popcll(misses) << 16);
    }
    __syncthreads();
    if (!hit_list) continue;
    // one read for the totals of all rounds: a row of 16 lanes holds a round's waves (counts: hits | misses << 16)
    const uint32_t upto_wave = ess_sel::row_incl_scan(lists_tot[lane]);
    uint32_t run = 0;                              // the query token's rounds so far
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= rounds) break;
      const int t = u / per_t;
      if (u % per_t == 0) run = 0;
      uint32_t off = run;
      if (wave > 0) off += (uint32_t)__builtin_amdgcn_readlane((int)upto_wave, u * 16 + wave - 1);
      const size_t rowoff = ((size_t)b * T + t) * kk;
      if (sl[u] >= 0) {
        if (slv[u] < 0) miss_list[rowoff + (off >> 16) + ex[u]] = sl[u];
        else hit_list[rowoff + (off & 0xffffu) + ex[u]] = sl[u];
      }
      run += (uint32_t)__builtin_amdgcn_readlane((int)upto_wave, u * 16 + 15);
      if (u % per_t == per_t - 1 && tid == 0) {
        n_hit[b * T + t] = (int32_t)(run & 0xffffu);
        n_miss[b * T + t] = (int32_t)(run >> 16);
      }
    }
    if constexpr (DYN) __syncthreads();            // lists_tot is free for the next sequence
    continue;
  }
  for (int t = 0; t < T; ++t) {
    const size_t rowoff = ((size_t)b * T + t) * kk;
    uint32_t base_hit = 0, base_miss = 0;
    for (int j0 = 0; j0 < kk; j0 += BT) {
      const int j = j0 + tid;
      int slot = -1;
      bool fresh = false;
      if (j < kk) {
        const int s = idx[rowoff + j];
        if (s >= 0 && s < Lmax) {
          slot = so[s];
          fresh = (bm[s >> 5] >> (s & 31)) & 1u;
        }
        if (slot_idx_out) slot_idx_out[rowoff + j] = slot;
        if (fresh_idx) fresh_idx[rowoff + j] = fresh ? slot | ESS_FRESH_BIT : slot;
      }
      if (hit_list) {
        const uint32_t is_hit = (slot >= 0 && !fresh) ? 1u : 0u;
        const uint32_t is_miss = (slot >= 0 && fresh) ? 1u : 0u;
        uint32_t tot;
        const uint32_t inc = block_incl_scan(is_hit | (is_miss << 16), sm.wave_tot, &tot);
        const uint32_t ex = inc - (is_hit | (is_miss << 16));
        if (is_hit) hit_list[rowoff + base_hit + (ex & 0xffffu)] = slot;
        if (is_miss) miss_list[rowoff + base_miss + (ex >> 16)] = slot;
        base_hit += tot & 0xffffu;
        base_miss += tot >> 16;
      }
    }
    if (hit_list && tid == 0) {
      n_hit[b * T + t] = (int32_t)base_hit;
      n_miss[b * T + t] = (int32_t)base_miss;
    }
  }
  }
}

// Fetch: one wave per missed entry, rows copied host pool -> slot pool in 16-byte pieces, two
// entries per wave in flight at once.  The kernel is a handful of 512-thread workgroups that loop
// over all sequences: its waves spend their life waiting on the host link.  The number of workgroups
// sets how many bytes are in flight on the link: 64 (1.2 MB in flight) reach 53 GB/s, 32 reach
// 50 GB/s, 16 reach 48 GB/s, 8 only 27 GB/s.  The long host reads also fill the L2 request queues of
// the XCDs the workgroups sit on, and every other memory access of those XCDs waits behind them: a
// kernel beside a 64-workgroup fetch spread over the chip takes about 2.2x its time alone (a
// latency-bound one more), beside 28-32 workgroups about 1.3x.  The launcher can therefore confine
// the fetch to some XCDs (`only_xcds`: the other workgroups exit, entries are handed out by ticket),
// and the kernels beside it stay off those (ess_xcd).
constexpr int FILL_WPB = 8;                                 // waves per workgroup
constexpr int FILL_MAX_B = 4096;

__global__ __launch_bounds__(FILL_WPB * 64) void k_fill(const ess_fetch f, uint32_t only_xcds, uint32_t* __restrict__ ticket) {
  // confined fetch: only workgroups on the XCDs in `only_xcds` work (or, should none sit there, the last one to
  // arrive), entries are handed out through `ticket`
  __shared__ int s_join;
  if (only_xcds && !ess_ticket_join(ticket, (only_xcds >> ess_xcc_id()) & 1u, &s_join)) return;
  extern __shared__ int32_t pref[];                          // [B + 1] pref[b] = entries of sequences < b (kept small:
                                                             // the kernel must fit beside workgroups that fill the LDS)
  const int tid = threadIdx.x, lane = tid & 63;
  const int gw = blockIdx.x * FILL_WPB + (tid >> 6);         // wave index in the grid
  const int FILL_WAVES = gridDim.x * FILL_WPB;
  if (!only_xcds) {
    ess_fill::entries<2>(f, pref, gw, FILL_WAVES);
    return;
  }
  const int M = ess_fill::prefix(f.miss_cnt, f.fill_cap, f.B, pref);
  const int chunks = f.row_stride >> 4;                      // <= 128 for the supported entry sizes
  const int c0 = lane, c1 = lane + 64;
  for (;;) {                                                 // entries r, r + 1 by ticket: two of this wave in flight
    uint32_t tk = 0;
    if (lane == 0) tk = atomicAdd(ticket, 2u);
    const int r = (int)__shfl(tk, 0, 64);
    if (r >= M) break;
    const bool two = r + 1 < M;
    const uint4 *srcA, *srcB;
    uint4 *dstA, *dstB;
    ess_fill::locate(f, pref, r, srcA, dstA);
    ess_fill::locate(f, pref, two ? r + 1 : r, srcB, dstB);
    uint4 a0 = make_uint4(0, 0, 0, 0), a1 = a0, b0 = a0, b1 = a0;
    if (c0 < chunks) a0 = srcA[c0];
    if (c1 < chunks) a1 = srcA[c1];
    if (two && c0 < chunks) b0 = srcB[c0];
    if (two && c1 < chunks) b1 = srcB[c1];
    if (c0 < chunks) ess_store_nt(dstA + c0, a0);
    if (c1 < chunks) ess_store_nt(dstA + c1, a1);
    if (two && c0 < chunks) ess_store_nt(dstB + c0, b0);
    if (two && c1 < chunks) ess_store_nt(dstB + c1, b1);
  }
}

// rows_out[b,t,j,:] = slot_pool[b, slot_idx[b,t,j], :] (zeros where the slot is -1).  A wave takes sixteen entries, their
// slots in one load, and copies four rows at a time.
// WHICH 1, 2: slot_idx marks the entries that this step fetches (ESS_FRESH_BIT); the others are gathered while the fetch
// runs, these after it.
constexpr int GATHER_ROWS = 16;
template <int WHICH>
__device__ __forceinline__ void gather_rows(int part, int b, const uint8_t* __restrict__ slot_pool,
                                            const int32_t* __restrict__ slot_idx, int per_seq, int S,
                                            int row_stride, uint8_t* __restrict__ rows_out) {
  const int lane = threadIdx.x & 63;
  const int i0 = (part * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * GATHER_ROWS;
  if (i0 >= per_seq) return;
  const int chunks = row_stride >> 4;                        // <= 128
  const bool in = lane < GATHER_ROWS && i0 + lane < per_seq;
  int v = in ? slot_idx[(size_t)b * per_seq + i0 + lane] : -1;
  bool mine = in;
  if (WHICH) {
    const bool fresh = v >= 0 && (v & ESS_FRESH_BIT);
    mine = in && fresh == (WHICH == 2);
    if (fresh) v &= ~ESS_FRESH_BIT;
  }
  uint32_t todo = (uint32_t)__ballot(mine);
  const uint8_t* pool = slot_pool + (size_t)b * S * row_stride;
  uint8_t* out = rows_out + ((size_t)b * per_seq + i0) * row_stride;
  while (todo) {
    uint4 x[4], y[4];
    int row[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      row[u] = todo ? __ffs(todo) - 1 : -1;
      if (row[u] < 0) continue;
      todo &= todo - 1;
      const int s = __builtin_amdgcn_readlane(v, row[u]);
      x[u] = y[u] = make_uint4(0, 0, 0, 0);
      if (s >= 0 && s < S) {
        const uint4* src = reinterpret_cast<const uint4*>(pool + (size_t)s * row_stride);
        if (lane < chunks) x[u] = src[lane];
        if (lane + 64 < chunks) y[u] = src[lane + 64];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (row[u] < 0) continue;
      uint4* dst = reinterpret_cast<uint4*>(out + (size_t)row[u] * row_stride);
      if (lane < chunks) dst[lane] = x[u];
      if (lane + 64 < chunks) dst[lane + 64] = y[u];
    }
  }
}

template <int WHICH>
__global__ __launch_bounds__(256) void k_gather_rows(const uint8_t* __restrict__ slot_pool, const int32_t* __restrict__ slot_idx,
                                                     int per_seq, int S, int row_stride, uint8_t* __restrict__ rows_out) {
  gather_rows<WHICH>(blockIdx.x, blockIdx.y, slot_pool, slot_idx, per_seq, S, row_stride, rows_out);
}

// The fetch and the gather of the rows that were resident in one launch (see ess_fetch for the roles): the two touch different
// slots.  `parts` workgroups gather a sequence.
__global__ __launch_bounds__(256) void k_fill_gather(const ess_fetch f, const int32_t* __restrict__ slot_idx, int per_seq, int parts,
                                                     uint8_t* __restrict__ rows_out) {
  extern __shared__ int32_t pref[];                          // [B + 1]
  const int i = blockIdx.x, low = i & 7;
  if (low < 2) {
    const int wg = 2 * (i >> 3) + low;
    if (wg < f.wgs) ess_fill::entries<2>(f, pref, wg * 4 + (int)(threadIdx.x >> 6), f.wgs * 4);
    return;
  }
  const int item = 6 * (i >> 3) + low - 2, b = item / parts;
  if (b < f.B) gather_rows<1>(item - b * parts, b, f.slot_pool, slot_idx, per_seq, f.S, f.row_stride, rows_out);
}

// Append (Sec. 3.3): the entries a step produced enter the caches.  One workgroup per sequence; for each
// of its T new tokens, in order: index key -> Indexer-Cache row p, entry -> host pool row p (stores
// through the device mapping of the pinned pool: the write-back to the Total Memory Pool), and admission
// to the slot pool as most recently used: the slot smallest in (stamp, slot) among slots with a stamp
// below `step` is taken -- the victim rule of the bookkeeping -- or, with every slot on stamp `step`,
// none (the entry then lives in the host pool only).  Without a host pool slot = position.
// OFFLOADED false: without a host pool, a form of its own: a resident append has no use for the stamps, and with their 16
// registers and the search beside it it took 0.6 us longer (6 sequences, two tokens: 4.8 us, now 4.2).
// What bounds it: a launch (3.5 us) and the chain context length -> page -> stores.  So all that does not wait for it -- stamps, new keys and
// rows of all tokens, each by threads of its own -- is asked for at the start; the tokens' victims are found one after the
// other from registers, a wave's smallest by lane moves in 32 bits (stamp, then slot); the tables are written at the end.  (Before, each token in turn loaded its rows, compared 64-bit keys through the LDS and waited
// for its victim's former token.)  us, before / now: 23 sequences, 9001 slots, two tokens, paged 8.6 / 7.1; 8 sequences, 20000 slots,
// four tokens, a call 21.8 / 14.3; a whole step of 10 sequences, two tokens, with its append 89.4 / 87.4.
constexpr int APPEND_NT = 1024;
constexpr int APPEND_T = 4;                      // query tokens at most
// smallest of the 64 lanes' values, in all lanes (see wave_max)
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  auto with = [&](auto ctrl, auto rows) {
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
  };
  using std::integral_constant;
  with(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
  with(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
  with(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
template <bool OFFLOADED>
__global__ __launch_bounds__(APPEND_NT) void k_append(
    const uint8_t* __restrict__ new_key, const uint8_t* __restrict__ new_rows, uint8_t* __restrict__ key,
    uint8_t* __restrict__ host_pool, uint8_t* __restrict__ slot_pool, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ token_of, uint32_t* __restrict__ stamp, int32_t* __restrict__ ctx_len,
    int32_t* __restrict__ placed, int T, int Di, int Lmax, int S, int row_stride, uint32_t step,
    const float* __restrict__ new_scale, const int32_t* __restrict__ block_table, int n_pages) {
  __shared__ uint2 red[APPEND_T][APPEND_NT / 64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* stp = stamp + (size_t)b * S;
  const int kchunks = Di >> 4, rchunks = row_stride >> 4;        // at most 8 and 128
  // threads 128 t .. bring the row of token t, threads 512 + 16 t .. its key, thread 512 + 16 t + 15 its scale
  const int rt = tid >> 7, rc = tid & 127, kt = (tid - 512) >> 4, kc = (tid - 512) & 15;
  const bool my_row = rt < T && rc < rchunks, my_key = tid >= 512 && kt < T && kc < kchunks, my_scale = tid >= 512 && kt < T && kc == 15 && new_scale;
  uint4 piece = make_uint4(0, 0, 0, 0);
  float scale = 0.f;
  if (my_row) piece = reinterpret_cast<const uint4*>(new_rows + ((size_t)b * T + rt) * row_stride)[rc];
  if (my_key) piece = reinterpret_cast<const uint4*>(new_key + ((size_t)b * T + kt) * Di)[kc];
  if (my_scale) scale = new_scale[(size_t)b * T + kt];
  // the stamps of a thread's slots (tid, tid + 1024, ..)
  constexpr int AS = 16;
  const bool held = OFFLOADED && S <= APPEND_NT * AS;
  uint32_t sr[AS];
  if (held) {
#pragma unroll
    for (int j = 0; j < AS; ++j) sr[j] = tid + j * APPEND_NT < S ? stp[tid + j * APPEND_NT] : 0xffffffffu;
  }
  const int L0 = max(0, min(ctx_len[b], Lmax));
  int n = min(T, Lmax - L0);
  // paged Indexer-Cache: a token needs a mapped page; the first one without stops the append
  const int32_t* bt = block_table ? block_table + (size_t)b * (Lmax / ESS_PAGE_TOKENS) : nullptr;
  if (bt)
    for (int t = 0; t < n; ++t) {
      const int pid = bt[(L0 + t) / ESS_PAGE_TOKENS];
      if (pid < 0 || pid >= n_pages) { n = t; break; }
    }
  // keys, and rows to the host pool
  if (tid >= 512 && kt < n) {
    const int p = L0 + kt;
    if (bt) {
      uint8_t* page = key + (size_t)bt[p / ESS_PAGE_TOKENS] * ((size_t)ESS_PAGE_TOKENS * (Di + 4));
      const int r = p % ESS_PAGE_TOKENS;
      if (my_key) reinterpret_cast<uint4*>(page + (size_t)r * Di)[kc] = piece;
      if (my_scale) reinterpret_cast<float*>(page + (size_t)ESS_PAGE_TOKENS * Di)[r] = scale;
    } else if (my_key) {
      reinterpret_cast<uint4*>(key + ((size_t)b * Lmax + p) * Di)[kc] = piece;
    }
  }
  if (OFFLOADED && my_row && rt < n) reinterpret_cast<uint4*>(host_pool + ((size_t)b * Lmax + L0 + rt) * row_stride)[rc] = piece;
  // slot of each token: its position, or the smallest in (stamp, slot) of those below `step`, each taken once
  int v[APPEND_T];
#pragma unroll
  for (int t = 0; t < APPEND_T; ++t) v[t] = t < n ? L0 + t : -1;
  if constexpr (OFFLOADED) {
    uint2 best = make_uint2(0xffffffffu, 0xffffffffu);         // the thread's smallest: stamp, slot
    auto mine = [&](int taken) {                   // ... of its slots but those taken
      best = make_uint2(0xffffffffu, 0xffffffffu);
      auto look = [&](uint32_t x, int s) {
        bool free_slot = s < S && x < step && x < best.x;      // (slots in ascending order: of equal stamps the first)
#pragma unroll
        for (int t = 0; t < APPEND_T; ++t) free_slot = free_slot && !(t < taken && v[t] == s);
        if (free_slot) best = make_uint2(x, (uint32_t)s);
      };
      if (held) {
#pragma unroll
        for (int j = 0; j < AS; ++j) look(sr[j], tid + j * APPEND_NT);
      } else {
        for (int s = tid; s < S; s += APPEND_NT) look(stp[s], s);
      }
    };
    mine(0);
#pragma unroll
    for (int t = 0; t < APPEND_T; ++t) {
      if (t >= n) break;                           // (the same in all threads)
      const uint32_t lo = wave_min_u32(best.x), at = wave_min_u32(best.x == lo ? best.y : 0xffffffffu);
      if (lane == 0) red[t][wave] = make_uint2(lo, at);
      __syncthreads();
      const uint2 r = lane < APPEND_NT / 64 ? red[t][lane] : make_uint2(0xffffffffu, 0xffffffffu);
      const uint32_t all = wave_min_u32(r.x), slot = wave_min_u32(r.x == all ? r.y : 0xffffffffu);
      v[t] = all == 0xffffffffu ? -1 : (int)slot;
      if (t + 1 < n && v[t] >= 0 && v[t] % APPEND_NT == tid) mine(t + 1);      // (after the last token nobody asks)
    }
  } else {
    __syncthreads();                               // (everyone has read ctx_len)
  }
#pragma unroll
  for (int t = 0; t < APPEND_T; ++t)
    if (v[t] >= 0 && rt == t && rc < rchunks) reinterpret_cast<uint4*>(slot_pool + ((size_t)b * S + v[t]) * row_stride)[rc] = piece;
  // The tables: one thread, token by token (a former token may be a position that this very call fills: a context that was
  // cut back), the former tokens asked for together.
  if (tid == APPEND_NT - 64) {
    int32_t* so = slot_of + (size_t)b * Lmax;
    int32_t* to = token_of + (size_t)b * S;
    int old[APPEND_T];
#pragma unroll
    for (int t = 0; t < APPEND_T; ++t) old[t] = v[t] >= 0 ? to[v[t]] : -1;
#pragma unroll
    for (int t = 0; t < APPEND_T; ++t) {
      if (v[t] >= 0) {
        if (old[t] >= 0) so[old[t]] = -1;
        to[v[t]] = L0 + t;
        so[L0 + t] = v[t];
        stp[v[t]] = step;
      }
      if (t < T && placed) placed[(size_t)b * T + t] = v[t];   // no room, no page or no slot: -1
    }
  }
  if (tid == 0) ctx_len[b] = L0 + n;               // (every thread has read it: a barrier lies between, or nothing is appended)
}

__global__ __launch_bounds__(256) void k_calib_copy(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

// Reads `n` 16-byte pieces and leaves one word per workgroup, so that the loads are not dead.  A workgroup streams
// one contiguous range (`per_wg` pieces); its four waves interleave 8 KiB pieces, each wave instruction covering
// 1 KiB, eight of them in flight per wave -- the pattern with which a pure read stream is fastest on this chip.
__global__ __launch_bounds__(256) void k_calib_read(const uint4* __restrict__ src, size_t n, size_t per_wg,
                                                    uint32_t* __restrict__ sink) {
  constexpr int U = 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t lo = (size_t)blockIdx.x * per_wg;
  const size_t hi = lo + per_wg < n ? lo + per_wg : n;
  uint32_t acc = 0;
  for (size_t base = lo + (size_t)wave * U * 64; base < hi; base += (size_t)4 * U * 64) {
    uint4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = base + (size_t)u * 64 + lane;
      x[u] = i < hi ? src[i] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= x[u].x ^ x[u].y ^ x[u].z ^ x[u].w;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) acc ^= __shfl_xor(acc, d, 64);
  if (lane == 0) atomicXor(&sink[blockIdx.x], acc);
}

__global__ void k_fill_u32(uint32_t* p, int n, uint32_t value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

__global__ void k_cache_reset(int32_t* slot_of, int32_t* token_of, uint32_t* stamp, int Lmax, int S, int identity) {
  const int b = blockIdx.y;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < Lmax) slot_of[(size_t)b * Lmax + i] = identity ? i : -1;
  if (i < S) {
    token_of[(size_t)b * S + i] = identity ? i : -1;
    stamp[(size_t)b * S + i] = 0;
  }
}

}  // namespace

int ess_launch_append(const ess_config& c, const ess_cache& cache, const uint8_t* new_key, const uint8_t* new_rows,
                      uint8_t* key, int32_t* ctx_len, int B, int T, uint32_t step, int32_t* placed,
                      const float* new_scale, const int32_t* block_table, int n_pages, hipStream_t st) {
  auto kern = cache.host_pool_dev ? &k_append<true> : &k_append<false>;
  hipLaunchKernelGGL(kern, dim3(B), dim3(APPEND_NT), 0, st, new_key, new_rows, key,
                     const_cast<uint8_t*>(cache.host_pool_dev), cache.slot_pool, cache.slot_of, cache.token_of,
                     cache.stamp, ctx_len, placed, T, c.idx_dim, c.max_ctx, c.slots_per_seq, c.row_stride, step,
                     block_table ? new_scale : nullptr, block_table, n_pages);   // (flat keys have no scales: what the caller gave is not read)
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_calib_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
  hipLaunchKernelGGL(k_calib_copy, dim3(8192), dim3(256), 0, st, static_cast<uint4*>(dst), static_cast<const uint4*>(src),
                     bytes / 16);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_calib_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t st) {
  const size_t n = bytes / 16;
  size_t per_wg = 16384;                                     // 256 KiB per workgroup, more when that needs too many workgroups
  while ((n + per_wg - 1) / per_wg > ESS_CALIB_READ_WGS) per_wg *= 2;
  const unsigned grid = (unsigned)((n + per_wg - 1) / per_wg);
  hipLaunchKernelGGL(k_calib_read, dim3(grid ? grid : 1), dim3(256), 0, st, static_cast<const uint4*>(src), n, per_wg, sink);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

// hist[x] += 1 for the XCD x this workgroup runs on
__global__ void k_xcd_probe(uint32_t* hist) {
  if (threadIdx.x == 0) atomicAdd(&hist[ess_xcc_id() & 7], 1u);
}

// Are 64 workgroups spread evenly over eight XCDs (8 each)?  Only then may a launch count on finding
// eight minus n of any eight consecutive workgroups off a set of n XCDs.  `hist8`: eight zeroed counters, zero again on return.
int ess_probe_xcds(uint32_t* hist8, bool* even) {
  hipLaunchKernelGGL(k_xcd_probe, dim3(64), dim3(64), 0, 0, hist8);
  ESS_HIP(hipGetLastError());
  uint32_t h[8];
  ESS_HIP(hipMemcpy(h, hist8, sizeof(h), hipMemcpyDeviceToHost));
  ESS_HIP(hipMemset(hist8, 0, sizeof(h)));
  *even = true;
  for (int i = 0; i < 8; ++i) *even = *even && h[i] == 8u;
  return ESS_OK;
}

int ess_launch_fill_u32(uint32_t* p, int n, uint32_t value, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_u32, dim3((n + 255) / 256), dim3(256), 0, st, p, n, value);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_cache_reset(const ess_config& c, const ess_cache& cache, int B, hipStream_t st) {
  const int n = c.max_ctx > c.slots_per_seq ? c.max_ctx : c.slots_per_seq;
  hipLaunchKernelGGL(k_cache_reset, dim3((n + 255) / 256, B), dim3(256), 0, st, cache.slot_of, cache.token_of,
                     cache.stamp, c.max_ctx, c.slots_per_seq, cache.host_pool_dev == nullptr ? 1 : 0);
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_bookkeeping(ess_ctx* ctx, const ess_cache& cache, const int32_t* idx, int B, int T, int kk,
                           uint32_t step, int32_t* slot_idx, int32_t* miss_count_out, hipStream_t st, int b0,
                           bool count_step, ess_xcd xcd, uint32_t* zero_tickets, int n_zero_tickets, hipEvent_t done, int32_t* fresh_idx) {
  const ess_config& c = ctx->cfg;
  if (!ctx->book_fits)
    return ess_fail(ESS_ERR_UNSUPPORTED, "the cache bookkeeping of max_ctx %d with T*k = %d does not fit the LDS (max_ctx / 8 + "
                    "12 * T*k bytes must stay below 160 KiB)", c.max_ctx, c.max_q_tokens * c.topk);
  const int cap = c.max_q_tokens * c.topk;
  const size_t lds = book_lds_bytes(c.max_ctx, cap);
  const bool lists = (kk == c.topk);           // compacted lists have the pitch of the top-k
  const size_t lo = (size_t)b0 * T * c.topk;   // offset of this sub-batch in the per-(b,t) lists
  const bool reg = c.slots_per_seq <= BT * 16;
  auto kern = xcd.ticket ? (reg ? &k_bookkeeping<true, true> : &k_bookkeeping<false, true>)
                         : (reg ? &k_bookkeeping<true, false> : &k_bookkeeping<false, false>);
  ESS_HIP(ess_launch_done(done, kern, dim3(ess_xcd_grid(B, xcd)), dim3(BT), lds, st, idx, T, kk, c.max_ctx, c.slots_per_seq,
                     cache.slot_of, cache.token_of, cache.stamp, step, slot_idx, fresh_idx,
                     lists ? ctx->hit_list + lo : nullptr, lists ? ctx->miss_list + lo : nullptr,
                     ctx->n_hit + (size_t)b0 * T, ctx->n_miss + (size_t)b0 * T, ctx->fill_tok + (size_t)b0 * cap,
                     ctx->fill_slot + (size_t)b0 * cap, cap, ctx->miss_cnt + b0, miss_count_out, ctx->stats, ctx->seq_stats + 4 * (size_t)b0,
                     c.row_stride, count_step ? 1 : 0, (c.flags & ESS_FLAG_AUTO) ? ctx->host_miss_dev + b0 : nullptr, xcd, B,
                     zero_tickets, n_zero_tickets, (int)book_words(c.max_ctx), (int)book_union_bytes(cap)));
  return ESS_OK;
}

// At context creation (on the context's device): the bookkeeping kernels keep their arrays in dynamic LDS (see
// BookShared).  The limit is a property of the function, shared by all contexts: it only grows.  A configuration
// whose arrays do not fit the CU's 160 KiB (a selection of 8192 entries per sequence together with a context
// above 500K) cannot use the cache calls: *fits tells.
int ess_init_cache_kernels(const ess_config& c, bool* fits) {
  static size_t have = 0;
  const size_t lds = book_lds_bytes(c.max_ctx, c.max_q_tokens * c.topk);
  *fits = lds + 256 <= 160 * 1024;             // + the kernel's small static arrays
  if (!*fits || lds <= have) return ESS_OK;
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bookkeeping<true, false>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bookkeeping<false, false>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bookkeeping<true, true>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bookkeeping<false, true>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  have = lds;
  return ESS_OK;
}

ess_fetch ess_fetch_of(ess_ctx* ctx, const ess_cache& cache, int B, int b0, int wgs) {
  const ess_config& c = ctx->cfg;
  const int cap = c.max_q_tokens * c.topk;
  return ess_fetch{cache.host_pool_dev, cache.slot_pool, ctx->fill_tok + (size_t)b0 * cap, ctx->fill_slot + (size_t)b0 * cap, ctx->miss_cnt + b0,
                   cap, B, c.max_ctx, c.slots_per_seq, c.row_stride, wgs};
}

int ess_launch_fill(ess_ctx* ctx, const ess_cache& cache, int B, hipStream_t st, int b0, int wgs, uint32_t only_xcds,
                    uint32_t* ticket, hipEvent_t done) {
  wgs = wgs < 1 ? 1 : (wgs > 256 ? 256 : wgs);
  if (only_xcds) {                             // `wgs` workgroups on the chosen XCDs, if any 8 consecutive ones cover all XCDs
    if (!ticket) return ess_fail(ESS_ERR_INVALID_ARG, "internal: confined fetch without a ticket");
    const int on = __builtin_popcount(only_xcds & 0xffu);
    wgs = (wgs + on - 1) / on * 8;
    if (ctx->ticket_grid > 0) wgs = ctx->ticket_grid;
  }
  ESS_HIP(ess_launch_done(done, &k_fill, dim3(wgs), dim3(FILL_WPB * 64), (size_t)(B + 1) * sizeof(int32_t), st,
                          ess_fetch_of(ctx, cache, B, b0, wgs), only_xcds, ticket));
  return ESS_OK;
}

// which: 0 every row, 1 the rows that were resident, with the fetch of the others in the same launch, 2 the fetched ones
int ess_launch_gather_rows(ess_ctx* ctx, const ess_cache& cache, const int32_t* slot_idx, int B, int T, uint8_t* rows_out, hipStream_t st, int which) {
  const ess_config& c = ctx->cfg;
  const int wgs = (T * c.topk + 4 * GATHER_ROWS - 1) / (4 * GATHER_ROWS);
  if (which == 1) {
    const int fetch_wgs = 2 * 64;                             // of 4 waves: the bytes in flight of the fetch kernel's 64
    const long gather = ((long)wgs * B + 5) / 6;              // groups of eight workgroups
    const long groups = gather > fetch_wgs / 2 ? gather : fetch_wgs / 2;
    hipLaunchKernelGGL(k_fill_gather, dim3((unsigned)(groups * 8)), dim3(256), (size_t)(B + 1) * sizeof(int32_t), st,
                       ess_fetch_of(ctx, cache, B, 0, fetch_wgs), slot_idx, T * c.topk, wgs, rows_out);
  } else {
    auto kern = which == 0 ? &k_gather_rows<0> : &k_gather_rows<2>;
    hipLaunchKernelGGL(kern, dim3(wgs, B), dim3(256), 0, st, cache.slot_pool, slot_idx, T * c.topk, c.slots_per_seq, c.row_stride, rows_out);
  }
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}
