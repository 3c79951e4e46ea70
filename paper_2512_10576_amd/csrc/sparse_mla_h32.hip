// Stage 4 for few rows, short lists and few heads: SparseMLA decode with 32 heads per workgroup.  The kernel in
// sparse_mla.hip gives a workgroup all 128 heads, one wave per 32 of them: an entry is brought from memory once, but a
// workgroup starts with 144 KiB of queries, ends with 128 KiB of results, and 16 heads use one wave of four.  Here a
// workgroup owns 32 heads and its eight waves share every tile: over entries and heads in the first product, over the value
// columns in the second.  It can also finish a row: merge its result with partial results written before it.
#include "attn_common.h"
#include "fetch.h"
#include <type_traits>

namespace {

constexpr int HT = 32;                             // heads per workgroup
constexpr int ET = 64;                             // entries per tile
constexpr int NT = 512;                            // eight waves, two per SIMD
constexpr int NW = NT / 64;
constexpr int MAX_LIST = 4 * NT;                   // list entries of a row at most: four per thread
constexpr int BF_BUF = ET * TRP + ET * 128;        // a tile: latent parts, then rope parts
constexpr int F8_BUF = ET * F8_PITCH;              // ... quantised, the entries as they are
constexpr int MAX_PREV = ESS_FINAL_PREV;
constexpr int OH_PITCH = 144;                      // 64 columns of a head as fp16, staged for 128-byte stores
constexpr int OF_PITCH = 272;                      // ... as fp32, for the merge
constexpr int WT_WORDS = MAX_PREV * HT;            // per wave: weights of earlier partial results

// LDS of a workgroup
template <int FMT>
struct Lay {
  static constexpr bool kBf = FMT == ESS_FMT_BF16;
  static constexpr int NBUF = kBf ? 2 : 3, BUF = kBf ? BF_BUF : F8_BUF;
  // probabilities of a tile, 128 bytes per head.  bf16: over the rope parts of the tile they belong to, which nothing reads
  // any more.  Quantised: an image per group of 128 columns, times the group's scale of the entry.
  static constexpr int P_BYTES = HT * 128, P_OFF = NBUF * BUF;
  static constexpr int X_OFF = P_OFF + (kBf ? 0 : 4 * P_BYTES);      // [HT][4] maxima, later sums, per head and group of 16 entries
  static constexpr int SLOT_OFF = X_OFF + HT * 16;                   // the row's list; after the loop [HT][8] largest results per head and wave
  static constexpr int BYTES = SLOT_OFF + MAX_LIST * 4;
  static constexpr int Q_OFF = (NBUF - 1) * BUF;                     // the queries on their way to registers, laid out like a bf16 tile
  static_assert(Q_OFF + HT * (TRP + 128) + 512 <= X_OFF, "the queries fit behind the first tiles");
  static_assert(NW * (32 * OF_PITCH + WT_WORDS * 4) <= X_OFF, "staged results fit the tiles");
  static_assert(BYTES <= 163840 - 256, "LDS of a CU");
};

typedef int int2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) int2v lds_int2v;

// every LDS access of this wave is done, and every wave has come here; memory loads stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float quad_max(float x) {     // over lanes l, l ^ 16, l ^ 32, l ^ 48
  uint2v a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return pair_max(fmaxf(__uint_as_float(a.x), __uint_as_float(a.y)));
}
__device__ __forceinline__ float quad_sum(float x) {
  uint2v a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return pair_sum(__uint_as_float(a.x) + __uint_as_float(a.y));
}
__device__ __forceinline__ float max4(const floatx4& v) { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); }
__device__ __forceinline__ floatx4 lds_float4(const float* p) { return *reinterpret_cast<const floatx4*>(p); }

// eight fp8 values as bf16 (exact)
__device__ __forceinline__ bf16x8 widen(uint32_t lo, uint32_t hi) {
  union { bf16x2 p[4]; bf16x8 v; } u;
  u.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
  u.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
  u.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
  u.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
  return u.v;
}

template <int N, typename F> __device__ __forceinline__ void unroll(F f) {
  [&]<int... I>(std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }(std::make_integer_sequence<int, N>{});
}

// ---------------------------------------------------------------- the kernel
// One workgroup: 32 heads, one range of a row's list, eight waves.  A tile is 64 entries, gathered straight into LDS (bf16 as
// 1024 + 128 bytes a row, quantised as they are).
//   S^T[r,h]  first product, v_mfma_f32_16x16x32_bf16: wave (eg, hb) has entries 16 eg .. and heads 16 hb ..; queries in registers
//   softmax   the waves' maxima meet in LDS, P goes to LDS as bf16
//   O^T[v,h]  second product, v_mfma_f32_32x32x16_bf16: wave w has value columns 64 w .. of all 32 heads, 32 accumulators
// Quantised entries are never written back as bf16: an fp8 value is exact in bf16, so fragments are widened on their way
// into the matrix core, an entry's scale (one per 128 dimensions) multiplies the partial logits of its group, and P for the
// group's columns.  Nothing is rounded that k_attn_partial_tr does not round, and its rounding of scale times value falls
// away: error against 64 bits 2.0e-3 instead of 2.5e-3 (2-norm, N(0,1) entries), log-sum-exp 1e-6 instead of 2e-4.
// What bounds it.  Short ranges: the chain of list, gathers, products and stores, about 7 us of which a lane issues for
// most -- an instruction of one wave takes five cycles, so the code before and after the loop is kept short (a first form
// with 1340 instructions before the loop took 2 us longer).  Long ranges: LDS, 316 KB a tile (K twice, V, P eight times,
// the gathers), 2500 cycles at 128 bytes a clock; measured 1.2 us a tile (bf16), 1.6 (quantised).  An eight-wave form is faster than one
// of four waves (1.95 us a tile); one whose waves own their entries with all value columns, without a barrier, takes
// 0.75 us a tile, but 4.4 us to add up the four waves' accumulators at the end.
// us a launch, merge included, k_attn_partial_tr / this: 1 row of 2048 entries, 128 heads 16.0 / 12.4, 16 rows 28.0 / 23.9, 2 x 16 rows
// with 16 heads 25.5 / 20.5; see pick_form for where the line lies.
template <int FMT, bool DYN>
__global__ __launch_bounds__(NT, 2) void k_attn_h32(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ pool, const int32_t* __restrict__ list,
    const int32_t* __restrict__ n_list, uint32_t t_inv, int H, int kk, int S, int row_stride, float scale_log2e, int split0,
    int nsplit, uint32_t ns_inv, int pitch, _Float16* __restrict__ o_part, float* __restrict__ lse_part, const uint8_t* __restrict__ zero_row,
    ess_xcd xcd, int n_bt, int n_hg, int quads, const int32_t* __restrict__ list_b, const int32_t* __restrict__ n_list_b, int nsplit_a,
    uint32_t ns_inv_a, uint32_t ns_inv_b, ess_attn_final fin, const ess_fetch fetch, uint32_t hg_inv) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int s_item;
  __shared__ __align__(16) int s_last[NW];
  using L = Lay<FMT>;
  constexpr bool kBf = L::kBf;
  constexpr int NBUF = L::NBUF, BUF = L::BUF;
  constexpr int PER_TILE = kBf ? 9 : 8;            // gathers of a wave per tile
  float* const xch = reinterpret_cast<float*>(lds + L::X_OFF);
  int32_t* const slot_cache = reinterpret_cast<int32_t*>(lds + L::SLOT_OFF);
  float* const xamax = reinterpret_cast<float*>(lds + L::SLOT_OFF);
  const uint32_t lds0 = lds_addr_of(lds);
  const int per_row = nsplit * n_hg;

  auto run_item = [&](const int split, const int bt, const int hg) {
  const int b = (int)((uint32_t)bt * t_inv >> 16);
  int tid = threadIdx.x;
  if constexpr (DYN) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int eg = wave & 3, hb = wave >> 2;         // first product: 16 entries, 16 heads
  const int g = lane >> 4, r16 = lane & 15;        // ... quarter of the wave, entry row or head
  const int hh = lane >> 5, h32 = lane & 31;       // second product: half of the wave, head
  const int head0 = hg * HT, heads = min(HT, H - head0);

  // (a launch may carry two lists: ranges 0 .. nsplit_a - 1 are the first's, the rest the second's)
  const bool second = split >= nsplit_a;
  const int32_t* const n_row = second ? n_list_b : n_list;
  const int ns = second ? nsplit - nsplit_a : nsplit_a;
  // the row's whole list and the queries are asked for together
  const int32_t* lrow = (second ? list_b : list) + (size_t)bt * kk;
  int4 mine = make_int4(-1, -1, -1, -1);
  if (quads) {                                     // whole quadruples, 16-byte aligned
    if (4 * tid < kk) mine = *reinterpret_cast<const int4*>(lrow + 4 * tid);
  } else {
    if (4 * tid < kk) mine.x = lrow[4 * tid];
    if (4 * tid + 1 < kk) mine.y = lrow[4 * tid + 1];
    if (4 * tid + 2 < kk) mine.z = lrow[4 * tid + 2];
    if (4 * tid + 3 < kk) mine.w = lrow[4 * tid + 3];
  }
  int n = n_row ? min(n_row[bt], kk) : kk;
  __builtin_amdgcn_sched_barrier(0);
  // Query rows in the layout of a bf16 tile: 1024 bytes and 128 bytes of a row, 16-byte pieces XOR-swizzled by row.  Past the
  // last head its row is repeated.
  {
    const uint8_t* qbase = reinterpret_cast<const uint8_t*>(q + ((size_t)bt * H + head0) * ESS_ROW_DIM);
    const uint32_t qdst = lds0 + (uint32_t)L::Q_OFF;
#pragma unroll
    for (int i = 0; i < HT / NW; ++i) {
      const int row = wave * (HT / NW) + i;
      dma16_base(qbase + (uint32_t)min(row, heads - 1) * (ESS_ROW_DIM * 2), (uint32_t)((lane ^ tr_swz(row)) << 4), qdst + (uint32_t)(row * TRP));
    }
    // (32 heads: a wave's lanes 32 and up bring the next wave's rows once more; the last wave's go past them)
    const int row = wave * (HT / NW) + (lane >> 3);
    dma16_base(qbase, (uint32_t)min(row, heads - 1) * (ESS_ROW_DIM * 2) + 1024u + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4),
               qdst + (uint32_t)(HT * TRP + wave * (HT / NW) * 128));
  }
  __builtin_amdgcn_sched_barrier(0);
  // Entries of the row: as given, or up to the last valid one -- what lies behind it is neither gathered nor multiplied,
  // and the ranges are cut from what is left (lists of uneven length).
  {
    auto masked = [&](int slot, int e) { return (uint32_t)slot < (uint32_t)S && e < n ? slot : (int)0xff800000; };
    mine.x = masked(mine.x, 4 * tid);
    mine.y = masked(mine.y, 4 * tid + 1);
    mine.z = masked(mine.z, 4 * tid + 2);
    mine.w = masked(mine.w, 4 * tid + 3);
    *reinterpret_cast<int4*>(slot_cache + 4 * tid) = mine;
    if (!n_row) {
      const int upto = mine.w >= 0 ? 4 : (mine.z >= 0 ? 3 : (mine.y >= 0 ? 2 : (mine.x >= 0 ? 1 : 0)));
      const unsigned long long m = __ballot(upto > 0);
      const int top = 63 - __builtin_clzll(m | 1ull);
      if (lane == 0) s_last[wave] = m ? 4 * (64 * wave + top) + __builtin_amdgcn_readlane(upto, top) : 0;
    }
  }
  wait_vmcnt<0>();                                 // the queries have landed
  lds_barrier();
  if (!n_row) {
    const int4 a = *reinterpret_cast<const int4*>(s_last), c = *reinterpret_cast<const int4*>(s_last + 4);
    n = __builtin_amdgcn_readfirstlane(max(max(max(a.x, a.y), max(a.z, a.w)), max(max(c.x, c.y), max(c.z, c.w))));
  }
  const int tiles_total = (n + ET - 1) / ET;
  const int tps = ns == 1 ? tiles_total : (int)__umulhi((uint32_t)(tiles_total + ns - 1), second ? ns_inv_b : ns_inv_a);
  const int tile_begin = (second ? split - nsplit_a : split) * tps;
  const int my_tiles = max(min(tile_begin + tps, tiles_total) - tile_begin, 0);
  const size_t part0 = ((size_t)bt * pitch + split0 + split) * H + head0;
  if (my_tiles == 0 && !fin.out) {                 // an empty range: its rows are never read
    if (tid < heads) *reinterpret_cast<float2*>(lse_part + 2 * (part0 + tid)) = make_float2(-__builtin_inff(), 1.f);
    return;
  }

  // Gathers of a tile: a wave brings rows 8 w .. 8 w + 7, one instruction each (bf16: the latent part, its 16-byte pieces
  // XOR-swizzled by row; quantised: the entry as it is), and for bf16 the rope parts by one more.  Lane l holds the
  // address of row l & 7; masked entries are rows of zeros.
  const uint8_t* pbase = pool + (size_t)b * S * row_stride;
  struct Rows { uint32_t lo, hi, rlo, rhi; };
  auto rows_of = [&](int it, Rows& a) {
    const int slot = slot_cache[(tile_begin + it) * ET + 8 * wave + (lane & 7)];
    const uint64_t p = (uint64_t)(uintptr_t)((slot >= 0 ? pbase : zero_row) + (uint32_t)max(slot, 0) * (uint32_t)row_stride);
    a.lo = (uint32_t)p;
    a.hi = (uint32_t)(p >> 32);
    if constexpr (kBf) {
      a.rlo = (uint32_t)__builtin_amdgcn_ds_bpermute((lane >> 3) * 4, (int)a.lo);
      a.rhi = (uint32_t)__builtin_amdgcn_ds_bpermute((lane >> 3) * 4, (int)a.hi);
    }
  };
  uint32_t go = kBf ? (uint32_t)((lane ^ ((wave & 1) << 1)) << 4) : (uint32_t)(lane << 4);      // (row 8 w + r: the swizzle of r, and w's)
  const uint32_t rope_off = 1024u + (uint32_t)(((lane & 7) ^ (((8 * wave + (lane >> 3)) >> 1) & 7)) << 4);
  auto gather_step = [&](const Rows& a, uint32_t dst, auto stepc) {      // 0..7: rows, 8: the rope parts
    constexpr int r = decltype(stepc)::value;
    if constexpr (r < 8) {
      const void* base = reinterpret_cast<const void*>((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)a.lo, r) |
                                                       (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)a.hi, r) << 32);
      if constexpr (kBf) dma16_base<true>(base, go ^ (uint32_t)(((r & 3) << 2 | (r >> 2)) << 4), dst + (uint32_t)((8 * wave + r) * TRP));
      else dma16_entry<true>(base, go, dst + (uint32_t)((8 * wave + r) * F8_PITCH));
    } else if constexpr (kBf) {
      dma16(reinterpret_cast<const uint8_t*>((uint64_t)a.rlo | (uint64_t)a.rhi << 32) + rope_off, dst + (uint32_t)(ET * TRP + wave * 1024));
    }
  };
  auto gather = [&](int it) {
    Rows a;
    rows_of(it, a);
    unroll<PER_TILE>([&](auto c) { gather_step(a, lds0 + (uint32_t)((it % NBUF) * BUF), c); });
  };
  if (my_tiles > 0) gather(0);
  if constexpr (NBUF == 3) if (my_tiles > 1) gather(1);

  // Q^T as the B operand of the first product (16x16x32), stationary: lane (g, head r16 of block j), eight dimensions per
  // k-step.  bf16: dims 32 ks + 8 g ..; quantised: a lane takes 16 consecutive dimensions for two k-steps.
  bf16x8 qb[18];
  {
    const uint8_t* qr = lds + L::Q_OFF + (16 * hb + r16) * TRP;
    const uint8_t* qp = lds + L::Q_OFF + HT * TRP + (16 * hb + r16) * 128;
    const int sw = tr_swz(r16);
    unroll<16>([&](auto kc) {
      constexpr int ks = decltype(kc)::value;
      const int c = kBf ? 4 * (ks & 3) + g : 8 * ((ks >> 1) & 1) + 2 * g + (ks & 1);
      qb[ks] = *reinterpret_cast<const bf16x8*>(qr + 256 * (ks >> 2) + ((c ^ sw) << 4));
    });
    unroll<2>([&](auto kc) { qb[16 + kc] = *reinterpret_cast<const bf16x8*>(qp + (((4 * kc + g) ^ ((r16 >> 1) & 7)) << 4)); });
  }
  floatx16 acc[2];                                 // O^T: columns 64 w + 32 cb + 8 q + 4 hh + i of head h32 at index 4 q + i
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[cb][i] = 0.f;
  // softmax state: the reference of the lane's head in the first product (16 hb + r16) and in the second (h32), and the
  // lane's share of the row sum of the former
  float ref = -__builtin_inff(), refp = ref, l = 0.f;

  const int krow = 16 * eg + r16;
  uint32_t kb = kBf ? (uint32_t)(krow * TRP + ((g ^ tr_swz(r16)) << 4)) : (uint32_t)(krow * F8_PITCH + 16 * g);
  uint32_t rb = kBf ? (uint32_t)(ET * TRP + krow * 128 + ((g ^ ((r16 >> 1) & 7)) << 4)) : (uint32_t)(krow * F8_PITCH + 520 + 16 * g);
  const int gi = g & 1, ti = r16 >> 2, tj = lane & 3;
  const int vrow0 = 4 * hh + ti;
  uint32_t vb = kBf ? (uint32_t)(vrow0 * TRP + (((8 * (wave & 1) + 2 * gi + (tj >> 1)) ^ tr_swz(vrow0)) << 4) + (tj & 1) * 8 + 256 * (wave >> 1))
                    : (uint32_t)((hh + 2 * (r16 >> 1)) * F8_PITCH + 64 * wave + 16 * gi + 8 * (r16 & 1));
  // P: 16-byte pieces XOR-swizzled by head.  Written 8 (bf16) or 4 bytes at a time, read whole.
  const uint32_t pw0 = (uint32_t)((16 * hb + r16) * 128 + (kBf ? 8 * (g >> 1) : 4 * g)), psw = (uint32_t)((r16 >> 1) & 7);
  const uint32_t pr0 = (uint32_t)(h32 * 128 + (kBf ? 0 : (wave >> 1) * L::P_BYTES));

  auto iteration = [&](int it, auto morec) {
    constexpr bool MORE = decltype(morec)::value;  // there is a tile it + NBUF - 1 to gather
    const uint32_t tb = (uint32_t)((it % NBUF) * BUF), dst = lds0 + (uint32_t)(((it + NBUF - 1) % NBUF) * BUF);
    const uint32_t pb = kBf ? tb + ET * TRP : (uint32_t)L::P_OFF;
    Rows a;
    if constexpr (MORE) rows_of(it + NBUF - 1, a);
    if (NBUF == 3 && it + 1 < my_tiles) wait_vmcnt<PER_TILE>(); else wait_vmcnt<0>();
    lds_barrier();                                 // the tile is there; everyone is done with the one before it

    // first product: 16 entries x 16 heads; fragments are read CK steps ahead, the gathers ride on the steps
    floatx4 s;
    floatx4 sc[4];                                 // quantised: by group of 128 dimensions, the scales of the lane's four entries
    const floatx4 init = lds_float4(reinterpret_cast<const float*>(slot_cache) + (tile_begin + it) * ET + 16 * eg + 4 * g);      // a slot number is a denormal, a masked entry -inf
    if constexpr (kBf) {
      constexpr int CK = 10;
      bf16x8 fa[CK];
      floatx4 s2 = {0, 0, 0, 0};                   // two chains
      s = init;
      auto read_k = [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if constexpr (t < 16) fa[t % CK] = *reinterpret_cast<const bf16x8*>(lds + tb + (kb ^ (uint32_t)((t >> 2) << 6)) + 256 * (t & 3));
        else fa[t % CK] = *reinterpret_cast<const bf16x8*>(lds + tb + (rb ^ (uint32_t)((t & 1) << 6)));
      };
      unroll<CK>(read_k);
      unroll<18>([&](auto tc) {
        constexpr int t = decltype(tc)::value, ks = t < 16 ? 4 * (t & 3) + (t >> 2) : t;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t & 1) s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[t % CK], qb[ks], s2, 0, 0, 0);
        else s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[t % CK], qb[ks], s, 0, 0, 0);
        if constexpr (t + CK < 18) read_k(std::integral_constant<int, t + CK>{});
        if constexpr (MORE && (t & 1)) gather_step(a, dst, std::integral_constant<int, t / 2>{});
      });
      __builtin_amdgcn_sched_barrier(0);
      s += s2;
    } else {
      constexpr int CK = 5;
      uint4 raw[CK];
      floatx4 d;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint2 w = *reinterpret_cast<const uint2*>(lds + tb + (16 * eg + 4 * g + i) * F8_PITCH + 512);
        sc[0][i] = __uint_as_float(w.x << 16); sc[1][i] = __uint_as_float(w.x & 0xffff0000u);
        sc[2][i] = __uint_as_float(w.y << 16); sc[3][i] = __uint_as_float(w.y & 0xffff0000u);
      }
      s = init;
      auto read_k = [&](auto tc) {                 // 0, 1: 32 rope values; 2..9: 64 dimensions each, a lane 16 of them
        constexpr int t = decltype(tc)::value;
        if constexpr (t >= 2) raw[t % CK] = *reinterpret_cast<const uint4*>(lds + tb + kb + 64 * (t - 2));
        else {
          const uint2* p = reinterpret_cast<const uint2*>(lds + tb + rb + 64 * t);
          const uint2 lo = p[0], hi = p[1];
          raw[t % CK] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
      };
      unroll<CK>(read_k);
      unroll<10>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t < 2) {
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, raw[t % CK]), qb[16 + t], s, 0, 0, 0);
        } else {
          constexpr int p = t - 2;
          const bf16x8 lo = widen(raw[t % CK].x, raw[t % CK].y), hi = widen(raw[t % CK].z, raw[t % CK].w);
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, qb[2 * p], (p & 1) ? d : floatx4{0, 0, 0, 0}, 0, 0, 0);
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, qb[2 * p + 1], d, 0, 0, 0);
          if constexpr (MORE) gather_step(a, dst, std::integral_constant<int, p>{});
          if constexpr (p & 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = fmaf(sc[p >> 1][i], d[i], s[i]);
          }
        }
        if constexpr (t + CK < 10) read_k(std::integral_constant<int, t + CK>{});
      });
      __builtin_amdgcn_sched_barrier(0);
    }
    // V^T fragments of the second product, on their way while the softmax waits
    bf16x8 fv[8];
    int2v rv[8];
    auto read_v = [&](auto xc) {                   // step x: entries 16 (x >> 1) .., columns 32 (x & 1) ..
      constexpr int x = decltype(xc)::value, st = x >> 1, cb = x & 1;
      if constexpr (kBf) {
        const uint32_t at = lds0 + tb + (uint32_t)(16 * st * TRP), v = vb ^ (uint32_t)(cb << 6);
        fv[x] = tr_frag(at + v, at + (v ^ 32u) + 8 * TRP);       // (row + 8: granule bit 1 of the swizzle differs)
      } else {
        rv[x] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<lds_int2v*>(lds0 + tb + vb + (uint32_t)(16 * st * F8_PITCH + 32 * cb)));
      }
    };
    const float tmax = quad_max(max4(s));
    if (g == 0) xch[(16 * hb + r16) * 4 + eg] = tmax;
    unroll<8>(read_v);
    lds_barrier();
    // the reference only moves when a tile exceeds it by more than 2^8 (always from -inf); all waves see the same maxima
    const float mq = max4(lds_float4(xch + 4 * (16 * hb + r16))) * scale_log2e;
    const float mp = max4(lds_float4(xch + 4 * h32)) * scale_log2e;
    const bool up = mp > refp + kLazyMax;
    if (__any(up)) {
      auto moved = [&](float& r, float m) {
        const float now = m > r + kLazyMax ? m : r;
        const float alpha = r == -__builtin_inff() ? 1.f : __builtin_amdgcn_exp2f(r - now);      // (from -inf: nothing added up yet)
        r = now;
        return alpha;
      };
      const bool rescale = __any(up && refp != -__builtin_inff());
      l *= moved(ref, mq);
      const float alpha = moved(refp, mp);
      if (rescale) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[cb][i] *= alpha;
      }
    }
    // P in LDS, per head, in the order in which the second product takes its entries: bf16: 16 s + 4 hh + i, then
    // 16 s + 8 + 4 hh + i (transposing reads of four rows); quantised: even entries, then odd ones (reads of eight rows,
    // two rows apart: the pitch of 656 bytes spreads them over all banks)
    {
      const float use = ref == -__builtin_inff() ? 0.f : ref;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], scale_log2e, -use));
        l += s[i];
      }
      uint8_t* const p = lds + pb + pw0;
      if constexpr (kBf) {
        *reinterpret_cast<uint2*>(p + (((uint32_t)(2 * eg + (g & 1)) ^ psw) << 4)) = make_uint2(pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3]));
      } else {
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          *reinterpret_cast<uint32_t*>(p + grp * L::P_BYTES + (((uint32_t)(2 * eg) ^ psw) << 4)) = pack_bf16(s[0] * sc[grp][0], s[2] * sc[grp][2]);
          *reinterpret_cast<uint32_t*>(p + grp * L::P_BYTES + (((uint32_t)(2 * eg + 1) ^ psw) << 4)) = pack_bf16(s[1] * sc[grp][1], s[3] * sc[grp][3]);
        }
      }
    }
    lds_barrier();
    // second product: 64 columns of this wave x 32 heads x 64 entries
    bf16x8 pf[2];
    auto read_p = [&](auto stc) {
      constexpr int st = decltype(stc)::value;
      pf[st & 1] = *reinterpret_cast<const bf16x8*>(lds + pb + pr0 + (((uint32_t)(2 * st + hh) ^ (uint32_t)((h32 >> 1) & 7)) << 4));
    };
    read_p(std::integral_constant<int, 0>{});
    unroll<8>([&](auto xc) {
      constexpr int x = decltype(xc)::value, st = x >> 1, cb = x & 1;
      if constexpr (cb == 0 && st < 3) read_p(std::integral_constant<int, st + 1>{});
      bf16x8 v;
      if constexpr (kBf) v = fv[x]; else v = widen((uint32_t)rv[x][0], (uint32_t)rv[x][1]);
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pf[st & 1], acc[cb], 0, 0, 0);
    });
  };
  int it = 0;
  for (; it + NBUF - 1 < my_tiles; ++it) iteration(it, std::true_type{});
  for (; it < my_tiles; ++it) iteration(it, std::false_type{});

  // row sums of the four groups of entries and, for a partial result, largest magnitudes of the eight waves meet in LDS
  l = quad_sum(l);
  if (g == 0) xch[(16 * hb + r16) * 4 + eg] = l;
  if (!fin.out) {
    float amax = 0.f;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(acc[cb][i]));        // (of the numbers: a NaN is skipped)
    amax = pair_max(amax);
    if (hh == 0) xamax[h32 * 8 + wave] = amax;
  }
  const int cr = lane >> 3, cc = lane & 7;         // stores: head 8 r4 + cr, piece cc of its 64 columns
  // earlier partial results of the row: the first PRE are asked for before the barrier
  constexpr int PRE = 4;
  const _Float16* const prev0 = o_part + ((size_t)bt * pitch * H + head0) * ESS_LATENT_DIM + 64 * wave + 8 * cc;
  const uint32_t prev_step = (uint32_t)H * ESS_LATENT_DIM;
  uint32_t prow[4];
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) prow[r4] = (uint32_t)min(8 * r4 + cr, heads - 1) * ESS_LATENT_DIM;
  const float* const plse = lse_part + 2 * ((size_t)bt * pitch * H + head0 + min(h32, heads - 1));
  float2 pv[MAX_PREV];
  halfx8 part[PRE][4];
  if (fin.out) {
#pragma unroll
    for (int s = 0; s < MAX_PREV; ++s) pv[s] = *reinterpret_cast<const float2*>(plse + 2 * (uint32_t)(max(min(s, fin.n_prev - 1), 0) * H));      // (past the last: again, unused)
#pragma unroll
    for (int s = 0; s < PRE; ++s)
      if (s < fin.n_prev)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) part[s][r4] = *reinterpret_cast<const halfx8*>(prev0 + s * prev_step + prow[r4]);
  }
  lds_barrier();                                   // also: everyone is done with the last tile
  auto wave_sync = [] {                            // lanes read what other lanes of their wave wrote: nothing may be moved across
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const floatx4 ls = lds_float4(xch + 4 * h32);
  const float l_tot = (ls[0] + ls[1]) + (ls[2] + ls[3]);
  const bool have = l_tot > 0.f;
  const float lse = have ? (refp + __builtin_amdgcn_logf(l_tot)) * kLn2 : -__builtin_inff();
  float inv = have ? 1.0f / l_tot : 0.f;
  if (!fin.out) {
    // A partial result, as fp16 (see attn_common.h).  Should a head's largest magnitude reach 2^15 (entry values of that
    // size: rare), it is divided by the power of two that brings it below -- exact, undone by the merge.
    const float top = fmaxf(max4(lds_float4(xamax + 8 * h32)), max4(lds_float4(xamax + 8 * h32 + 4))) * inv;
    float down = 1.f;
    const bool big = __any(top >= 32768.f);
    if (big) {
      int ex = 0;
      (void)frexpf(top, &ex);                      // top < 2^ex
      down = (top >= 32768.f && top <= 3.0e38f) ? ldexpf(1.f, ex - 15) : 1.f;
      inv = inv / down;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {             // never inf in the fp16 image; what is no number stays so (fmed3 would make it -65504)
          const float v = acc[cb][i] * inv, in_range = __builtin_amdgcn_fmed3f(v, -65504.f, 65504.f);
          acc[cb][i] = v != v ? v : in_range;
        }
      inv = 1.f;
    }
    uint8_t* const stage = lds + wave * (HT * OH_PITCH);
    uint8_t* const orow = stage + h32 * OH_PITCH + 8 * hh;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<halfx4*>(orow + (32 * cb + 8 * qd) * 2) = __builtin_convertvector(
            (floatx4{acc[cb][4 * qd] * inv, acc[cb][4 * qd + 1] * inv, acc[cb][4 * qd + 2] * inv, acc[cb][4 * qd + 3] * inv}), halfx4);
    wave_sync();
    _Float16* const orow0 = o_part + part0 * ESS_LATENT_DIM + 64 * wave + 8 * cc;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int r = 8 * r4 + cr;
      const uint4 v = *reinterpret_cast<const uint4*>(stage + r * OH_PITCH + cc * 16);
      if (r < heads) ess_store_nt(reinterpret_cast<uint4*>(orow0 + r * ESS_LATENT_DIM), v);
    }
    if (wave == 0 && hh == 0 && h32 < heads)
      *reinterpret_cast<float2*>(lse_part + 2 * (part0 + h32)) = make_float2(lse, down);
    return;
  }
  // The row is finished here: this range's result in fp32 and the fin.n_prev partial results of the row that earlier
  // launches wrote, weighted as in k_attn_merge.
  float* const wt = reinterpret_cast<float*>(lds + NW * HT * OF_PITCH) + wave * WT_WORDS;      // [MAX_PREV][HT]
  float mx = lse;
#pragma unroll
  for (int s = 0; s < MAX_PREV; ++s) {
    pv[s].x = s < fin.n_prev ? pv[s].x : -__builtin_inff();
    mx = fmaxf(mx, pv[s].x);
  }
  const float mu = mx == -__builtin_inff() ? 0.f : mx;
  float w0 = have ? __expf(lse - mu) : 0.f, den = w0;
  float w[MAX_PREV];
#pragma unroll
  for (int s = 0; s < MAX_PREV; ++s) {
    w[s] = __expf(pv[s].x - mu);
    den += w[s];
  }
  const float dinv = den > 0.f ? 1.0f / den : 0.f;
  w0 *= inv * dinv;
  bool gap = false;                                // a result that is not there: its place may hold anything
#pragma unroll
  for (int s = 0; s < MAX_PREV; ++s) {
    const bool none = pv[s].x == -__builtin_inff();
    gap |= none && s < fin.n_prev;
    if (hh == 0) wt[s * HT + h32] = none ? -1.f : w[s] * pv[s].y * dinv;
  }
  gap = __any(gap);
  if (__any(!have))
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[cb][i] = have ? acc[cb][i] : 0.f;
  uint8_t* const stage = lds + wave * (HT * OF_PITCH);
  {
    uint8_t* const orow = stage + h32 * OF_PITCH + 16 * hh;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<floatx4*>(orow + (32 * cb + 8 * qd) * 4) =
            floatx4{acc[cb][4 * qd] * w0, acc[cb][4 * qd + 1] * w0, acc[cb][4 * qd + 2] * w0, acc[cb][4 * qd + 3] * w0};
  }
  wave_sync();
  float o[4][8];
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    const floatx4* src = reinterpret_cast<const floatx4*>(stage + (8 * r4 + cr) * OF_PITCH + cc * 32);
    const floatx4 lo = src[0], hi = src[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) { o[r4][i] = lo[i]; o[r4][4 + i] = hi[i]; }
  }
  auto add = [&](int s, halfx8 (&x)[4]) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      float ws = wt[s * HT + 8 * r4 + cr];
      if (gap) {
        const bool none = ws == -1.f;
        x[r4] = none ? halfx8{0, 0, 0, 0, 0, 0, 0, 0} : x[r4];
        ws = none ? 0.f : ws;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) o[r4][i] = fmaf(ws, (float)x[r4][i], o[r4][i]);
    }
  };
#pragma unroll
  for (int s = 0; s < PRE; ++s)
    if (s < fin.n_prev) add(s, part[s]);
  for (int s = PRE; s < fin.n_prev; ++s) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) part[0][r4] = *reinterpret_cast<const halfx8*>(prev0 + s * prev_step + prow[r4]);
    add(s, part[0]);
  }
  uint16_t* const orow0 = fin.out + ((size_t)bt * H + head0) * ESS_LATENT_DIM + 64 * wave + 8 * cc;
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4)
    if (8 * r4 + cr < heads)
      ess_store_nt(reinterpret_cast<uint4*>(orow0 + (8 * r4 + cr) * ESS_LATENT_DIM),
                   make_uint4(pack_bf16(o[r4][0], o[r4][1]), pack_bf16(o[r4][2], o[r4][3]), pack_bf16(o[r4][4], o[r4][5]), pack_bf16(o[r4][6], o[r4][7])));
  if (fin.lse && wave == 0 && hh == 0 && h32 < heads)
    fin.lse[(size_t)bt * H + head0 + h32] = den > 0.f ? mx + __logf(den) : -__builtin_inff();
  };
  if constexpr (DYN) {
    // handed out XCD by XCD (see k_attn_partial_tr): the head groups of a row read its entries into one L2
    if (!ess_ticket_join(xcd, &s_item)) return;
    const uint32_t avail = ~xcd.avoid & 0xffu;
    const int x = ess_xcc_id() & 7;
    const int nw = max(__popc(avail), 1);
    int cls = ((avail >> x) & 1u) ? __popc(avail & ((1u << x) - 1u)) : 0, tried = 1;
    for (;;) {
      int item;
      for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
          const uint32_t tk = atomicAdd(xcd.ticket + ESS_TK_CLASS + ESS_TK_STRIDE * cls, 1u);
          const uint32_t row = (tk / (uint32_t)per_row) * (uint32_t)nw + (uint32_t)cls;
          s_item = row < (uint32_t)n_bt ? (int)(row * (uint32_t)per_row + tk % (uint32_t)per_row) : -1;
        }
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= 0 || tried == nw) break;
        ++tried;
        cls = cls + 1 == nw ? 0 : cls + 1;
      }
      if (item < 0) break;
      run_item((item % per_row) / n_hg, item / per_row, item % n_hg);
    }
  } else {
    // consecutive workgroups go round the eight XCDs: the head groups of one range are eight workgroups apart, on one XCD,
    // whose L2 then holds the entries they share
    if (blockIdx.x == 0 && blockIdx.y == 0) {
      for (int i = threadIdx.x; i < fin.n_zero; i += NT) fin.zero_cnt[i] = 0;
      if (fin.chk.tickets && threadIdx.x == 0) ess_check_tickets(fin.chk);
    }
    uint32_t u = 8 * blockIdx.y + (blockIdx.x & 7), hg = blockIdx.x >> 3;
    if (fetch.wgs) {                               // (see ess_fetch)
      const uint32_t x = blockIdx.x & 7, j = blockIdx.x >> 3, jg = j * hg_inv >> 16;
      if (x < 2) {
        if (2 * j + x < (uint32_t)fetch.wgs) ess_fill::entries<2>(fetch, reinterpret_cast<int32_t*>(lds), (int)((2 * j + x) * NW + (threadIdx.x >> 6)), fetch.wgs * NW);
        return;
      }
      u = 6 * jg + x - 2;
      hg = j - jg * n_hg;
    }
    const uint32_t bt = nsplit == 1 ? u : __umulhi(u, ns_inv);
    if (bt < (uint32_t)n_bt) run_item((int)(u - bt * nsplit), (int)bt, (int)hg);
  }
}

}  // namespace

int ess_init_attn_h32() {
#define ESS_H32_ATTR(FMT, DYN)                                                                         \
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_h32<FMT, DYN>),                   \
                              hipFuncAttributeMaxDynamicSharedMemorySize, Lay<FMT>::BYTES))
  ESS_H32_ATTR(ESS_FMT_BF16, false);
  ESS_H32_ATTR(ESS_FMT_BF16, true);
  ESS_H32_ATTR(ESS_FMT_FP8, false);
  ESS_H32_ATTR(ESS_FMT_FP8, true);
#undef ESS_H32_ATTR
  return ESS_OK;
}

int ess_launch_attn_h32(ess_ctx* ctx, const void* q, const uint8_t* slot_pool, const int32_t* list, const int32_t* n_list, int B, int T,
                        int split0, int nsplit, int pitch, hipStream_t st, int b0, ess_xcd xcd, hipEvent_t done, const ess_attn_final* final,
                        const int32_t* list_b, const int32_t* n_list_b, int nsplit_b, const ess_fetch* fetch) {
  const ess_config& c = ctx->cfg;
  if (split0 + nsplit + nsplit_b > pitch || (size_t)(b0 + B) * T * pitch > ctx->part_cap) return ess_fail(ESS_ERR_INVALID_ARG, "internal: partial results");
  if (c.topk > MAX_LIST) return ess_fail(ESS_ERR_INVALID_ARG, "internal: attention form");
  ess_attn_final fin{};
  if (final) fin = *final;
  if (fin.out && (nsplit + nsplit_b != 1 || fin.n_prev > MAX_PREV || fin.n_prev > split0)) return ess_fail(ESS_ERR_INVALID_ARG, "internal: final attention launch");
  const int ns = nsplit + nsplit_b, n_hg = (c.attn_heads + HT - 1) / HT;
  dim3 grid(8 * n_hg, (B * T * ns + 7) / 8);
  if (xcd.ticket) grid = dim3(ess_xcd_grid(ns * B * T * n_hg, xcd));
  ess_fetch fe{};
  if (fetch) {
    if (xcd.ticket || fin.out) return ess_fail(ESS_ERR_INVALID_ARG, "internal: attention launch with a fetch");
    fe = *fetch;
    const int groups = (ns * B * T + 5) / 6 * n_hg;
    grid = dim3(8 * (groups > (fe.wgs + 1) / 2 ? groups : (fe.wgs + 1) / 2));
  }
  const float sc = c.sm_scale * kLog2e;
  const uint16_t* qq = static_cast<const uint16_t*>(q);
  _Float16* op = reinterpret_cast<_Float16*>(ctx->o_part) + (size_t)b0 * T * pitch * c.attn_heads * ESS_LATENT_DIM;
  float* lp = ctx->lse_part + (size_t)b0 * T * pitch * c.attn_heads * 2;
  if (fin.out) {
    fin.out += (size_t)b0 * T * c.attn_heads * ESS_LATENT_DIM;
    if (fin.lse) fin.lse += (size_t)b0 * T * c.attn_heads;
  }
  const int quads = (c.topk & 3) == 0 && ((reinterpret_cast<uintptr_t>(list) | reinterpret_cast<uintptr_t>(list_b)) & 15) == 0;
  const uint32_t hg_inv = 65535u / n_hg + 1;
  const uint32_t t_inv = 65535u / T + 1, ns_inv = 0xffffffffu / ns + 1, ns_inv_a = 0xffffffffu / nsplit + 1,
                 ns_inv_b = 0xffffffffu / (nsplit_b > 0 ? nsplit_b : 1) + 1;      // divisions by T of numbers up to 16384, by nsplit > 1 up to 2^20: exact
#define ESS_H32_LAUNCH(FMT, DYN)                                                                                                       \
  ESS_HIP(ess_launch_done(done, &k_attn_h32<FMT, DYN>, grid, dim3(NT), (size_t)Lay<FMT>::BYTES, st, qq, slot_pool, list, n_list, t_inv, \
                          c.attn_heads, c.topk, c.slots_per_seq, c.row_stride, sc, split0, ns, ns_inv, pitch, op, lp, ctx->zero_row, xcd, \
                          B * T, n_hg, quads, list_b, n_list_b, nsplit, ns_inv_a, ns_inv_b, fin, fe, hg_inv))
  if (c.latent_fmt == ESS_FMT_BF16) { if (xcd.ticket) ESS_H32_LAUNCH(ESS_FMT_BF16, true); else ESS_H32_LAUNCH(ESS_FMT_BF16, false); }
  else { if (xcd.ticket) ESS_H32_LAUNCH(ESS_FMT_FP8, true); else ESS_H32_LAUNCH(ESS_FMT_FP8, false); }
#undef ESS_H32_LAUNCH
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}
