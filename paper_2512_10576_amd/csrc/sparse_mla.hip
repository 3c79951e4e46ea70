// Stage 4: SparseMLA decode over the selected Latent-Cache entries (ESS paper
// Sec. 3.3), absorbed form: the 576 values of an entry are the key, the first
// 512 the value.  Flash-decoding layout: every (b,t) is cut into `nsplit`
// ranges of its entry list; each workgroup produces a softmax-normalised
// partial output and its log-sum-exp for all heads, and a merge kernel
// combines the partial results -- the same merge that joins Attn0 (resident
// entries) and Attn1 (fetched entries) of the DA overlap.
//
// Matrix-core mapping (v_mfma_f32_32x32x16_bf16, wave64).  A workgroup is four
// waves, one per SIMD, each owning 32 heads with the whole 512-wide output row
// in 256 accumulator registers and its queries stationary (144 VGPRs): 128 heads
// per workgroup, so the entries of a range are brought from memory once for all
// heads.  The kernel is built for one wave per SIMD and the register budget that
// comes with it.  Both products are computed transposed so that nothing is
// re-laid out between them; see the comment at the kernel.
#include "attn_common.h"
#include "fetch.h"
#include <utility>

namespace {

constexpr int TILE = ESS_ATTN_TILE;            // 32 entries
constexpr int NTH = 256;                       // four waves
constexpr int MAX_TPS = 64;                    // tiles per split (the launcher picks nsplit accordingly): a list of 2048 entries fits one split
// ---------------------------------------------------------------------------------------------
// bf16 entries are brought into LDS by the memory system itself
// (global_load_lds_dwordx4: a wave instruction moves 64 x 16 bytes from per-lane global addresses to
// consecutive LDS addresses, no registers involved).  One wave instruction per 1024-byte latent
// part of a row, one per eight 128-byte rope parts.  The loads are issued through inline assembly
// because the compiler, seeing an LDS-writing load, would wait for every outstanding one before the
// next LDS read; completion is tracked by hand with s_waitcnt vmcnt (memory loads complete in issue
// order, 9 of them per wave and tile).
constexpr int RP_BYTES = TILE * 128;           // 4096: rope parts, 16-byte pieces XOR-swizzled by row
constexpr int DMA_PER_TILE = 9;                // wave instructions per tile: 8 latent rows + 1 rope group

// ---------------------------------------------------------------- the partial-attention kernel
// Four waves, one per SIMD, 32 heads each: a workgroup covers all (up to 128) heads of one range of the entry
// list, so an entry is brought from memory once per range.  Tiles of 32 entries sit in LDS as bf16 rows: bf16
// entries gathered there by global_load_lds, quantised entries (512 fp8 + 4 scales + rope) brought whole into a raw ring
// in the same way, a tile ahead, and dequantised from it into the same layout.  Matrix-core mapping (v_mfma_f32_32x32x16_bf16), both
// products transposed so that nothing is re-laid out between them:
//   S^T[r,h] = sum_d K[r,d] Q[h,d]      A = entry rows from LDS (lane: row l%32, 8 dims), B = Q^T (registers)
//   O^T[v,h] = sum_r V^T[v,r] P^T[r,h]  A = V^T, read transposed from the same rows, B = P^T (registers)
// The accumulator of S^T gives lane (hh = l/32, h = l%32) the sixteen logits of head h for tile rows
// 8q + 4hh + i (q, i = 0..3), and registers 8s..8s+7 are, in that order, the eight k-values the lane supplies for
// the B operand of k-step s of the second product: P^T never leaves registers.  Softmax state is per lane = per
// (head, half); the two halves of a head meet in one v_permlane32_swap.
// What bounds it.  Per tile a SIMD's matrix pipe is busy for 2176 cycles (68 MFMAs of 32), and one wave issues its
// instructions one at a time, four cycles each or more, so what a tile costs is decided by what the wave waits for and
// by how many instructions it needs.  The LDS is close behind: to one wave per SIMD it delivers 127 bytes per clock of K
// fragments and 78 of transposed ones (215 and 168 to four waves per SIMD), so the 144 + 128 KiB of a tile alone are
// about 2800 cycles of reads beside the 2176 of MFMAs.  Measured with phase timers, cycles per tile: before, 5500-5900 (bf16; 760 instructions) and 6900
// (quantised); now 2250 + 1400 (first + second product, bf16; 530 instructions) and 2350 + 2240 (quantised).  What did it:
//  * the accumulation of S^T in two chains (a dependent MFMA of this shape waits for twice its 32 cycles);
//  * fragments read six and eight steps ahead, in a program order pinned by scheduling barriers, with the softmax, the
//    gathers and the conversion of quantised entries cut into pieces between the MFMAs;
//  * no wait for memory inside the loop other than the one for the tile: queries still in flight at the loop's start made
//    the compiler wait there for the newest gathers (1300 cycles per tile);
//  * fewer instructions: pairs rounded by v_cvt_pk_bf16_f32, fragment addresses with the tile's swizzle variants
//    outermost so that offsets are immediate, row addresses in scalar registers, masks through the accumulator's start.
// Under this load the clock falls to 1.6-2.0 GHz (2.2 in a short launch), so the time follows the cycles only in part:
// batch 128 x 2 tokens, 2048 entries, 128 heads: 233 -> 200 us (bf16), 241 -> 207 us (quantised), merge included.
// A workgroup's start and end weigh as much as ten tiles (71 k cycles for eight tiles before, 59 k now): the queries
// come through LDS by the gather path, half at a time, beside the gathers of the first two tiles (were: 36 loads per
// lane and two barriers in front of the first gather), and the result leaves in 256-byte pieces while it is converted.
//  * V^T is never built.  ds_read_b64_tr_b16 delivers, in each group of 16 lanes, column n of four consecutive
//    rows to lane n (source lane 4i+j points at columns 4j..4j+3 of row i); two such reads (rows 16s+4hh+i and
//    16s+8+4hh+i) make one A fragment whose k order is the order in which S^T leaves the first product.
//  * Rows have no padding (pitch 1024 bytes); the 16-byte granules of a row are XOR-swizzled with
//    f(row) = (row&3)<<2 | (row>>2)&3, applied on the way in by letting lane l of the gather fetch granule
//    l ^ f(row).  The LDS has 64 banks: K fragments (16 rows of one granule per clock) are
//    conflict-free because f is a bijection of the row's low four bits, transposing reads (4 rows x 64 bytes per
//    clock) because f puts the row's low two bits above the granule pair.
//  * The running maximum is only moved when a tile exceeds it by more than 2^8, so the 256 accumulator registers
//    are rescaled a few times per split instead of once per tile.
//  * bf16: four tile buffers, two tiles in use (the pipeline overlaps two) and two in flight.  Quantised: three buffers
//    and a ring of two raw tiles, brought whole by the gather path and converted by the wave that brought them.
// Masked entries (slot < 0) are gathered from a row of zeros, so that no product meets stale LDS.
constexpr int HPW_ = 32;
constexpr int TR_KL_BYTES = TILE * TRP;          // 32768
constexpr int TR_RAW_BYTES = TR_KL_BYTES + RP_BYTES;
constexpr int tr_nbuf(int fmt) { return fmt == ESS_FMT_BF16 ? 4 : 3; }
constexpr int F8_RAW_BYTES = TILE * F8_PITCH;    // 20992
constexpr int tr_nraw(int fmt) { return fmt == ESS_FMT_BF16 ? 0 : 2; }
constexpr int O_PITCH = 264;                     // result rows are staged in LDS 128 columns at a time: 256 bytes of fp16 and 8 of padding
constexpr int Q_HALF_BYTES = HPW_ * 576;         // 18432: half the dimensions of a wave's 32 query rows, on their way to registers
constexpr int tr_slot_off(int fmt) { return tr_nbuf(fmt) * TR_RAW_BYTES + tr_nraw(fmt) * F8_RAW_BYTES; }
constexpr int tr_lds_bytes(int fmt) { return tr_slot_off(fmt) + MAX_TPS * TILE * 4; }     // 155648 | 160768: tile buffers, raw entries, slot list
constexpr int HPW = HPW_;                        // heads per wave
constexpr int HPG = 4 * HPW;                     // heads per workgroup
constexpr int KS16 = ESS_ROW_DIM / 16;           // 36 k-steps of the first product
constexpr int VB32 = ESS_LATENT_DIM / 32;        // 16 blocks of 32 value columns

template <int FMT, bool DYN>
__global__ __launch_bounds__(NTH, 1) void k_attn_partial_tr(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ pool, const int32_t* __restrict__ list,
    const int32_t* __restrict__ n_list, int T, int H, int kk, int S, int row_stride, float scale_log2e, int split0,
    int nsplit, int pitch, _Float16* __restrict__ o_part, float* __restrict__ lse_part, const uint8_t* __restrict__ zero_row,
    ess_xcd xcd, int n_bt, int n_hg, const int32_t* __restrict__ list_b, const int32_t* __restrict__ n_list_b, int nsplit_b, const ess_fetch fetch,
    uint32_t bt_inv) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int s_item;
  constexpr bool kDma = FMT == ESS_FMT_BF16;       // rows go to their tile as they are; else to the raw ring, and from there dequantised
  constexpr int NBUF = tr_nbuf(FMT), NRAW = tr_nraw(FMT), RAW_OFF = NBUF * TR_RAW_BYTES;
  constexpr int PER_TILE = kDma ? DMA_PER_TILE : 8;    // memory instructions of a wave per tile
  int32_t* slot_cache = reinterpret_cast<int32_t*>(lds + tr_slot_off(FMT));   // [MAX_TPS][32], masked entries -inf
  const uint32_t lds0 = lds_addr_of(lds);
  // Work item = (bt, split, head group).  The work items of one (b,t) share its queries (144 KiB for 128 heads),
  // so they should meet in one L2.  By workgroup index: bt is the fastest grid dimension, and consecutive
  // workgroups go round the eight XCDs, so the splits of a row land on one XCD whenever the number of rows is a
  // multiple of eight.  Drawn from counters (off the XCDs to be avoided): every XCD that takes work has a counter
  // of its own (class c of nw) that hands out the items of rows c, c + nw, c + 2 nw .. one after the other; a
  // workgroup whose class has run out goes on with the next class, so any one workgroup could finish the launch.
  const int per_row = (nsplit + nsplit_b) * n_hg;
  int cls = 0, nw = 1, tried = 1;
  if constexpr (DYN) {
    if (!ess_ticket_join(xcd, &s_item)) return;
    const uint32_t work = ~xcd.avoid & 0xffu;
    const int x = ess_xcc_id() & 7;
    nw = max(__popc(work), 1);
    cls = ((work >> x) & 1u) ? __popc(work & ((1u << x) - 1u)) : 0;
  }
  auto run_item = [&](const int split, const int bt, const int hg) {
  const int b = bt / T;
  // the thread index passes through an empty asm statement so that what is derived from it (lane constants, LDS
  // offsets) is computed per work item, where it is needed, instead of being kept in registers across the loop
  int tid = threadIdx.x;
  if constexpr (DYN) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, h32 = lane & 31;       // half of the wave, head within the wave
  const int head0 = hg * HPG + wave * HPW;
  const bool wave_active = head0 < H;

  // (a launch may carry two lists: ranges 0 .. nsplit - 1 are the first's, the rest the second's)
  const bool second = split >= nsplit;
  const int32_t* const my_list = second ? list_b : list;
  const int32_t* const my_n = second ? n_list_b : n_list;
  const int ns = second ? nsplit_b : nsplit;
  const int n = my_n ? min(my_n[bt], kk) : kk;
  const int tiles_total = (n + TILE - 1) / TILE;
  const int tps = min((tiles_total + ns - 1) / ns, MAX_TPS);
  const int tile_begin = (second ? split - nsplit : split) * tps;
  const int tile_end = min(tile_begin + tps, tiles_total);
  const int my_tiles = max(tile_end - tile_begin, 0);
  if (my_tiles == 0) {                             // an empty range (a short miss list): its rows are never read
    if (tid < HPG && hg * HPG + tid < H)
      *reinterpret_cast<float2*>(lse_part + 2 * ((((size_t)bt * pitch + split0 + split) * H) + hg * HPG + tid)) = make_float2(-__builtin_inff(), 1.f);
    return;
  }
  __builtin_amdgcn_sched_barrier(0);

  // this thread's share of the split's entry list: asked for first, so that it arrives while the queries are staged
  const int32_t* lrow = my_list + (size_t)bt * kk;
  const uint8_t* pbase = pool + (size_t)b * S * row_stride;
  constexpr int SLOTS_PT = MAX_TPS * TILE / NTH;   // 8 list entries per thread at most
  int my_slot[SLOTS_PT];
#pragma unroll
  for (int u = 0; u < SLOTS_PT; ++u) {
    const int j = tid + NTH * u, e = tile_begin * TILE + j;
    const int sl = (j < my_tiles * TILE && e < n) ? lrow[e] : -1;
    my_slot[u] = (sl < 0 || sl >= S) ? (int)0xff800000 : sl;
  }
  // Q^T as the B operand, stationary: lane (hh, h) holds dims 16 ks + 8 hh .. + 7 of head h for every k-step.  A wave
  // brings its own 32 rows, half the dimensions at a time, through the part of the tile buffers that the first two
  // tiles do not use (no other wave touches its part, so there is no barrier): whole cache lines from memory, 16-byte
  // granules XOR-swizzled by row so that the fragment reads are conflict-free.  Lanes past the last head repeat it:
  // their results are not written.
  constexpr int QOFF = (kDma ? 2 : 1) * TR_RAW_BYTES;
  const uint32_t qlds = lds0 + (uint32_t)(QOFF + wave * Q_HALF_BYTES);
  const uint8_t* qbase = reinterpret_cast<const uint8_t*>(q + ((size_t)bt * H + (size_t)min(head0, H - 1)) * ESS_ROW_DIM);
  constexpr int QLOADS = Q_HALF_BYTES / 1024;      // 18
  uint32_t qoff[QLOADS];
#pragma unroll
  for (int i = 0; i < QLOADS; ++i) {
    const uint32_t gr = (uint32_t)(64 * i + lane), row = (gr * 1821u) >> 16, c = gr - 36u * row;     // row = gr / 36 (gr < 1152)
    qoff[i] = (uint32_t)min((int)row, max(H - 1 - head0, 0)) * (ESS_ROW_DIM * 2) + ((c ^ ((row >> 2) & 3u)) << 4);
  }
  auto q_bring = [&](int half) {
    if (wave_active) {
#pragma unroll
      for (int i = 0; i < QLOADS; ++i) dma16_base(qbase + half * 576, qoff[i], qlds + (uint32_t)(i * 1024));
    }
  };
  bf16x8 qb[KS16];
  const uint8_t* const qread = lds + QOFF + wave * Q_HALF_BYTES + h32 * 576;
  const uint32_t qx = (uint32_t)((hh ^ ((h32 >> 2) & 3)) << 4);
  auto q_take = [&](auto halfc) {
    constexpr int half = decltype(halfc)::value;
#pragma unroll
    for (int ks = 0; ks < KS16 / 2; ++ks)
      qb[half * (KS16 / 2) + ks] = *reinterpret_cast<const bf16x8*>(qread + (qx ^ (uint32_t)((ks & 1) << 5)) + 64 * (ks >> 1));
#pragma unroll
    for (int ks = 0; ks < KS16 / 2; ++ks) asm volatile("" : "+v"(qb[half * (KS16 / 2) + ks]) : : "memory");     // read, before the place is written again
  };
  __builtin_amdgcn_sched_barrier(0);
  q_bring(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < SLOTS_PT; ++u)
    if (tid + NTH * u < my_tiles * TILE) slot_cache[tid + NTH * u] = my_slot[u];
  wait_vmcnt<0>();
  asm volatile("" ::: "memory");
  q_take(std::integral_constant<int, 0>{});
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);

  // Gathers of one tile: this wave brings rows 8w..8w+7, one instruction per row (bf16: the latent part, the row's
  // granules swizzled by the per-lane offset; quantised: the whole entry as it is), and for bf16 the rope parts of
  // the same rows by one more.  Row addresses are scalar arithmetic (a pool is below 4 GiB per sequence).
  const int rr = wave * 8 + (lane >> 3);
  uint32_t goff = kDma ? (uint32_t)((lane ^ (2 * (wave & 1))) << 4) : (uint32_t)(lane << 4);
  const uint32_t rope_off = 1024u + (uint32_t)(((lane & 7) ^ (rr & 7)) * 16);
  auto row_base = [&](int slot) -> const uint8_t* {
    return (slot >= 0 ? pbase : zero_row) + (uint32_t)max(slot, 0) * (uint32_t)row_stride;
  };
  struct Slots { int row[8]; int rope; };          // slots of the rows a wave brings: read before they are needed
  auto gather_slots = [&](int it, Slots& g) {
    const int32_t* ts = slot_cache + it * TILE;
#pragma unroll
    for (int r8 = 0; r8 < 8; ++r8) g.row[r8] = __builtin_amdgcn_readfirstlane(ts[wave * 8 + r8]);
    g.rope = kDma ? ts[rr] : 0;
  };
  auto gather_step = [&](int it, int step, const Slots& g, uint32_t go) {       // step 0..7: a row, 8: the rope parts
    if constexpr (kDma) {
      const uint32_t raw = lds0 + (uint32_t)((it % NBUF) * TR_RAW_BYTES);
      if (step < 8) {
        dma16_base(row_base(g.row[step]), go ^ (uint32_t)(((step & 3) << 6) | ((step >> 2) << 4)), raw + (uint32_t)((wave * 8 + step) * TRP));
      } else {
        dma16((g.rope >= 0 ? pbase : zero_row) + (uint32_t)max(g.rope, 0) * (uint32_t)row_stride + rope_off, raw + (uint32_t)(TR_KL_BYTES + wave * 1024));
      }
    } else if (step < 8) {
      dma16_entry(row_base(g.row[step]), go, lds0 + (uint32_t)(RAW_OFF + (it % NRAW) * F8_RAW_BYTES + (wave * 8 + step) * F8_PITCH));
    }
  };
  auto gather = [&](int it) {
    Slots g;
    gather_slots(it, g);
#pragma unroll
    for (int step = 0; step < PER_TILE; ++step) gather_step(it, step, g, goff);
  };
  gather(0);
  q_bring(1);
  if (my_tiles > 1) gather(1);

  __builtin_amdgcn_sched_barrier(0);
  AgprHold hold;
  agpr_claim(hold);
  acc_zero();
  __builtin_amdgcn_sched_barrier(0);
  float m_ref = -__builtin_inff(), l_run = 0.f;

  // lane constants of the two LDS access patterns.  K fragment of k-step ks: row h32, granule 2 ks + hh, i.e.
  // kbase ^ ((ks & 7) << 5) plus 256 (ks >> 3) (the swizzle touches the low four granule bits only); rope
  // k-steps read the rope region.  V^T fragment of block vb, k-step s: rows 16 s + 4 hh + ti (+ 8), columns
  // 32 vb + 16 gi + 4 tj ..: vbase{0,1} ^ ((vb & 3) << 6) plus 256 (vb >> 2) plus 16 s rows.
  const int fk = tr_swz(h32);
  uint32_t kbase = (uint32_t)(h32 * TRP + ((hh ^ fk) << 4));
  uint32_t rbase = (uint32_t)(TR_KL_BYTES + h32 * 128 + ((hh ^ (h32 & 7)) << 4));
  const int gi = (lane >> 4) & 1, ti = (lane & 15) >> 2, tj = lane & 3;
  const int vrow0 = 4 * hh + ti;
  uint32_t vbase0 = (uint32_t)(vrow0 * TRP + (((2 * gi + (tj >> 1)) ^ tr_swz(vrow0)) << 4) + (tj & 1) * 8);
  // (row vrow0 + 8: granule bit 1 of the swizzle differs)

  // Quantised entries: the wave's own rows of a tile go from the raw ring to the tile's buffer as bf16, in the layout
  // the gathers of bf16 entries produce; unit u = rows 2u + hh of the wave's eight, 16 values per lane.
  struct Raw { uint4 x; uint32_t sc; };
  int ctid = tid;                                // laundered per iteration: nothing derived from it stays in registers
  struct Places { const uint8_t *x, *sc; uint32_t dst; };
  auto cv_places = [&](int it) {                 // of unit 0; unit u is 2 u rows further on
    const int c = ctid & 31, hi = (ctid >> 5) & 1;
    const uint8_t* raw = lds + RAW_OFF + (it % max(NRAW, 1)) * F8_RAW_BYTES + (wave * 8 + hi) * F8_PITCH;
    return Places{raw + c * 16, raw + 512 + 2 * (c >> 3),
                  (uint32_t)((it % NBUF) * TR_RAW_BYTES + (wave * 8 + hi) * TRP + (((2 * c) ^ (hi << 2) ^ (2 * (wave & 1))) << 4))};
  };
  auto cv_load = [&](const Places& at, int u, Raw& r) {
    r.x = *reinterpret_cast<const uint4*>(at.x + 2 * u * F8_PITCH);
    r.sc = *reinterpret_cast<const uint16_t*>(at.sc + 2 * u * F8_PITCH);
  };
  // a quarter of the lane's 16 values; the second and the fourth complete a 16-byte granule and write it
  auto cv_quarter = [&](const Places& at, int u, int quarter, const Raw& r, uint32_t (&o)[4]) {
    const float sc = __uint_as_float(r.sc << 16);
    const uint32_t w = quarter == 0 ? r.x.x : (quarter == 1 ? r.x.y : (quarter == 2 ? r.x.z : r.x.w));
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
    const int half = quarter >> 1, d = quarter & 1;
    o[2 * d] = pack_bf16(lo[0] * sc, lo[1] * sc);
    o[2 * d + 1] = pack_bf16(hi[0] * sc, hi[1] * sc);
    // the swizzle of row 8w + 2u + hi differs from that of row 8w + hi by constants of u
    if (d)
      *reinterpret_cast<uint4*>(lds + (at.dst ^ (uint32_t)(((u & 1) << 7) | (((u >> 1) ^ half) << 4))) + 2 * u * TRP) = make_uint4(o[0], o[1], o[2], o[3]);
  };
  auto cv_rope = [&](int it) {                   // 8 rows x 8 pieces; the rope part starts 520 bytes into the entry (8-byte aligned)
    const int r = (ctid & 63) >> 3, c = ctid & 7;
    const uint2* src = reinterpret_cast<const uint2*>(lds + RAW_OFF + (it % max(NRAW, 1)) * F8_RAW_BYTES + (wave * 8 + r) * F8_PITCH + 520 + c * 16);
    const uint2 lo = src[0], hi = src[1];
    *reinterpret_cast<uint4*>(lds + (it % NBUF) * TR_RAW_BYTES + TR_KL_BYTES + (wave * 8 + r) * 128 + ((c ^ r) * 16)) = make_uint4(lo.x, lo.y, hi.x, hi.y);
  };
  auto convert = [&](int it) {                   // a whole tile, outside the pipeline
    const Places at = cv_places(it);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      Raw r;
      uint32_t o[4];
      cv_load(at, u, r);
#pragma unroll
      for (int qr = 0; qr < 4; ++qr) cv_quarter(at, u, qr, r, o);
    }
    cv_rope(it);
  };
  // at most `left` tiles of this wave's gathers still in flight
  auto wait_tiles = [&](int left) {
    if (left >= 1) wait_vmcnt<PER_TILE>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
  };
  wait_tiles(my_tiles > 1 ? 1 : 0);              // tile 0 and the second half of the queries
  q_take(std::integral_constant<int, 1>{});
  if constexpr (!kDma) {
    convert(0);
  }

  // One wave per SIMD issues its instructions one at a time, so the loop is a software pipeline in which everything
  // else rides in the shadow of the 68 MFMAs of a tile (32 cycles each), in a pinned order.  Iteration `it`
  //   1. computes S^T of tile it (a chain of 36 MFMAs) and, between them, turns the logits of tile it-1 into P^T
  //      (exponentials, row sums, bf16 pairs) and issues the gathers of tile it+2;
  //   2. issues the second product of tile it-1 and, between its MFMAs, takes the maxima of S^T of tile it (which
  //      may move the softmax reference: the accumulators are then rescaled before the next second product) and, for
  //      quantised entries, brings tile it+1 to bf16.
  // The accumulator of S^T starts from the slot list itself: a valid slot number, read as a float, is a denormal below
  // 1e-38, and a masked entry's word is -inf.
  floatx16 sprev;                              // S^T of the previous tile (rows 8 q + 4 hh + i at index 4 q + i)
  float m_use = 0.f;                           // the reference its exponentials are taken against
  float alpha_pending = 1.f;                   // rescale of the accumulators due before the next second product
  bool scale_pending = false;
  // one iteration; QK: there is a tile `it` to start, PV: there is a tile it-1 to finish, MORE: there is a tile it+2 to
  // gather, NEXT: there is a tile it+1 (to convert, if quantised)
  auto iteration = [&](int it, auto qkc, auto pvc, auto nextc, auto morec) {
    constexpr bool QK = decltype(qkc)::value, PV = decltype(pvc)::value, MORE = decltype(morec)::value,
                   CONV = !kDma && decltype(nextc)::value;
    const uint32_t KLo = (uint32_t)((it % NBUF) * TR_RAW_BYTES);
    const uint32_t KLp = lds0 + (uint32_t)(((it + NBUF - 1) % NBUF) * TR_RAW_BYTES);     // tile it-1
    Slots gs;
    // (the lane constants pass through an empty statement, so that what is derived from them is computed where it is
    // used instead of being kept in registers that the loop does not have)
    asm volatile("" : "+v"(kbase), "+v"(rbase), "+v"(vbase0), "+v"(goff));
    if constexpr (!kDma) asm volatile("" : "+v"(ctid));
    agpr_fence(hold);
    if constexpr (QK && kDma) {
      wait_tiles(min(my_tiles - 1 - it, 1));      // this wave's rows of tile `it` have landed
    }
    __syncthreads();                           // ... everyone's did; and everyone is done with tile it-2
    if constexpr (MORE) gather_slots(it + 2, gs);
    if (!wave_active) {
      if constexpr (MORE) {
#pragma unroll
        for (int step = 0; step < PER_TILE; ++step) gather_step(it + 2, step, gs, goff);
      }
    } else {
    floatx16 sacc, sodd;                       // two chains: a dependent MFMA waits twice its 32 cycles
    uint32_t pq[8];                            // P^T of tile it-1 as bf16 pairs: k-step 0 in [0..3], k-step 1 in [4..7]
    float psum = 0.f;
    auto exp_row = [&](auto ic) {              // one row of tile it-1: exponential, row sum, and every second row a bf16 pair
      constexpr int i = decltype(ic)::value;
      sprev[i] = __builtin_amdgcn_exp2f(fmaf(sprev[i], scale_log2e, -m_use));     // the argument is <= kLazyMax: no range reduction needed
      psum += sprev[i];
      if constexpr (i & 1) {
        pq[i >> 1] = pack_bf16(sprev[i - 1], sprev[i]);
        asm volatile("" : "+v"(pq[i >> 1]), "+v"(psum));        // here, not where it is used
      }
    };
    if constexpr (QK) {
      // 36 k-steps: the eight swizzle variants one after the other, four 256-byte groups each, then the rope; A
      // fragments are read CK steps ahead
      constexpr int CK = 6;
      bf16x8 fa[CK];
      uint32_t ka = 0;
      auto read_k = [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        if constexpr ((t & 3) == 0) {
          ka = KLo + (t < 32 ? (kbase ^ (uint32_t)((t >> 2) << 5)) : rbase);
          asm volatile("" : "+v"(ka));
        }
        if constexpr (t < 32) fa[t % CK] = *reinterpret_cast<const bf16x8*>(lds + ka + 256 * (t & 3));
        else fa[t % CK] = *reinterpret_cast<const bf16x8*>(lds + (ka ^ (uint32_t)((t & 3) << 5)));
      };
      const int32_t* tile_slot = slot_cache + it * TILE + 4 * hh;
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(tile_slot + 8 * qd);
        sacc[4 * qd] = v[0]; sacc[4 * qd + 1] = v[1]; sacc[4 * qd + 2] = v[2]; sacc[4 * qd + 3] = v[3];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) sodd[i] = 0.f;
      [&]<int... J>(std::integer_sequence<int, J...>) { (read_k(std::integral_constant<int, J>{}), ...); }
      (std::make_integer_sequence<int, CK>{});
      auto qk_step = [&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int ks = t < 32 ? 8 * (t & 3) + (t >> 2) : t;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t & 1) sodd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[t % CK], qb[ks], sodd, 0, 0, 0);
        else sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[t % CK], qb[ks], sacc, 0, 0, 0);
        if constexpr (t + CK < KS16) read_k(std::integral_constant<int, t + CK>{});
        if constexpr (MORE && (t & 3) == 3) gather_step(it + 2, t >> 2, gs, goff);
        if constexpr (PV && (t & 1) == 0 && (t >> 1) < 16) exp_row(std::integral_constant<int, (t >> 1)>{});
      };
      [&]<int... K>(std::integer_sequence<int, K...>) { (qk_step(std::integral_constant<int, K>{}), ...); }
      (std::make_integer_sequence<int, KS16>{});
      __builtin_amdgcn_sched_barrier(0);
    } else {
      [&]<int... I>(std::integer_sequence<int, I...>) { (exp_row(std::integral_constant<int, I>{}), ...); }
      (std::make_integer_sequence<int, 16>{});
    }
    if constexpr (PV) l_run += psum;
    agpr_fence(hold);
    if (scale_pending) {                       // wave-uniform; rare
      acc_scale(alpha_pending);
      scale_pending = false;
    }
    if constexpr (CONV) wait_tiles(min(my_tiles - 2 - it, 1));     // this wave's raw rows of tile it+1 have landed
    // second product of tile it-1: 32 MFMAs
    constexpr int CV = 8;
    bf16x8 fv[CV];
    uint32_t va = 0, vc = 0;
    auto read_v = [&](auto jc) {               // step j: swizzle variant x = j >> 3, k-step s = (j >> 2) & 1, group y = j & 3: block 4 y + x
      constexpr int j = decltype(jc)::value, x = j >> 3, s = (j >> 2) & 1, y = j & 3;
      if constexpr ((j & 7) == 0) {
        va = KLp + (vbase0 ^ (uint32_t)(x << 6));
        vc = KLp + (vbase0 ^ (uint32_t)((x << 6) | 32)) + 8 * TRP;
        asm volatile("" : "+v"(va), "+v"(vc));
      }
      fv[j % CV] = tr_frag(va + 256u * y + 16u * s * TRP, vc + 256u * y + 16u * s * TRP);
    };
    if constexpr (PV) {
      [&]<int... J>(std::integer_sequence<int, J...>) { (read_v(std::integral_constant<int, J>{}), ...); }
      (std::make_integer_sequence<int, CV>{});
    }
    Raw raw;
    Places places;
    uint32_t conv[4];
    if constexpr (CONV) places = cv_places(it + 1);
    float mx = 0.f;
    auto step = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PV) {
        constexpr int vb = 4 * (j & 3) + (j >> 3);
        uint4 pw = ((j >> 2) & 1) == 0 ? make_uint4(pq[0], pq[1], pq[2], pq[3]) : make_uint4(pq[4], pq[5], pq[6], pq[7]);
        pv_mfma<vb, (j == 0 || j == 4)>(fv[j % CV], *reinterpret_cast<bf16x8*>(&pw));
        if constexpr (j + CV < 2 * VB32) read_v(std::integral_constant<int, j + CV>{});
      }
      if constexpr (CONV) {                    // four units of 16 values per lane, eight steps each; the rope parts
        constexpr int u = j >> 3;
        if constexpr ((j & 7) == 0) cv_load(places, u, raw);
        if constexpr ((j & 7) >= 3 && (j & 7) < 7) cv_quarter(places, u, (j & 7) - 3, raw, conv);
        if constexpr (j == 31) cv_rope(it + 1);
      }
      if constexpr (QK) {
        if constexpr (j >= 8 && j < 16) {
          constexpr int i = 2 * (j - 8);
          sacc[i] += sodd[i];
          sacc[i + 1] += sodd[i + 1];
          mx = j == 8 ? fmaxf(sacc[0], sacc[1]) : fmaxf(mx, fmaxf(sacc[i], sacc[i + 1]));
        }
      }
    };
    [&]<int... J>(std::integer_sequence<int, J...>) { (step(std::integral_constant<int, J>{}), ...); }
    (std::make_integer_sequence<int, 2 * VB32>{});
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (QK) {
      const float tmax = pair_max(mx) * scale_log2e;
      // move the reference only when this tile exceeds it by more than 2^kLazyMax (always from -inf)
      const bool move = tmax > m_ref + kLazyMax;
      if (__any(move)) {
        const float m_new = move ? tmax : m_ref;
        alpha_pending = m_ref == -__builtin_inff() ? 1.f : exp2f(m_ref - m_new);   // m_ref = -inf: nothing has been added up yet
        l_run *= alpha_pending;
        // The accumulators are rescaled once the MFMAs of tile it-1 are through -- 1280 instructions, 2.5 us -- but not where
        // every head that moves comes from -inf, as in the first tile of nearly every range.
        scale_pending = __any(move && m_ref != -__builtin_inff());
        m_ref = m_new;
      }
      m_use = (m_ref == -__builtin_inff()) ? 0.f : m_ref;
      sprev = sacc;
    }
    }
    if constexpr (CONV) {
      if (!wave_active) {
        wait_tiles(min(my_tiles - 2 - it, 1));
        convert(it + 1);
      }
    }
  };
  using T_ = std::true_type; using F_ = std::false_type;
  iteration(0, T_{}, F_{}, F_{}, F_{});          // (past its barrier every wave has its queries: their place is free)
  if (my_tiles > 2) gather(2);
  if constexpr (!kDma) {
    if (my_tiles > 1) {
      wait_tiles(min(my_tiles - 2, 1));
      convert(1);
    }
  }
  int it = 1;
  for (; it + 2 < my_tiles; ++it) iteration(it, T_{}, T_{}, T_{}, T_{});
  if (it + 1 < my_tiles) { iteration(it, T_{}, T_{}, T_{}, F_{}); ++it; }
  if (it < my_tiles) iteration(it, T_{}, T_{}, F_{}, F_{});
  iteration(my_tiles, F_{}, T_{}, F_{}, F_{});
  // the hazard logic does not see the MFMAs inside the asm statements: let the last ones retire
  // before their results are read
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
  agpr_fence(hold);

  {
    // lane constants afresh (see above): nothing of the epilogue is carried through the tile loop
    int tid2 = threadIdx.x;
    asm volatile("" : "+v"(tid2));
    const int hh2 = (tid2 >> 5) & 1, h2 = tid2 & 31, head = head0 + h2;
    const float l_tot = pair_sum(l_run);
    float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    const size_t prow = ((size_t)bt * pitch + split0 + split) * H + min(head, H - 1);
    // The partial result goes through LDS (the tile buffers are free now), 128 columns at a time, so that it leaves in
    // pieces of 256 bytes per row: a lane holds four consecutive columns at a time, of a row 1 KiB away from its
    // neighbour's.  A wave stages and writes its own 32 rows; rows at a pitch of 264 bytes: the 32 heads of a
    // half-wave write 8 bytes each to 64 different banks.
    // fp16 holds magnitudes below 65504.  The rows are written as they are, the largest magnitude noted on the way;
    // should a head's reach 2^15 (entry values of that size: rare) the wave writes once more, such heads divided by the
    // power of two that brings their largest value below 2^15 -- exact, and undone by the merge -- and what fp16 still
    // cannot hold clamped.  A value that is no number is written as one in either pass.
    __syncthreads();                                 // every wave is done with the last tile
    float amax = 0.f, down = 1.f;
    const int rows_here = min(HPW, H - head0);
    uint8_t* const obytes = reinterpret_cast<uint8_t*>(o_part + (((size_t)bt * pitch + split0 + split) * H + head0) * ESS_LATENT_DIM);
    auto write_rows = [&](auto clampc) {
      constexpr bool CLAMP = decltype(clampc)::value;
      auto chunk = [&](auto cc) {                    // columns 128 c ..
        constexpr int c = decltype(cc)::value;
        int t3 = threadIdx.x;
        asm volatile("" : "+v"(t3));                 // (addresses are computed per chunk, not kept)
        uint8_t* const stage = lds + (wave * 2 + (c & 1)) * (HPW * O_PITCH);
        uint8_t* const orow = stage + (t3 & 31) * O_PITCH + 8 * ((t3 >> 5) & 1);
        auto block = [&](auto vbc) {
          constexpr int v4 = decltype(vbc)::value;
          float o[16];
          acc_read_block<4 * c + v4>(o, std::make_integer_sequence<int, 16>{});
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) {
            floatx4 ov = floatx4{o[4 * qd] * inv, o[4 * qd + 1] * inv, o[4 * qd + 2] * inv, o[4 * qd + 3] * inv};
            if constexpr (CLAMP) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {          // never inf in the fp16 image; what is no number stays so (fmed3 would make it -65504)
                const float in_range = __builtin_amdgcn_fmed3f(ov[i], -65504.f, 65504.f);
                ov[i] = ov[i] != ov[i] ? ov[i] : in_range;
              }
            } else {
              amax = fmaxf(amax, fmaxf(fabsf(ov[0]), fabsf(ov[1])));       // (of the numbers: a NaN is skipped)
              amax = fmaxf(amax, fmaxf(fabsf(ov[2]), fabsf(ov[3])));
            }
            *reinterpret_cast<halfx4*>(orow + (v4 * 32 + 8 * qd) * 2) = __builtin_convertvector(ov, halfx4);   // round to nearest even
          }
        };
        block(std::integral_constant<int, 0>{}); block(std::integral_constant<int, 1>{});
        block(std::integral_constant<int, 2>{}); block(std::integral_constant<int, 3>{});
        // lanes read what other lanes of their wave wrote: a wave's LDS accesses are in order, and nothing may be moved across
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int r4 = 0; r4 < HPW / 4; ++r4) {
          const int r = min(4 * r4 + ((t3 & 63) >> 4), rows_here - 1);      // past the last head: its row once more
          const uint2* src = reinterpret_cast<const uint2*>(stage + r * O_PITCH + (t3 & 15) * 16);
          const uint2 lo = src[0], hi = src[1];
          ess_store_nt(reinterpret_cast<uint4*>(obytes + (uint32_t)(r * (ESS_LATENT_DIM * 2) + 256 * c + (t3 & 15) * 16)), make_uint4(lo.x, lo.y, hi.x, hi.y));
        }
      };
      chunk(std::integral_constant<int, 0>{}); chunk(std::integral_constant<int, 1>{});
      chunk(std::integral_constant<int, 2>{}); chunk(std::integral_constant<int, 3>{});
    };
    if (wave_active) {
    write_rows(std::false_type{});
    amax = pair_max(amax);
    if (__any(amax >= 32768.f)) {
      int ex = 0;
      (void)frexpf(amax, &ex);                       // amax < 2^ex
      down = (amax >= 32768.f && amax <= 3.0e38f) ? ldexpf(1.f, ex - 15) : 1.f;
      inv = inv / down;
      write_rows(std::true_type{});
    }
    }
    agpr_release(hold);                              // the accumulators are read out: the AGPRs are the compiler's again
    if (head < H && hh2 == 0)
      *reinterpret_cast<float2*>(lse_part + 2 * prow) = make_float2(l_tot > 0.f ? (m_ref + log2f(l_tot)) * kLn2 : -__builtin_inff(), down);
  }
  };
  if constexpr (DYN) {
    for (;;) {
      int item;
      for (;;) {
        // ticket v of class cls: row (v / per_row) * nw + cls, item v % per_row of that row
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
    int split = blockIdx.y, bt = blockIdx.x;
    if (fetch.wgs) {                               // (see ess_fetch; one head group)
      const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
      if (x < 2) {
        if (2 * j + x < fetch.wgs) ess_fill::entries<4>(fetch, reinterpret_cast<int32_t*>(lds), (2 * j + x) * 4 + (int)(threadIdx.x >> 6), fetch.wgs * 4);
        return;
      }
      const uint32_t item = (uint32_t)(6 * j + x - 2);
      split = (int)(n_bt == 1 ? item : __umulhi(item, bt_inv));
      bt = (int)item - split * n_bt;
      if (split >= nsplit) return;
    }
    run_item(split, bt, blockIdx.z);
  }
}

// out[bt,h,:] = sum_s exp(lse_s - lse) * o_s ;  lse = log sum_s exp(lse_s), s < nsplit <= 64.  WPR waves per (bt,h): one,
// or four (a workgroup per row) where the rows are too few to fill the chip and their many splits would be read a few
// at a time; then each wave sums every fourth split and the first adds them up.  Lane s holds the weight of split s;
// the partial results of eight splits are requested before any is used, those of empty splits not at all.
// `zero_cnt` (may be NULL): n_zero counters the first workgroup clears, for steps that have no other kernel to do it in.
template <int WPR>
__global__ __launch_bounds__(256) void k_attn_merge(const _Float16* __restrict__ o_part, const float* __restrict__ lse_part,
                                                    int H, int nsplit, int total_rows, uint16_t* __restrict__ out,
                                                    float* __restrict__ lse_out, int32_t* __restrict__ zero_cnt,
                                                    int n_zero, ess_ticket_check chk) {
  __shared__ float s_part[WPR == 1 ? 1 : 3][WPR == 1 ? 1 : 8][64];
  if (zero_cnt && blockIdx.x == 0)
    for (int i = threadIdx.x; i < n_zero; i += 256) zero_cnt[i] = 0;
  if (chk.tickets && blockIdx.x == 0 && threadIdx.x == 0) ess_check_tickets(chk);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int sub = WPR == 1 ? 0 : wave;
  const int rowi = WPR == 1 ? blockIdx.x * 4 + wave : blockIdx.x;          // bt*H + h
  if (rowi >= total_rows) return;                                          // (whole workgroups with WPR 4: their grid is exact)
  const int bt = rowi / H, h = rowi % H;
  const size_t base = ((size_t)bt * nsplit) * H + h;
  constexpr int U = 16 / (WPR == 1 ? 2 : 1);        // splits of a wave requested at a time
  // one load per lane for the split weights ...
  const float2 lu = lane < nsplit ? *reinterpret_cast<const float2*>(lse_part + 2 * (base + (size_t)lane * H)) : make_float2(-__builtin_inff(), 1.f);
  // ... and, with four waves per row (at most 16 splits each), all partial results beside it: waiting for the weights
  // first would be most of such a kernel.  What the place of an empty split holds is not used.
  halfx8 xy[U];
  if constexpr (WPR > 1) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      xy[u] = *reinterpret_cast<const halfx8*>(o_part + (base + (size_t)min(sub + u * WPR, nsplit - 1) * H) * ESS_LATENT_DIM + lane * 8);
  }
  float mx = lu.x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
  const bool any = mx > -__builtin_inff();
  const float wgt = lu.x == -__builtin_inff() || !any ? 0.f : __expf(lu.x - mx);
  float den = wgt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) den += __shfl_xor(den, d, 64);
  const float wu = wgt * lu.y;                       // .y: the power of two a split's fp16 values were divided by
  // (every split that is not empty: a weight that underflows to 0 still meets the split's values)
  const unsigned long long full = any ? __ballot(lu.x != -__builtin_inff()) : 0ull;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s0 = sub; s0 < nsplit; s0 += U * WPR) {
    if constexpr (WPR == 1) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = s0 + u;
        xy[u] = halfx8{0, 0, 0, 0, 0, 0, 0, 0};
        if (s < nsplit && ((full >> s) & 1ull))       // the same for the whole wave
          xy[u] = *reinterpret_cast<const halfx8*>(o_part + (base + (size_t)s * H) * ESS_LATENT_DIM + lane * 8);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + u * WPR;
      if (s >= nsplit || !((full >> s) & 1ull)) continue;
      const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wu), s));
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] += w * (float)xy[u][i];
    }
  }
  if constexpr (WPR > 1) {
    if (sub > 0)
#pragma unroll
      for (int i = 0; i < 8; ++i) s_part[sub - 1][i][lane] = a[i];
    __syncthreads();
    if (sub > 0) return;
#pragma unroll
    for (int x = 0; x < WPR - 1; ++x)
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] += s_part[x][i][lane];
  }
  const float inv = den > 0.f ? 1.0f / den : 0.f;
  uint4 o = make_uint4(pack_bf16(a[0] * inv, a[1] * inv), pack_bf16(a[2] * inv, a[3] * inv),
                       pack_bf16(a[4] * inv, a[5] * inv), pack_bf16(a[6] * inv, a[7] * inv));
  ess_store_nt(reinterpret_cast<uint4*>(out + (size_t)rowi * ESS_LATENT_DIM + lane * 8), o);
  if (lse_out && lane == 0) lse_out[rowi] = den > 0.f ? mx + __logf(den) : -__builtin_inff();
}

}  // namespace

int ess_attn_min_splits(const ess_config& c) {
  const int tiles = (c.topk + TILE - 1) / TILE;
  return (tiles + MAX_TPS - 1) / MAX_TPS;
}

// At context creation (on the context's device): the partial-attention kernels use more dynamic LDS than the default limit.
int ess_init_attn_kernels() {
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_partial_tr<ESS_FMT_BF16, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, tr_lds_bytes(ESS_FMT_BF16)));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_partial_tr<ESS_FMT_BF16, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, tr_lds_bytes(ESS_FMT_BF16)));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_partial_tr<ESS_FMT_FP8, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, tr_lds_bytes(ESS_FMT_FP8)));
  ESS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attn_partial_tr<ESS_FMT_FP8, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, tr_lds_bytes(ESS_FMT_FP8)));
  return ess_init_attn_h32();
}

int ess_launch_attn_partial(ess_ctx* ctx, const void* q, const uint8_t* slot_pool, const int32_t* list,
                            const int32_t* n_list, int B, int T, int split0, int nsplit, int pitch, hipStream_t st, int b0, ess_xcd xcd,
                            hipEvent_t done, const int32_t* list_b, const int32_t* n_list_b, int nsplit_b, const ess_fetch* fetch) {
  const ess_config& c = ctx->cfg;
  if (split0 + nsplit + nsplit_b > pitch || (size_t)(b0 + B) * T * pitch > ctx->part_cap) return ess_fail(ESS_ERR_INVALID_ARG, "internal: partial results");
  if (nsplit < ess_attn_min_splits(c)) return ess_fail(ESS_ERR_INVALID_ARG, "internal: too few attention splits");
  const int n_hg = (c.attn_heads + HPG - 1) / HPG;      // 128 heads per workgroup
  dim3 grid(B * T, nsplit + nsplit_b, n_hg);
  if (xcd.ticket) grid = dim3(ess_xcd_grid((nsplit + nsplit_b) * B * T * n_hg, xcd));     // one workgroup per CU
  ess_fetch fe{};
  if (fetch) {
    if (xcd.ticket || nsplit_b || n_hg != 1) return ess_fail(ESS_ERR_INVALID_ARG, "internal: attention launch with a fetch");
    fe = *fetch;
    const int groups = (nsplit * B * T + 5) / 6;
    grid = dim3(8 * (groups > (fe.wgs + 1) / 2 ? groups : (fe.wgs + 1) / 2));
  }
  const uint32_t bt_inv = 0xffffffffu / (uint32_t)(B * T) + 1;      // division by B * T > 1 of numbers up to 2^18: exact
  const float sc = c.sm_scale * kLog2e;
  const uint16_t* qq = static_cast<const uint16_t*>(q);
  // partial results of sequence b0 onward
  _Float16* op = reinterpret_cast<_Float16*>(ctx->o_part) + (size_t)b0 * T * pitch * c.attn_heads * ESS_LATENT_DIM;
  float* lp = ctx->lse_part + (size_t)b0 * T * pitch * c.attn_heads * 2;
#define ESS_ATTN_LAUNCH(FMT, DYN)                                                                                      \
  ESS_HIP(ess_launch_done(done, &k_attn_partial_tr<FMT, DYN>, grid, dim3(NTH), (size_t)tr_lds_bytes(FMT), st, qq, slot_pool, list, n_list, T, \
                     c.attn_heads, c.topk, c.slots_per_seq, c.row_stride, sc, split0, nsplit, pitch, op, lp, ctx->zero_row, xcd,  \
                     B * T, n_hg, list_b, n_list_b, nsplit_b, fe, bt_inv))
  if (c.latent_fmt == ESS_FMT_BF16) {
    if (xcd.ticket) ESS_ATTN_LAUNCH(ESS_FMT_BF16, true); else ESS_ATTN_LAUNCH(ESS_FMT_BF16, false);
  } else {
    if (xcd.ticket) ESS_ATTN_LAUNCH(ESS_FMT_FP8, true); else ESS_ATTN_LAUNCH(ESS_FMT_FP8, false);
  }
#undef ESS_ATTN_LAUNCH
  ESS_HIP(hipGetLastError());
  return ESS_OK;
}

int ess_launch_attn_merge(ess_ctx* ctx, int B, int T, int nsplit_total, bool wide, void* out_bf16, float* lse, hipStream_t st,
                          int32_t* zero_cnt, int n_zero, int b0, const ess_ticket_check* check, hipEvent_t done) {
  const int H = ctx->cfg.attn_heads;
  ess_ticket_check chk{};
  if (check) chk = *check;
  const int rows = B * T * H;
  const size_t r0 = (size_t)b0 * T * H;                       // first (bt, h) row of the sub-batch
  const _Float16* op = reinterpret_cast<const _Float16*>(ctx->o_part) + r0 * nsplit_total * ESS_LATENT_DIM;
  const float* lp = ctx->lse_part + r0 * nsplit_total * 2;
  uint16_t* o = static_cast<uint16_t*>(out_bf16) + r0 * ESS_LATENT_DIM;
  float* ls = lse ? lse + r0 : nullptr;
  if (wide)
    ESS_HIP(ess_launch_done(done, &k_attn_merge<4>, dim3(rows), dim3(256), 0, st, op, lp, H, nsplit_total, rows, o, ls, zero_cnt, n_zero, chk));
  else
    ESS_HIP(ess_launch_done(done, &k_attn_merge<1>, dim3((rows + 3) / 4), dim3(256), 0, st, op, lp, H, nsplit_total, rows, o, ls, zero_cnt, n_zero, chk));
  return ESS_OK;
}
