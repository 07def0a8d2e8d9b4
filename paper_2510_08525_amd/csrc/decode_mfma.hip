// Split-K decode attention, MFMA variant (tiled bf16 stores).
//
// Same operation as the row-major variant (softmax attention of the G query heads of a
// group over the rows a store holds; paper Sec. 3.1 Eq. 1 at gate 0/1, Sec. 3.3), with the
// two contractions on the matrix cores:
//   scores  S[slot][head] = sum_d K[slot][d] * Q[head][d]   v_mfma_f32_16x16x32_bf16,
//                           A = K tile (16 slots x 32 d), B = Q^T (heads padded to 16)
//   output  O[head][d]    = sum_slot P[head][slot] * V[slot][d]   same instruction,
//                           A = V^T tile (k runs over the 32 slots of a tile), B = P^T
// The score accumulator leaves lane l holding head l%16 and slots 4*(l/16)..+3 of each
// 16-slot half, which is exactly the B-operand register layout, so P never moves between
// lanes; O comes out as O^T, each head in the lanes that hold its scores.  The stores are laid out (see rlkv_internal.h) so that
// every 128-bit load per lane is one contiguous kilobyte per wavefront and lands directly in operand registers: no
// LDS staging, no transposes, and the wavefronts of a workgroup run independently until
// the merge.  P is split into a bf16 head and a bf16 remainder (two MFMAs per V block) so
// the weights carry ~16 mantissa bits; the matrix cores are idle most of the time anyway.
//
// Start: the address of the list, and whatever else the first loads need, is in scalar registers before the first instruction
// (kernel arguments loaded ahead, see kShapeGroup); the workgroup's record is one scalar load of 64 bytes, and what the
// scores need of the other arguments comes in its shadow; then the new row's loads, Q's and the first tile's go out together.  (Compiled from one struct of arguments and
// plain pointers, the same start was five to six round trips to memory in a row.)
// Loop: eight wavefronts, two per SIMD, whatever the list; one register image each, K refilled behind the scores and V behind the
// products, every wait for its own registers only.  That last needs care: with a FLAT store possibly in flight - the output through a
// generic pointer - the compiler turns every wait for a load into one for all of them.
// Measured, before / now, us a call: one sequence of 333 tokens and 32 steps (32 query, 8 KV heads) 246 / 219, the launch by itself
// 7.1 / 5.6; 8 x 8192 40.3 / 38.6; 16 gated of 3000 .. 5000 28.8 / 25.1; 24 paged of 2000 .. 20 000 46.6 / 42.5; a 28-layer step of
// 16 x 16 384 1152 / 1088; 32 of 4000 .. 32 000 184.2 / 181.9; 64 of 16 000 .. 64 000 783 / 777.
// Arguments and addresses that the loads do not need behind them (late_arguments): a launch after another, decode / step of one sequence, 32
// and 8 heads, 340 tokens 5.00 / 5.78 -> 4.92 / 5.64, 1030 5.35 / 5.86 -> 5.28 / 5.65.
// Four wavefronts with two register images, exact waits: 185.5 for the 32, 1132 for the step; with one image 185.7 and 1120.
//
// Gated heads (GATED = true; paper Sec. 3.1, Eq. 1): a full head with gate g < 1 returns
// g * full + (1 - g) * local attention.  The local positions (first S, last R) are a subset of
// the full ones, so the same pass keeps a second accumulator that only the tiles touching
// those ranges update; the scores of a tile are computed once for both.
//
// Fused single-token append (FUSED = true): the kernel also performs this step's append.
// Every sequence grows by one position; the wavefront that owns the tile holding the new
// slot of a pair writes the new K/V row into the store (sink slot, ring slot - evicting
// position p - R - or next row of a full head); each lane writes exactly the bytes it later loads, so no other wavefront ever
// depends on the write, and where the tile is the first one, asked for already, the row goes into its registers as well.  No
// workgroup reads a length from the table: a pair's length is its length when the work list was
// planned plus the list's growth counter (ListHeader::grow), which no workgroup writes while another
// one reads it, so the kernel needs no grid-wide fence: with a merge kernel behind it every workgroup reads
// the counter and that kernel advances it - no per-step argument, and a captured
// launch can be replayed; without one (whole pairs, or partials merged here, share_merge.h) the count comes as an
// argument, nobody reads the counter, and the first workgroup writes it.  The new lengths are written
// to both copies of the length table for the kernels that do read it.
#include "share_merge.h"

namespace rlkv {
namespace {

// The first 14 words of a kernel's arguments are loaded into scalar registers before its first instruction (the build asks for
// it, -amdgpu-kernarg-preload-count): they are what a workgroup needs to ask for its record.  The others are loaded beside the record.
constexpr uint32_t kShapeGroup = 31, kShapeInTurn = 32, kShapeMore = 64;   // of `shape`; kShapeMore: another layer's list follows
constexpr int kShapeWgs = 8;                                               // workgroups << 8
constexpr int kWaves = 8, kThreads = kWaves * 64;
struct DecodeRest {
  uint16_t* out;
  float scale_log2;
  int32_t n_kv_heads;
  Partials part;
  int64_t list_stride;
  int32_t pair_off, batch;
  int32_t *len0, *len1;          // both copies of the layer's lengths
  int32_t *slot_pos, *v_wide;    // (v_wide: of this layer)
  const int32_t* block_table;
  int64_t page_bytes;
  int32_t page_shift, page_mask, table_stride;
  uint32_t recent_inverse;       // inverse_of(recent)
};

// Online-softmax update and P.V accumulation of one tile into `st`.  A slot counts if it
// lies in the valid prefix [0, n_eff) and, for the local attention of a gated head (LOCAL),
// also in the sink range [0, keep_lo) or the recent range [keep_from, n_eff).  Clears the V
// operands of slots that do not count (they may hold anything).
template <bool LOCAL>
__device__ __forceinline__ void tile_accumulate(TileRegs& t, const float (&raw)[8], Softmax& st, int tile, int n_eff,
                                                int kb, int keep_lo = 0, int keep_from = 0) {
  auto counts = [&](int slot) { return slot < n_eff && (!LOCAL || slot < keep_lo || slot >= keep_from); };
  float sc[8];
  const int slot0 = tile * kTile + kb * 4;
  const bool ragged_tile = tile * kTile + kTile > n_eff ||
                           (LOCAL && tile * kTile + kTile > keep_lo && tile * kTile < keep_from);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int slot = slot0 + (e >> 2) * 16 + (e & 3);
    sc[e] = (!ragged_tile || counts(slot)) ? raw[e] : -INFINITY;
  }
  if (ragged_tile) {
    uint32_t msk[4];
#pragma unroll
    for (int jw = 0; jw < 4; ++jw) {
      const int e0 = 2 * jw, e1 = 2 * jw + 1;
      const int sl0 = slot0 + (e0 >> 2) * 16 + (e0 & 3), sl1 = slot0 + (e1 >> 2) * 16 + (e1 & 3);
      msk[jw] = (counts(sl0) ? 0x0000ffffu : 0u) | (counts(sl1) ? 0xffff0000u : 0u);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      t.v[j].u.x &= msk[0]; t.v[j].u.y &= msk[1]; t.v[j].u.z &= msk[2]; t.v[j].u.w &= msk[3];
    }
  }
  softmax_pv(t, sc, st);
}

// N = 4 / 8 lanes of every 16 hold something in each of 16 / N registers: the first N lanes keep a, the next N get b's, and so on.
template <int N>
__device__ __forceinline__ floatx4 pack_lanes(const floatx4& a, const floatx4& b, const floatx4& c, const floatx4& d) {
  floatx4 p;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int x = __float_as_int(a[e]);
    if (N == 4) {
      x = __builtin_amdgcn_update_dpp(x, __float_as_int(b[e]), 0x114, 0xf, 0x2, false);      // row_shr:4, lanes 4 .. 7 of a row
      x = __builtin_amdgcn_update_dpp(x, __float_as_int(c[e]), 0x118, 0xf, 0x4, false);
      x = __builtin_amdgcn_update_dpp(x, __float_as_int(d[e]), 0x11c, 0xf, 0x8, false);
    } else {
      x = __builtin_amdgcn_update_dpp(x, __float_as_int(b[e]), 0x118, 0xf, 0xc, false);      // row_shr:8, lanes 8 .. 15
    }
    p[e] = __int_as_float(x);
  }
  return p;
}

// One tile of a head: full attention into st_full and, for a gated head (Eq. 1), the local
// attention into st_local when the tile touches the sink or the recent range.  The scores
// are computed once; the full update runs first because its V clearing (slots past the
// prefix) is a subset of the local one.
// `scored` runs between the scores and the weights: the tile's K registers are free from there on.
template <bool GATED, typename F>
__device__ __forceinline__ void process_tile(TileRegs& t, const Frag (&qb)[4], Softmax& st_full, Softmax& st_local,
                                             bool two_sets, int tile, int n_eff, float scale_log2, int kb, int keep_lo,
                                             int keep_from, F scored) {
  float raw[8];
  tile_scores(t, qb, scale_log2, raw);
  scored();
  tile_accumulate<false>(t, raw, st_full, tile, n_eff, kb);
  if (GATED && two_sets && (tile * kTile < keep_lo || tile * kTile + kTile > keep_from))
    tile_accumulate<true>(t, raw, st_local, tile, n_eff, kb, keep_lo, keep_from);
}

// (A launch whose `grow_known` is -1 - one whose growth only the device knows, or a recorded call, replayed under other lists - takes
// the growth from the list's header.)
// Bound: HBM; a launch over short contexts is a chain of latencies: record, first tile (a CU takes 64 bytes a clock: eight tiles are
// 2048), scores to products, merge.
template <bool FUSED, bool GATED, bool PAGED>
__global__ __launch_bounds__(kThreads, 1) void decode_mfma_kernel(const char* __restrict__ list, char* __restrict__ kv_base,
                                                                const uint16_t* __restrict__ q,
                                                                const uint16_t* __restrict__ k_new,
                                                                const uint16_t* __restrict__ v_new, uint32_t shape,
                                                                int grow_known, int window, int recent, DecodeRest r) {
  constexpr int kRow = kHeadDim + 4;                   // (the 16 heads of a store fall into different banks)
  __shared__ floatx4 sm_o[kWaves][kMaxGroup][kRow / 4];
  __shared__ float2 sm_ml[kMaxGroup][kWaves];
  __shared__ alignas(16) float sm_w[kMaxGroup][kMergeFew];     // (merge_duo reads four weights at a time)
  __shared__ LeftPair sm_left[2];                      // (in LDS only to spare registers)

  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of
  // shares so that its L2 and TLBs see one compact slice of the stores.
  const int n_wg = shape >> kShapeWgs;
  // (Not where half of the shares or more are empty: the others would sit on few XCDs.)
  const bool in_turn = (shape & kShapeInTurn) != 0;
  const int wg = (n_wg & 7) == 0 && !in_turn ? (blockIdx.x & 7) * (n_wg >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  WgDesc wd = load_wg(list, wg);
  // tokens since the list was planned: known to the host, or asked for beside the record
  int grow = grow_known;
  if (grow_known < 0) grow = load_const<int32_t>(list);
  // The other arguments: what the loads and scores need is asked for in the shadow of the record, the rest behind the loads
  // (late_args: left alone the compiler asks for all of it in front of them, and keeps it in lanes of vector registers).
  asm volatile("" : "+s"(r.scale_log2));
  if (FUSED) asm volatile("" : "+s"(r.recent_inverse));
  auto late_args = [] { return late_arguments<DecodeRest>(); };
  // (a generic pointer would make flat stores of them: with one in flight every wait for a load waits for all)
  typedef __attribute__((address_space(1))) uint16_t GlobalOut;
  typedef __attribute__((address_space(1))) int32_t GlobalInt;
  if (PAGED) asm volatile("" : "+s"(r.block_table), "+s"(r.page_bytes), "+s"(r.page_shift), "+s"(r.page_mask), "+s"(r.table_stride));

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int u_begin = wd.u_begin, u_end = wd.u_end;
  // (no workgroup of this launch reads the counter)
  const bool advance = FUSED && grow_known >= 0 && blockIdx.x == 0 && tid == 0;
  if (u_begin >= u_end) {
    if (advance) *reinterpret_cast<int32_t*>(const_cast<char*>(list)) = grow + 1;
    return;
  }
  int pi = wd.first_pair, b = wd.seq, h = wd.head;
  PairDesc pd = wd.first;
  int n_left = 0;
  uint32_t warm = 0;

  const int G = shape & kShapeGroup;
  auto emit = [&](GlobalOut* out, int pair, int g, int d4, const floatx4& v) {
    GlobalOut* dst = out + ((int64_t)pair * G + g) * kHeadDim + d4 * 4;
    const uint2 four = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
    if (((uintptr_t)out & 7) == 0) {                             // (a caller's may start at any element)
      *(__attribute__((address_space(1))) i32x2*)dst = i32x2{(int)four.x, (int)four.y};
    } else {
      dst[0] = (uint16_t)four.x;
      dst[1] = (uint16_t)(four.x >> 16);
      dst[2] = (uint16_t)four.y;
      dst[3] = (uint16_t)(four.y >> 16);
    }
  };
  const int hd = lane & 15;     // score layout: head; operand layouts: row / column
  const int kb = lane >> 4;     // k-group of the operand layouts; slot quad of the score layout

  for (int u = u_begin; u < u_end;) {
    // segment = the units [u, seg_end) of pair pi = tiles [tile_lo, tile_hi) of its store
    const int ps = pd.unit_start, pe = pd.unit_end;
    const int seg_end = u_end < pe ? u_end : pe;
    // the first unit(s) of a pair carry no tiles (they stand for its fixed cost)
    const int r_lo = u - ps > kPairOverheadUnits ? u - ps - kPairOverheadUnits : 0;
    const int r_hi = seg_end - ps > kPairOverheadUnits ? seg_end - ps - kPairOverheadUnits : 0;
    const int tile_lo = r_lo * kRound;
    const bool whole_pair = u == ps && seg_end == pe;
    const int n_old = pd.n_build + grow;
    const int n = FUSED ? n_old + 1 : n_old;
    const bool full = pd.ring < 0;
    const int n_eff = full ? n : (n < window ? n : window);
    TileMap<PAGED> store;
    store.base = kv_base + pd.koff;
    store.paged = PAGED && full;
    if (PAGED) {
      store.row = r.block_table + (int64_t)b * r.table_stride;
      store.page_bytes = r.page_bytes;
      store.shift = r.page_shift;
      store.mask = r.page_mask;
      store.last = r.table_stride - 1;
    }
    // the list was built with room to grow: tiles past the valid prefix are still empty
    const int tiles_valid = (n_eff + kTile - 1) / kTile;
    const int tile_hi = r_hi * kRound < tiles_valid ? r_hi * kRound : tiles_valid;
    int tile = tile_lo + wave;

    // This step's append: position n_old goes to slot_new (sink / ring / next row of a full head).  The wavefront that will read the
    // tile with the new slot writes the row (`mine`): its loads go out first, its stores behind the first tile's loads.
    const int sink = window - recent;
    int slot_new = 0, tile_new = 0;
    bool mine = false;
    if (FUSED) {
      slot_new = (full || n_old < sink) ? n_old : sink + remainder_of(n_old - sink, recent, r.recent_inverse);
      tile_new = slot_new >> 5;
      mine = tile_new >= tile_lo && tile_new < tile_hi && ((tile_new - tile_lo) & (kWaves - 1)) == wave;
    }
    // the next pair's record, for the (rare) share that crosses a pair boundary
    PairDesc pd_next = pd;
    auto fetch_next = [&]() { if (seg_end < u_end) pd_next = load_pair(list + late_args()->pair_off, pi + 1); };
    // Eq. 1 gate: a full head with gate < 1 also accumulates its local attention (sink + recent
    // positions) over the same tiles; out = gate * full + (1 - gate) * local.
    const bool two_sets = GATED && full && pd.gate < 1.f;
    const int keep_lo = sink, keep_from = n - recent;                 // local: slot < S or slot >= n - R
    Softmax st[GATED ? 2 : 1];
#pragma unroll
    for (int k = 0; k < (GATED ? 2 : 1); ++k) {
      st[k].m = -INFINITY;
      st[k].l = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) st[k].o[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    if (tile < tile_hi) {
      uint4 kn[4];
      uint32_t vn[8];
      if (FUSED && mine) {
        // K: the lanes that hold row slot % 16 need it; V: the lanes that hold this slot's k-group
        const int64_t src = (int64_t)pi * kHeadDim;
#pragma unroll
        for (int s = 0; s < 4; ++s) kn[s] = *reinterpret_cast<const uint4*>(k_new + src + (s * 4 + kb) * 8);
#pragma unroll
        for (int j = 0; j < 8; ++j) vn[j] = v_new[src + j * 16 + hd];
      }

      // Q as the B operand of the score MFMA: column = head, k-group kb, step s (columns past the group repeat its last head;
      // nobody reads them)
      Frag qb[4];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        qb[s].u = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(q) +
                                                  (((int64_t)pi * G + (hd < G ? hd : G - 1)) * kHeadDim + s * 32 + kb * 8) * 2);
      // each wavefront keeps one tile in flight behind the one it is working on
      TileRegs ra;
      load_tile(ra, store.at(tile), lane);
      // address of the tile after this one, looked up one iteration ahead
      const char* next_base = store.at(tile + kWaves);
      fetch_next();
      // The record this workgroup will start the next layer's launch with: asked for now, so that it is in
      // L2 by then (its record is the first thing a workgroup waits for).  Looked at only at the very end.
      if (u == u_begin && (shape & kShapeMore) && wave == 0)
        warm = *reinterpret_cast<const uint32_t*>(list + late_args()->list_stride + sizeof(ListHeader) + (int64_t)wg * (int)sizeof(WgDesc));

      if (FUSED && mine) {
        // The row goes into the store, every 16-byte unit by the lane that later loads it (so program order makes later loads see
        // it), and, where the tile is the one that has just been asked for, into its registers: a load behind the stores would
        // be another memory latency for the wavefront the workgroup waits for at the merge.
        const int st = slot_new & 31, hf = st >> 4, e = hf * 4 + (st & 3);
        const bool k_lane = hd == (st & 15), v_lane = kb == ((st & 15) >> 2);
        if (tile == tile_new) {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const uint32_t m = k_lane && hf == half ? 0xffffffffu : 0u;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              uint4& u4 = ra.k[half][s].u;
              u4.x = (kn[s].x & m) | (u4.x & ~m); u4.y = (kn[s].y & m) | (u4.y & ~m);
              u4.z = (kn[s].z & m) | (u4.z & ~m); u4.w = (kn[s].w & m) | (u4.w & ~m);
            }
          }
          uint32_t m[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) m[w] = v_lane && (e >> 1) == w ? ((e & 1) ? 0xffff0000u : 0xffffu) : 0u;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint32_t two = vn[j] | (vn[j] << 16);
            uint4& u4 = ra.v[j].u;
            u4.x = (two & m[0]) | (u4.x & ~m[0]); u4.y = (two & m[1]) | (u4.y & ~m[1]);
            u4.z = (two & m[2]) | (u4.z & ~m[2]); u4.w = (two & m[3]) | (u4.w & ~m[3]);
          }
        }
        char* tile_base = store.at(tile_new);
        if (k_lane) {
#pragma unroll
          for (int s = 0; s < 4; ++s) *reinterpret_cast<uint4*>(tile_base + hf * 4096 + s * 1024 + lane * 16) = kn[s];
        }
        if (v_lane) {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            *reinterpret_cast<uint16_t*>(tile_base + 8192 + j * 1024 + lane * 16 + e * 2) = (uint16_t)vn[j];
        }
        bool wide = false;                       // the fp16 range test, for prefill
#pragma unroll
        for (int j = 0; j < 8; ++j) wide |= bf16_beyond_fp16(vn[j]);
        auto* late = late_args();
        if (wide) *(GlobalInt*)late->v_wide = 1;
        if (lane == 0 && !full) ((GlobalInt*)late->slot_pos)[((int64_t)pd.ring * late->batch + b) * window + slot_new] = n_old;
      }

      // One image, refilled as it is used up: K behind the scores, V behind the products.  Every wait is for its own registers only, the
      // refills behind them in flight.
      for (; tile + kWaves < tile_hi; tile += kWaves) {
        const char* refill = next_base;
        next_base = store.at(tile + 2 * kWaves);
        process_tile<GATED>(ra, qb, st[0], st[GATED ? 1 : 0], two_sets, tile, n_eff, r.scale_log2, kb, keep_lo, keep_from,
                            [&] { load_tile_k(ra, refill, lane); });
        load_tile_v(ra, refill, lane);
      }
      process_tile<GATED>(ra, qb, st[0], st[GATED ? 1 : 0], two_sets, tile, n_eff, r.scale_log2, kb, keep_lo, keep_from, [] {});
    } else {
      fetch_next();
    }

    // Merge of the wavefronts: four outputs of a head per thread.  The accumulators are packed first, so that a store to LDS is of
    // 64 lanes where the group is small (of 4 heads, 16 lanes hold a head: eight stores a wavefront, 16 clocks each and more
    // whatever the lanes, were 1150 clocks of the merge).
    constexpr int kPasses = kMaxGroup * kHeadDim / 4 / kThreads;
    floatx4 held[kPasses];                                             // full-attention results of a whole pair
    // (What the merge computes from the thread's number and reads of the arguments stays behind the loads: the compiler would place it
    // before the loop, in front of the first of them.)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int hd = tid & 15, kb = (tid >> 4) & 3;
    auto* late = late_args();
    const Partials part = partials_at(late->part);
    GlobalOut* out = (GlobalOut*)late->out;
#pragma unroll
    for (int set = 0; set < (GATED ? 2 : 1); ++set) {
      if (set == 1 && !two_sets) break;
      const Softmax& ss = st[set];
      const TwoValues l16 = swap16(ss.l);
      const TwoValues l32 = swap32(l16.a + l16.b);

      if (u != u_begin || set > 0) __syncthreads();   // the previous merge has finished reading LDS
      if (set == 0 && tid == 0 && !whole_pair) sm_left[n_left] = LeftPair{pi, pd.wg_first, pd.n_seg, two_sets ? pd.gate : 1.f};
      if (kb == 0) sm_ml[hd][wave] = make_float2(ss.m, l32.a + l32.b);
      if (G <= 4) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          sm_o[wave][hd & 3][(t * 4 + (hd >> 2)) * 4 + kb] = pack_lanes<4>(ss.o[t * 4], ss.o[t * 4 + 1], ss.o[t * 4 + 2], ss.o[t * 4 + 3]);
      } else if (G <= 8) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          sm_o[wave][hd & 7][(t * 2 + (hd >> 3)) * 4 + kb] = pack_lanes<8>(ss.o[t * 2], ss.o[t * 2 + 1], ss.o[t * 2], ss.o[t * 2]);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) sm_o[wave][hd][j * 4 + kb] = ss.o[j];
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < kPasses; ++it) {
        const int idx = tid + it * kThreads, g = idx >> 5, d4 = idx & 31;
        if (g >= G) break;
        float2 ml[kWaves];
        floatx4 o[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) ml[w] = sm_ml[g][w];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) o[w] = sm_o[w][g][d4];
        float M = ml[0].x;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) M = fmaxf(M, ml[w].x);
        floatx4 O = floatx4{0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const float sc = exp2_or_zero(ml[w].x, M);
          O += sc * o[w];
          L += sc * ml[w].y;
        }
        if (whole_pair) {
          floatx4 res = quotients(O, L);
          if (two_sets) {
            if (set == 0) { held[it] = res; continue; }
            res = pd.gate * held[it] + (1.f - pd.gate) * res;
          }
          emit(out, pi, g, d4, res);
        } else {
          leave_partial(part, set, wg + pi, G, g, d4, O, M, L);
        }
      }
    }
    if (!whole_pair && part.arrived) ++n_left;
    // whoever owns tile 0 of head 0 publishes the new length, in both copies of the table (nobody reads either during this launch)
    if (FUSED && h == 0 && tile_lo == 0 && tid == 0) {
      ((GlobalInt*)late->len0)[b] = n;
      ((GlobalInt*)late->len1)[b] = n;
    }
    u = seg_end;
    auto step_on = [&]() { ++pi; if (++h == late->n_kv_heads) { h = 0; ++b; } };
    step_on();
    pd = pd_next;
    if (u < u_end)
      while (pd.unit_end <= u) { step_on(); pd = load_pair(list + late->pair_off, pi); }       // pairs of inactive slots own no units
  }
  if (n_left > 0) {
    auto* late = late_args();
    finish_pairs<kThreads, GATED>(partials_at(late->part), sm_left, n_left, G, sm_w,
                                  [&](int pair, int g, int d4, const floatx4& v) { emit((GlobalOut*)late->out, pair, g, d4, v); });
  }
  if (advance) *reinterpret_cast<int32_t*>(const_cast<char*>(list)) = grow + 1;
  asm volatile("" ::"v"(warm));                        // keeps the load above alive
}

}  // namespace

hipError_t launch_decode_mfma(const DeviceView& dv, int layer, bool gated, const void* q, void* out, float scale_log2,
                              const void* k_new, const void* v_new, int grow, bool merge_here, bool in_turn, hipStream_t stream,
                              hipEvent_t ev_start, hipEvent_t ev_stop) {
  const dim3 grid(dv.n_wg);
  const char* list = dv.list_base + layer * dv.list_stride;
  const uint32_t shape = (uint32_t)dv.group | (in_turn ? kShapeInTurn : 0u) | (layer + 1 < dv.n_layers ? kShapeMore : 0u) |
                         ((uint32_t)dv.n_wg << kShapeWgs);
  DecodeRest r = {};
  r.out = (uint16_t*)out; r.scale_log2 = scale_log2; r.n_kv_heads = dv.n_kv_heads;
  r.pair_off = dv.list_pair_off; r.batch = dv.batch; r.list_stride = dv.list_stride;
  r.part = {dv.part_o, dv.part_m, dv.part_l, dv.part_set_o, dv.part_set_ml, merge_here ? dv.arrived + (int64_t)layer * dv.n_pairs * (kMaxGroup / 2) : nullptr};
  r.len0 = len_of(dv, 0, layer); r.len1 = len_of(dv, 1, layer);
  r.slot_pos = dv.slot_pos; r.v_wide = dv.v_wide + layer;
  r.block_table = dv.block_table; r.page_bytes = dv.page_bytes; r.page_shift = dv.page_shift; r.page_mask = dv.page_mask;
  r.table_stride = dv.table_stride;
  r.recent_inverse = inverse_of(dv.recent);
  // (the plain launch when no timestamps are asked for: that form can be recorded into a graph)
#define RLKV_LAUNCH(F, GT, PG)                                                                                    \
  do {                                                                                                            \
    static_assert(late_arguments_are_last<decltype(&decode_mfma_kernel<F, GT, PG>), DecodeRest>());               \
    if (ev_start || ev_stop)                                                                                      \
      hipExtLaunchKernelGGL((decode_mfma_kernel<F, GT, PG>), grid, dim3(kThreads), 0, stream, ev_start, ev_stop, 0, \
                            list, dv.kv_base, (const uint16_t*)q, (const uint16_t*)k_new, (const uint16_t*)v_new, \
                            shape, grow, dv.window, dv.recent, r);                                                \
    else                                                                                                          \
      hipLaunchKernelGGL((decode_mfma_kernel<F, GT, PG>), grid, dim3(kThreads), 0, stream, list, dv.kv_base,      \
                         (const uint16_t*)q, (const uint16_t*)k_new, (const uint16_t*)v_new, shape, grow,         \
                         dv.window, dv.recent, r);                                                                \
  } while (0)
#define RLKV_PICK(F, GT) do { if (dv.page_shift >= 0) RLKV_LAUNCH(F, GT, true); else RLKV_LAUNCH(F, GT, false); } while (0)
  if (k_new) { if (gated) RLKV_PICK(true, true); else RLKV_PICK(true, false); }
  else       { if (gated) RLKV_PICK(false, true); else RLKV_PICK(false, false); }
#undef RLKV_PICK
#undef RLKV_LAUNCH
  return hipGetLastError();
}

}  // namespace rlkv
