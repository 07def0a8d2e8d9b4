// Split-K decode attention, MFMA variant (tiled bf16 stores).
//
// Same operation as the vector-ALU variant (softmax attention of the G query heads of a
// group over the rows a store holds; paper Sec. 3.1 Eq. 1 at gate 0/1, Sec. 3.3), with the
// two contractions on the matrix cores:
//   scores  S[slot][head] = sum_d K[slot][d] * Q[head][d]   v_mfma_f32_16x16x32_bf16,
//                           A = K tile (16 slots x 32 d), B = Q^T (heads padded to 16)
//   output  O[head][d]    = sum_slot P[head][slot] * V[slot][d]   same instruction,
//                           A = V^T tile (k runs over the 32 slots of a tile), B = P^T
// The score accumulator leaves lane l holding head l%16 and slots 4*(l/16)..+3 of each
// 16-slot half, which is exactly the B-operand register layout, so P never moves between
// lanes; O comes out as O^T, each head in the lanes that hold its scores.  The stores are laid out (see rlkv_internal.h) so that every 128-bit load per lane
// is one contiguous kilobyte per wavefront and lands directly in operand registers: no
// LDS staging, no transposes, and the wavefronts of a workgroup run independently until
// the merge.  P is split into a bf16 head and a bf16 remainder (two MFMAs per V block) so
// the weights carry ~16 mantissa bits; the matrix cores are idle most of the time anyway.
//
// At its start a workgroup learns its share and its first store from one wave-uniform record and issues the loads of Q, and
// then of its first tile (four wavefronts, plain: once Q has arrived; the fused forms: once the new row is in the store).
// Each wavefront keeps one tile (16 KiB) in flight behind the one it works on; with one
// workgroup per CU that is 64 KiB in flight per CU, which measurement shows is where this
// part's HBM streams best (more in flight lowers the achieved bandwidth).
//
// Gated heads (GATED = true; paper Sec. 3.1, Eq. 1): a full head with gate g < 1 returns
// g * full + (1 - g) * local attention.  The local positions (first S, last R) are a subset of
// the full ones, so the same pass keeps a second accumulator that only the tiles touching
// those ranges update; the scores of a tile are computed once for both.
//
// Fused single-token append (FUSED = true): the kernel also performs this step's append.
// Every sequence grows by one position; the wavefront that owns the tile holding the new
// slot of a pair writes the new K/V row into the store (sink slot, ring slot - evicting
// position p - R - or next row of a full head) before it loads that tile; each lane writes
// exactly the bytes it later loads, so no other wavefront ever depends on the write.  No
// workgroup reads a length from the table: a pair's length is its length when the work list was
// planned plus the list's growth counter (ListHeader::grow), which no workgroup writes while another
// one reads it, so the kernel needs no grid-wide fence: under a list of shares every workgroup reads
// the counter and the merge kernel that follows advances it - no per-step argument, and a captured
// launch can be replayed; under a list of whole pairs, which has no merge kernel, the count comes as an
// argument, nobody reads the counter, and the first workgroup writes it.  The new lengths are written
// to both copies of the length table for the kernels that do read it.
#include "mfma_tile.h"

namespace rlkv {
namespace {

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

// The gated variant carries two accumulator sets: it is built for one wavefront per SIMD (the
// configuration the library launches), which leaves it 512 registers.
//
// WAVES = 8 (kWholeWaves): the form for lists of whole pairs (share_plan.hip), two wavefronts per SIMD.  A launch whose
// `grow` is -1 (one whose growth only the device knows, or a recorded decode call, replayed under other lists) takes the growth from
// the list's header, and if the list is not of whole pairs, the upper four wavefronts have no tiles and every pair is worked as the
// four-wavefront form does, to the bit.
// Bound: a whole-pair launch is a chain of latencies (record, first tiles, merge, store) plus its longest pair at what
// one CU can draw.  Decode call of 1 / 8 / 32 sequences of 300 tokens, 32 query and 8 KV heads: 7.4 / 7.4 / 8.3 us against
// 10.6 / 10.5 / 10.7 us of shares and merge launch; 32 of 1500 tokens: 21.9 against 23.9 us.  (Four wavefronts with a tile
// in flight behind the one in work need 450 registers; two per SIMD cover each other instead.)
template <bool FUSED, bool GATED, bool PAGED, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void decode_mfma_kernel(DeviceView dv, int layer,
                                                                const uint16_t* __restrict__ q,
                                                                uint16_t* __restrict__ out, float scale_log2,
                                                                const uint16_t* __restrict__ k_new,
                                                                const uint16_t* __restrict__ v_new, int grow_known,
                                                                int in_turn) {
  constexpr int kRow = kHeadDim + 4;                   // (the 16 heads of a store fall into different banks)
  __shared__ floatx4 sm_o[WAVES][kMaxGroup][kRow / 4];
  __shared__ float sm_m[WAVES][kMaxGroup];
  __shared__ float sm_l[WAVES][kMaxGroup];
  constexpr int kThreads = WAVES * 64;

  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of
  // shares so that its L2 and TLBs see one compact slice of the stores.
  const int n_wg = gridDim.x;
  // (Not where half of the shares or more are empty, `in_turn`: the others would sit on few XCDs.)
  const int wg = (n_wg & 7) == 0 && !in_turn ? (blockIdx.x & 7) * (n_wg >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  const WgDesc* __restrict__ wdp = wg_desc_of(dv, layer) + wg;
  // tokens since the list was planned: asked for beside the record, or (eight wavefronts) known to the host
  int grow = grow_known, stride = WAVES;               // stride: wavefronts that share a segment's tiles
  if (WAVES == kRound) {
    grow = list_header(dv, layer)->grow;
  } else if (grow_known < 0) {
    grow = list_header(dv, layer)->grow;
    if (!list_header(dv, layer)->whole) stride = kRound;
  } else if (FUSED && blockIdx.x == 0 && threadIdx.x == 0) {
    list_header(dv, layer)->grow = grow + 1;           // (no workgroup of this launch reads it)
  }
  const int u_begin = wdp->u_begin, u_end = wdp->u_end;
  // The record this workgroup will start the next layer's launch with: asked for now, so that it is in
  // L2 by then (its record is the first thing a workgroup waits for).  Looked at only at the very end.
  uint32_t warm = 0;
  if (threadIdx.x == 0 && layer + 1 < dv.n_layers)
    warm = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(wdp) + dv.list_stride);
  if (u_begin >= u_end) return;
  int pi = wdp->first_pair;
  PairDesc pd = wdp->first;
  const PairDesc* __restrict__ pairs = pair_desc_of(dv, layer);

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int hd = lane & 15;     // score layout: head; operand layouts: row / column
  const int kb = lane >> 4;     // k-group of the operand layouts; slot quad of the score layout
  const int G = dv.group;

  for (int u = u_begin; u < u_end;) {
    // segment = the units [u, seg_end) of pair pi = tiles [tile_lo, tile_hi) of its store
    const int ps = pd.unit_start, pe = pd.unit_end;
    const int seg_end = u_end < pe ? u_end : pe;
    // the first unit(s) of a pair carry no tiles (they stand for its fixed cost)
    const int r_lo = u - ps > kPairOverheadUnits ? u - ps - kPairOverheadUnits : 0;
    const int r_hi = seg_end - ps > kPairOverheadUnits ? seg_end - ps - kPairOverheadUnits : 0;
    const int tile_lo = r_lo * kRound;
    const bool whole_pair = u == ps && seg_end == pe;
    const int b = pi / dv.n_kv_heads, h = pi % dv.n_kv_heads;
    const int n_old = pd.n_build + grow;
    const int n = FUSED ? n_old + 1 : n_old;
    const bool full = pd.full != 0;
    const int n_eff = full ? n : (n < dv.window ? n : dv.window);
    TileMap<PAGED> store;
    store.base = dv.kv_base + pd.koff;
    store.paged = PAGED && full;
    if (PAGED) {
      store.row = dv.block_table + (int64_t)b * dv.table_stride;
      store.page_bytes = dv.page_bytes;
      store.shift = dv.page_shift;
      store.mask = dv.page_mask;
      store.last = dv.table_stride - 1;
    }
    // the list was built with room to grow: tiles past the valid prefix are still empty
    const int tiles_valid = (n_eff + kTile - 1) / kTile;
    const int tile_hi = r_hi * kRound < tiles_valid ? r_hi * kRound : tiles_valid;

    if (FUSED) {
      // whoever owns tile 0 of head 0 publishes the new length, in both copies of the table (nobody reads
      // either during this launch)
      if (h == 0 && tile_lo == 0 && tid == 0) { len_of(dv, 0, layer)[b] = n; len_of(dv, 1, layer)[b] = n; }
      // position n_old goes to slot_new (sink / ring / next row of a full head)
      const int slot_new = (full || n_old < dv.sink) ? n_old : dv.sink + (n_old - dv.sink) % dv.recent;
      const int tile_new = slot_new >> 5;
      if (tile_new >= tile_lo && tile_new < tile_hi && ((tile_new - tile_lo) & (stride - 1)) == wave) {
        // This wavefront will read the tile that holds the new slot: it writes the row first.
        // Every 16-byte unit below is written by the lane that later loads it, so program
        // order makes the loads see the new row.
        const int st = slot_new & 31, hf = st >> 4;
        char* tile_base = store.at(tile_new);
        const int64_t src = ((int64_t)b * dv.n_kv_heads + h) * kHeadDim;
        // (all loads of the new row first, then the stores: one memory latency instead of two in a row
        // for the one wavefront per pair that does this, and whose workgroup waits for it at the merge)
        const bool k_lane = hd == (st & 15);            // K: the lanes that hold row slot % 16
        const bool v_lane = kb == ((st & 15) >> 2);     // V: the lanes that hold this slot's k-group
        uint4 kn[4];
        uint16_t vn[8];
#pragma unroll
        for (int s = 0; s < 4; ++s)
          kn[s] = k_lane ? *reinterpret_cast<const uint4*>(k_new + src + (s * 4 + kb) * 8) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) vn[j] = v_lane ? v_new[src + j * 16 + hd] : (uint16_t)0;
        if (k_lane) {
#pragma unroll
          for (int s = 0; s < 4; ++s) *reinterpret_cast<uint4*>(tile_base + hf * 4096 + s * 1024 + lane * 16) = kn[s];
        }
        if (v_lane) {
          const int e = hf * 4 + (st & 3);
#pragma unroll
          for (int j = 0; j < 8; ++j)
            *reinterpret_cast<uint16_t*>(tile_base + 8192 + j * 1024 + lane * 16 + e * 2) = vn[j];
        }
        if (WAVES > kRound) {
          // (no merge kernel follows a list of whole pairs: the fp16 range test is made here; in the four-wavefront
          // form it cost the launch 2 us)
          bool wide = false;
#pragma unroll
          for (int j = 0; j < 8; ++j) wide |= bf16_beyond_fp16(vn[j]);
          if (wide) dv.v_wide[layer] = 1;
        }
        if (lane == 0 && !full)
          dv.slot_pos[dv.slotpos_off[layer * dv.n_kv_heads + h] + (int64_t)b * dv.window + slot_new] = n_old;
      }
    }

    // Q as the B operand of the score MFMA: column = head, k-group kb, step s
    Frag qb[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (hd < G) {
        const int64_t qrow = (int64_t)b * dv.n_q_heads + h * G + hd;
        qb[s].u = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(q) +
                                                  (qrow * kHeadDim + s * 32 + kb * 8) * 2);
      } else {
        qb[s].u = make_uint4(0, 0, 0, 0);
      }
    }
    // each wavefront keeps one tile in flight behind the one it is working on
    int tile = WAVES > kRound && wave >= stride ? tile_hi : tile_lo + wave;
    TileRegs ra, rb;
    if (tile < tile_hi) load_tile(ra, store.at(tile), lane);
    // address of the tile after this one, looked up one iteration ahead.  (Paged: the compiled loop reads the table entry through
    // a vector load and waits for it, and with it for every load before it, at the lookup.)
    const char* next_base = store.at(tile + stride);
    // the next pair's record, for the (rare) share that crosses a pair boundary
    PairDesc pd_next = pd;
    // (the compiler moves it to scalar registers here, which waits for the loads before it, the first tile's included)
    if (seg_end < u_end) pd_next = pairs[pi + 1];

    // Eq. 1 gate: a full head with gate < 1 also accumulates its local attention (sink + recent
    // positions) over the same tiles; out = gate * full + (1 - gate) * local.
    const bool two_sets = GATED && full && pd.gate < 1.f;
    const int keep_lo = dv.sink, keep_from = n - dv.recent;          // local: slot < S or slot >= n - R
    Softmax st[GATED ? 2 : 1];
#pragma unroll
    for (int k = 0; k < (GATED ? 2 : 1); ++k) {
      st[k].m = -INFINITY;
      st[k].l = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) st[k].o[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // Two register images that swap roles, and the last tile of the segment outside the steady state: inside it the loads of the
    // next tile are unconditional.  As compiled, the second half of the loop waits for its own tile only, the next tile's 16 loads in
    // flight beside it (`vmcnt(16)`); between the second half and the first the image is copied from one set of registers
    // to the other with 8 loads left, and the next tile is asked for with 2 left (fused: 0), since its addresses take registers
    // that loads still fill.  (With one loop and a conditional load every half waited for all loads, the next tile's included.)
    auto work = [&](TileRegs& t, int tl) {
      process_tile<GATED>(t, qb, st[0], st[GATED ? 1 : 0], two_sets, tl, n_eff, scale_log2, kb, keep_lo, keep_from,
                          [] {});
    };
    if constexpr (WAVES > kRound || GATED || PAGED) {
      // One image, refilled as it is used up - K behind the scores, V behind the products: half the registers, which
      // eight wavefronts and two accumulator sets need, and faster where the next tile's address comes out of a table.
      // (Gated, 16 sequences of 3000 .. 5000 tokens: 30.8 us against 32.2 with a copy per tile from the image in flight,
      // 63 with two images; paged, 24 of 2000 .. 20 000: 46.9 against 51.4 us with two images.  Contiguous stores: the
      // same for a plain launch, a 28-layer fused step 1170 against 1165 us.)  As compiled, all of these loops but the fused one
      // that blends wait for V too before the scores, which need K only.
      for (; tile + stride < tile_hi; tile += stride) {
        const char* refill = next_base;
        next_base = store.at(tile + 2 * stride);
        process_tile<GATED>(ra, qb, st[0], st[GATED ? 1 : 0], two_sets, tile, n_eff, scale_log2, kb, keep_lo, keep_from,
                            [&] { load_tile_k(ra, refill, lane); });
        load_tile_v(ra, refill, lane);
      }
      if (tile < tile_hi) work(ra, tile);
    } else
    for (;;) {
      if (tile + stride >= tile_hi) {
        if (tile < tile_hi) work(ra, tile);
        break;
      }
      load_tile(rb, next_base, lane);
      next_base = store.at(tile + 2 * stride);
      work(ra, tile);
      tile += stride;
      if (tile + stride >= tile_hi) {
        work(rb, tile);
        break;
      }
      load_tile(ra, next_base, lane);
      next_base = store.at(tile + 2 * stride);
      work(rb, tile);
      tile += stride;
    }

    // Merge of the wavefronts: four outputs of a head per thread, so that all of a group of 8 heads are one pass of 256 threads.
    // (With one output per thread and pass, and O instead of O^T in the accumulators - four times the LDS stores here, shuffles in every
    // rescaling - a 28-layer step of 16 x 16 384 tokens took 1187 us, now 1153; blending heads, 16 x 3000 .. 5000, 31.1 us, now 28.7;
    // 24 paged sequences of 2000 .. 20 000 47.1, now 46.6; 32 of 4000 .. 32 000 185, now 185.)
    constexpr int kPasses = kMaxGroup * kHeadDim / 4 / kThreads;
    floatx4 held[kPasses];                                             // full-attention results of a whole pair
#pragma unroll
    for (int set = 0; set < (GATED ? 2 : 1); ++set) {
      if (set == 1 && !two_sets) break;
      const Softmax& ss = st[set];
      const TwoValues l16 = swap16(ss.l);
      const TwoValues l32 = swap32(l16.a + l16.b);

      __syncthreads();   // the previous merge has finished reading LDS
      if (hd < G) {
        if (kb == 0) { sm_m[wave][hd] = ss.m; sm_l[wave][hd] = l32.a + l32.b; }
#pragma unroll
        for (int j = 0; j < 8; ++j) sm_o[wave][hd][j * 4 + kb] = ss.o[j];
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < kPasses; ++it) {
        const int idx = tid + it * kThreads, g = idx >> 5, d4 = idx & 31;
        if (g >= G) break;
        float M = sm_m[0][g];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sm_m[w][g]);
        floatx4 O = floatx4{0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
          const float sc = exp2_or_zero(sm_m[w][g], M);
          O += sc * sm_o[w][g][d4];
          L += sc * sm_l[w][g];
        }
        if (whole_pair) {
          floatx4 res = O / L;
          if (two_sets) {
            if (set == 0) { held[it] = res; continue; }
            res = pd.gate * held[it] + (1.f - pd.gate) * res;
          }
          uint16_t* dst = out + ((int64_t)b * dv.n_q_heads + h * G + g) * kHeadDim + d4 * 4;
          const uint2 four = make_uint2(bf16_pair(res[0], res[1]), bf16_pair(res[2], res[3]));
          if ((reinterpret_cast<uintptr_t>(out) & 7) == 0) {            // (a caller's may start at any element)
            *reinterpret_cast<uint2*>(dst) = four;
          } else {
            dst[0] = (uint16_t)four.x;
            dst[1] = (uint16_t)(four.x >> 16);
            dst[2] = (uint16_t)four.y;
            dst[3] = (uint16_t)(four.y >> 16);
          }
        } else {
          const int64_t slot = (int64_t)wg + pi;
          *reinterpret_cast<floatx4*>(dv.part_o + set * dv.part_set_o + (slot * G + g) * kHeadDim + d4 * 4) = O;
          if (d4 == 0) {
            dv.part_m[set * dv.part_set_ml + slot * G + g] = M;
            dv.part_l[set * dv.part_set_ml + slot * G + g] = L;
          }
        }
      }
    }
    u = seg_end;
    ++pi;
    pd = pd_next;
    if (u < u_end)
      while (pd.unit_end <= u) pd = pairs[++pi];       // pairs of inactive slots own no units
  }
  asm volatile("" ::"v"(warm));                        // keeps the load above alive
}

}  // namespace

hipError_t launch_decode_mfma(const DeviceView& dv, int layer, bool gated, const void* q, void* out, float scale_log2,
                              const void* k_new, const void* v_new, bool whole, int grow, bool few, hipStream_t stream,
                              hipEvent_t ev_start, hipEvent_t ev_stop) {
  const dim3 grid(dv.n_wg);
  // (the plain launch when no timestamps are asked for: that form can be recorded into a graph)
#define RLKV_LAUNCH(F, GT, PG, W)                                                                                 \
  do {                                                                                                            \
    const dim3 block(W * 64);                                                                                     \
    if (ev_start || ev_stop)                                                                                      \
      hipExtLaunchKernelGGL((decode_mfma_kernel<F, GT, PG, W>), grid, block, 0, stream, ev_start, ev_stop, 0, dv, \
                            layer, (const uint16_t*)q, (uint16_t*)out, scale_log2, (const uint16_t*)k_new,       \
                            (const uint16_t*)v_new, grow, (int)(few && !whole));                                  \
    else                                                                                                          \
      hipLaunchKernelGGL((decode_mfma_kernel<F, GT, PG, W>), grid, block, 0, stream, dv, layer,                   \
                         (const uint16_t*)q, (uint16_t*)out, scale_log2, (const uint16_t*)k_new,                  \
                         (const uint16_t*)v_new, grow, (int)(few && !whole));                                     \
  } while (0)
#define RLKV_WAVES(F, GT, PG) do { if (whole) RLKV_LAUNCH(F, GT, PG, kWholeWaves); else RLKV_LAUNCH(F, GT, PG, kRound); } while (0)
#define RLKV_PICK(F, GT) do { if (dv.page_shift >= 0) RLKV_WAVES(F, GT, true); else RLKV_WAVES(F, GT, false); } while (0)
  if (k_new) { if (gated) RLKV_PICK(true, true); else RLKV_PICK(true, false); }
  else       { if (gated) RLKV_PICK(false, true); else RLKV_PICK(false, false); }
#undef RLKV_PICK
#undef RLKV_WAVES
#undef RLKV_LAUNCH
  return hipGetLastError();
}

}  // namespace rlkv
