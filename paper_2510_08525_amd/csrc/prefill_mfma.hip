// Prefill (chunked prefill) attention for mixed heads, MFMA variant (tiled bf16 stores).
//
// One chunk of T new positions per sequence attends over the positions already cached plus the
// chunk itself, under the two masks of paper Sec. 3.1 (App. B: prefilling applies them as mask
// matrices): a full head uses the causal mask, j <= i; a compressed head the local mask,
// j <= i and (j < S or i - j < R).  Here nothing is materialised: a query block walks only the
// tiles its mask rows can touch and masks inside the tile.
//
// Keys and values come from two places, both in the tiled MFMA-operand layout:
//   - the store.  Of a full head it holds every position, the chunk's own included: place_chunk_kernel
//     appends them first.  Of a compressed head it holds positions before the chunk: the sink slots and,
//     while the chunk's first R queries still reach back, the ring slots, whose positions are read from
//     the slot table;
//   - of a compressed head, a staging buffer with the chunk's own K/V, tiled by place_chunk_kernel.  Its
//     ring cannot hold a chunk longer than R, and early queries of the chunk need keys that later ones
//     evict, so the chunk is attended from the staging buffer and appended afterwards.
//
// Work split and the two loops of a wavefront: see the comment on prefill_mfma_kernel below.
// Scores use the same instruction and operand layouts as the decode kernel; a column of the score
// tile is a (position, head) pair instead of a head.  For the weights x V product the hot loop sends
// both operands to the matrix cores as fp16 (V converted on its way into LDS, exact for magnitudes in
// [2^-14, 65536), at most 2^-24 absolute below; tiles with larger values are taken as bf16); the
// general loop keeps the decode kernel's two-part bf16 weights.
#include <type_traits>

#include "mfma_tile.h"
#include "prefill_deal.h"
#include "tile_rows.h"

namespace rlkv {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Tiles re-read by many query blocks: ordinary (cached) loads.
__device__ __forceinline__ void load_k_cached(TileRegs& r, const char* tile_base, int lane) {
  const char* kb = tile_base + lane * 16;
#pragma unroll
  for (int hf = 0; hf < 2; ++hf)
#pragma unroll
    for (int s = 0; s < 4; ++s) r.k[hf][s].u = *reinterpret_cast<const uint4*>(kb + hf * 4096 + s * 1024);
}
__device__ __forceinline__ void load_v_cached(TileRegs& r, const char* tile_base, int lane) {
  const char* vb = tile_base + 8192 + lane * 16;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.v[j].u = *reinterpret_cast<const uint4*>(vb + j * 1024);
}

// Scores of one 32-slot tile against one group's Q operands, unscaled.
__device__ __forceinline__ void raw_scores(const TileRegs& t, const Frag (&qb)[4], float (&raw)[8]) {
  floatx4 s0 = floatx4{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.k[0][s].v, qb[s].v, s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.k[1][s].v, qb[s].v, s1, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) raw[e] = e < 4 ? s0[e] : s1[e - 4];
}

// Eight fp32 weights as two bf16 operands: the head keeps the top 16 bits of each weight
// (truncated, one byte permute per pair), the remainder p - head is exact in fp32 and is rounded
// to bf16; together they carry ~16 mantissa bits.
__device__ __forceinline__ void split_weights(const float (&p)[8], Frag& hi, Frag& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t b0 = __float_as_uint(p[2 * k]), b1 = __float_as_uint(p[2 * k + 1]);
    h[k] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);            // {b1.hi16, b0.hi16}
    const float r0 = p[2 * k] - __uint_as_float(b0 & 0xffff0000u);
    const float r1 = p[2 * k + 1] - __uint_as_float(b1 & 0xffff0000u);
    l[k] = bf16_pair(r0, r1);
  }
  hi.u = make_uint4(h[0], h[1], h[2], h[3]);
  lo.u = make_uint4(l[0], l[1], l[2], l[3]);
}

// The weights of the hot loop go to the matrix cores as one fp16 operand (11 significant bits, against
// 8 for bf16), which needs V in fp16 as well: the threads that move a tile into LDS convert its V
// half on the way.  A bf16 value converts exactly while its magnitude lies in [2^-14, 65536); smaller
// ones lose at most 2^-24 absolute.  Larger ones do not occur here: the kernels that write V into the
// stores and the staging buffer raise the layer's v_wide flag when they see one, and the hot loop
// then takes V as stored.
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t x) {
  const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u));
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ uint4 bf16x8_to_f16x8(uint4 w) {
  return make_uint4(bf16x2_to_f16x2(w.x), bf16x2_to_f16x2(w.y), bf16x2_to_f16x2(w.z), bf16x2_to_f16x2(w.w));
}

// Eight fp32 weights (at most 2^(kSlack + kWeightShift) < 65504) as one fp16 operand, truncated: the
// normaliser is accumulated from the same operand, so the common part of the truncation cancels.
__device__ __forceinline__ void half_weights(const float (&p)[8], Frag& ph) {
  uint32_t h[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) h[k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(p[2 * k], p[2 * k + 1]));
  ph.u = make_uint4(h[0], h[1], h[2], h[3]);
}

// All weights of this kernel carry a factor 2^kWeightShift (it cancels between the accumulators and
// the normaliser): it keeps fp16 weights as small as 2^-30 of the reference maximum representable.
constexpr float kWeightShift = 6.f;

// What the wavefront's lanes have written to LDS is there for its other lanes (its LDS instructions run in order: the compiler only
// has to keep that order).
__device__ __forceinline__ void wave_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Online-softmax state of one 16-column group.  In the general loop the weights go to the matrix
// cores as in the decode kernel, a bf16 head plus a bf16 remainder (~16 mantissa bits; a single
// bf16 weight measurably misses the 1e-2 bar).  This kernel is bound by its vector instruction count, so the
// normaliser is accumulated by the matrix cores too, from the same two parts against a tile of
// ones: it needs no cross-lane sums.  V is the first operand of the products and the weights the second, so that a
// lane's accumulators, its scores, its normaliser and its reference all belong to its own column: rescaling takes no
// lane shuffles, and a lane's four outputs of a product lie side by side.  (With the operands the other way round one prompt
// of 32 500 tokens took 4404 us, against 4375, 16 x 16 384 16.23 ms, against 16.18.)
struct GroupState {
  float m;          // reference maximum of column lane%16 (log2 domain; same in all four k-groups)
  float ref;        // what the exponent subtracts: m (0 while m is -inf) minus kWeightShift
  float thr;        // a raw score above this makes the reference move: (m + slack) / scale
  floatx4 l;        // normaliser of column lane%16 (four equal rows)
  floatx4 o[8];     // O[column lane%16][d = 16*j + 4*(lane/16) + r]
};

// This file is compiled with -fno-honor-nans: fmaxf would otherwise first quiet a possible signalling
// NaN in every operand (three instructions per maximum); scores are never NaN here, and -inf (a masked
// score, an empty running maximum) is still honoured.
__device__ __forceinline__ float max8(const float (&v)[8]) {
  return fmaxf(fmaxf(fmaxf(fmaxf(v[0], v[1]), v[2]), fmaxf(fmaxf(v[3], v[4]), v[5])), fmaxf(v[6], v[7]));
}

// The reference maximum only moves when a score outgrows it by more than 2^kSlack; what depends on it
// is kept beside it, so that a tile costs one comparison and no arithmetic on the reference.
constexpr float kSlack = 8.f;
// (the reciprocal of the scale comes from the host: a division here was 20 instructions for a threshold that has slack, and the
// reciprocal's instruction gives 0 for scales beyond 2^126, whose reciprocal is a subnormal)
__device__ __forceinline__ void set_reference(GroupState& st, float m_new, float inv_scale) {
  st.m = m_new;
  st.ref = (m_new == -INFINITY ? 0.f : m_new) - kWeightShift;
  st.thr = (m_new + kSlack) * inv_scale;       // -inf while no key has been seen: any score moves it
}

// Accumulators and normaliser of the lane's column times `a`.
__device__ __forceinline__ void rescale(GroupState& st, float a) {
  st.l *= a;
#pragma unroll
  for (int j = 0; j < 8; ++j) st.o[j] *= a;
}

// Folds the masked raw scores `sc` of one tile (-inf = does not count) into the group's state;
// `scale` (> 0, log2 domain) is applied inside the exponent's fused multiply-add.
__device__ __forceinline__ void group_update(const TileRegs& t, const float (&sc)[8], float scale, float inv_scale, GroupState& st,
                                             const Frag& ones) {
  // The reference maximum only moves when some column's scores outgrow it by more than 2^kSlack:
  // until then the weights are simply larger than 1 (fp32 accumulators and the two-part bf16 split
  // are relative, so nothing is lost) and the accumulators need no rescaling.  Every lane holds its
  // column's reference, so the test needs the lane's own eight scores only; the column's maximum
  // (two cross-lane steps) is formed when the test fires.
  const float mx_lane = max8(sc);
  if (__any(mx_lane > st.thr)) {
    const float mx = column_max(mx_lane) * scale;
    const float m_new = fmaxf(st.m, mx);
    // a column that has seen no key yet still has a zero accumulator: factor 1
    const float alpha = st.m == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(st.m - m_new);
    set_reference(st, m_new, inv_scale);
    if (__any(alpha != 1.f)) rescale(st, alpha);
  }
  float p[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], scale, -st.ref));
  Frag phi, plo;
  split_weights(p, phi, plo);
  st.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, phi.v, st.l, 0, 0, 0);
  st.l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, plo.v, st.l, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    st.o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.v[j].v, phi.v, st.o[j], 0, 0, 0);
    st.o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.v[j].v, plo.v, st.o[j], 0, 0, 0);
  }
}

// A table entry that no workgroup of the launch writes, the same in all lanes: a scalar load (behind an asm statement the compiler
// takes an ordinary pointer's memory for possibly changed and loads lane by lane).
template <typename T> __device__ __forceinline__ T table_entry(const T* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// Brings the chunk's K/V rows (row-major [batch][n_kv_heads][stride][128]) into tiles of the MFMA layout, and the lengths
// forward (len_in -> len_out).  A full head's rows go where they stay, into its store: every query sees what it needs there, and
// nothing is evicted.  A compressed head's go to the staging buffer: staging tile t of a pair holds chunk rows 32 t .. 32 t + 31.
// Slots behind the last row are written as zeros: a staged tile never holds stale bits, and the last tile of a store goes out in
// whole units (8 x 1000 .. 4000 tokens that blend 643 -> 639 us).
// Bound: HBM, as tile_rows.h.  (Every head staged here and appended behind the attention launch took a second pass over the
// full heads' rows: 8 sequences of 1000 to 4000 tokens
// that blend, chunks of 1024: 700 -> 666 us; a prompt of 333 tokens and 32 decode steps: 291 -> 274 us; 16 x 16 384 tokens, half the
// heads full: 15.65 -> 15.57 ms.)
__global__ __launch_bounds__(kBlock) void place_chunk_kernel(DeviceView dv, int layer, SeqCounts seqs, const int32_t* __restrict__ len_in,
                                                             int32_t* __restrict__ len_out, const uint16_t* __restrict__ k_new,
                                                             const uint16_t* __restrict__ v_new, int stride_tokens,
                                                             char* __restrict__ staging, int staging_tiles,
                                                             uint64_t full_heads /* one bit a head; layers of up to kPrefillArgHeads */) {
  // (what has to be known before the first row is asked for, in two turns: the arguments, the tables)
  asm volatile("" :: "s"(dv.n_kv_heads), "s"(dv.n_pairs), "s"(dv.append_cnt), "s"(dv.store_off), "s"(dv.kv_base), "s"(dv.page_shift), "s"(layer),
                     "s"(seqs.in_args), "s"(len_in), "s"(len_out), "s"(k_new), "s"(v_new), "s"(stride_tokens), "s"(staging),
                     "s"(staging_tiles), "s"(full_heads));
  const int h = blockIdx.y, b = blockIdx.z, pair = b * dv.n_kv_heads + h;
  int t = seqs.in_args ? seqs.tok[b] : table_entry(dv.append_cnt + b);
  int n_old = table_entry(len_in + b);
  int64_t store_at = table_entry(dv.store_off + (int64_t)layer * dv.n_pairs + pair);
  asm volatile("" : "+s"(t), "+s"(n_old), "+s"(store_at));
  if (blockIdx.x == 0 && h == 0 && threadIdx.x == 0) len_out[b] = n_old + t;
  if (t == 0) return;
  const bool full = dv.n_kv_heads <= kPrefillArgHeads ? (full_heads >> h & 1) != 0 : dv.full_mask[layer * dv.n_kv_heads + h] != 0;
  const int tile = (full ? n_old / kTile : 0) + blockIdx.x;
  const int first = tile * kTile - (full ? n_old : 0);         // chunk row of slot 0 (a full head's first tile: may lie before the chunk)
  if (first >= t) return;
  const int64_t src_head = (int64_t)pair * stride_tokens * kHeadDim;
  __shared__ TileRowsLds lds;
  auto row_of = [&](int slot) { return first + slot >= 0 && first + slot < t ? first + slot : -1; };
  bool wide;
  if (full) {
    char* tile_base = dv.kv_base + store_at;
    if (dv.page_shift >= 0)
      tile_base += dv.block_table[(int64_t)b * dv.table_stride + (tile >> dv.page_shift)] * dv.page_bytes +
                   (int64_t)(tile & dv.page_mask) * kTileBytes;
    else
      tile_base += (int64_t)tile * kTileBytes;
    wide = rows_to_tile<false>(lds, row_of, [&](int slot) { return first + slot < 0; }, k_new + src_head, v_new + src_head, tile_base);
  } else {
    wide = rows_to_tile<false>(lds, row_of, [](int) { return false; }, k_new + src_head, v_new + src_head,
                               staging + ((int64_t)pair * staging_tiles + tile) * kTileBytes);
  }
  if (wide) dv.v_wide[layer] = 1;          // seen by the attention kernel that follows on the stream
}

// The items of a launch (see prefill_deal.h) and the heads of either class.  The heads come with the kernel arguments (one load
// instead of a loop of dependent loads over the layer's mask at the start of every workgroup), unless the layer has more than
// fit there.
struct PrefillGrid {
  PrefillItems items;
  int32_t n_split;                         // shares of every heavy item (1 = undivided; else dealt in plain order, not ragged)
  int32_t inv_group;                       // 65536 / group, rounded up
  float inv_scale;                         // 1 / scale_log2; 1 where that is not positive
  int32_t heads_given;                     // 1: `head` holds the heads
  uint64_t head[2][kPrefillArgHeads / 8];  // [0]: the full heads in ascending order, [1]: the compressed ones, 8 bits each
  int32_t first[kFirstEntries];
};
// Number in its class -> KV head.  first8: the class's first word of grid.head.
__device__ __forceinline__ int head_of_class(const DeviceView& dv, int layer, const PrefillGrid& grid, uint64_t first8, int head, bool full) {
  if (grid.heads_given) {
    if (head >= 8) first8 = grid.head[full ? 0 : 1][head >> 3];
    return (int)(first8 >> ((head & 7) * 8)) & 255;
  }
  for (int i = 0, k = head; i < dv.n_kv_heads; ++i) {
    if ((dv.full_mask[layer * dv.n_kv_heads + i] != 0) == full) {
      if (k == 0) return i;
      --k;
    }
  }
  return 0;
}

// Split prefill (few long workgroups: one or two sequences, few full heads): the unmasked tiles of a
// full head's workgroup are divided among n_split workgroups, each of which leaves its 256 columns'
// unnormalised accumulators, normalisers and reference maxima in a slot of scratch memory
// ([256][128] O, then [256] m, then [256] l, fp32); prefill_merge_kernel combines them.
constexpr int kSplitCols = 256;
constexpr int kSplitSlotFloats = kSplitCols * (kHeadDim + 2);
constexpr int kMergeColsPerGroup = 8;      // columns a workgroup of the merge kernel combines

constexpr int kPrefillWaves = 8;                 // wavefronts per workgroup: two per SIMD
constexpr int kPrefillBlock = kPrefillWaves * 64;



// A workgroup = one (sequence, KV head) pair x 8 wavefronts, two per SIMD so that one wavefront's
// vector work (exponentials, weight split, maxima) runs beside the other's matrix work.  Each
// wavefront owns NG 16-column groups of the workgroup's (position, head) columns, flattened
// position-major across the whole workgroup.
//
// MIX (some full head of the layer has an Eq. 1 gate below 1: out = gate * causal + (1 - gate) * local): the causal
// positions are the local ones and the rest, so a blending head's tiles are walked in two passes that share one set of
// accumulators - first what is local (sinks and recent band), whose finished result is put aside in LDS, then the rest, on
// top of it.  Every key is thus folded in once, a tile at the edge of the two in both passes.  (The form with two column groups takes
// all 256 registers and spills 4 more, 7 if paged: a Q operand, read back in the loop that takes V as stored.)  (Two accumulator sets side by side left room for one column group per wavefront, which makes the hot loop wait
// for LDS - 16 KiB of operands per wavefront and tile for 16 columns - and folded every local tile in twice, in the general
// loop: 8 sequences of 1000 to 4000 tokens in chunks of 1024, 28 query and 4 KV heads, 984 -> 775 us with the two passes,
// 880 us with one column group per wavefront.)
//
// Two loops.  The hot one takes the tiles that every query of the workgroup sees whole: those of a
// full head that lie wholly before the workgroup's first query (nearly all of a prefill's work),
// and for a compressed head its complete sink tiles and the chunk tiles before the first query
// that no query's recent band has left yet.  The eight wavefronts walk them together, every tile is
// fetched from memory once per workgroup into LDS (one barrier per tile; K straight into LDS, V
// through registers) and read from there as MFMA operands; no masks.  Of a blending head it takes, in the first pass, the complete
// sink tiles and those wholly inside the recent band of all queries, in the second those wholly between.  The general one takes
// everything else (partly filled tiles, a compressed head's ring, the causal diagonal, the tiles at the end of the sinks and at the
// band's edge), each wavefront on its own, with per-slot positions and masks.
template <bool PAGED, int NG, bool MIX>
__global__ __launch_bounds__(kPrefillBlock) void prefill_mfma_kernel(DeviceView dv, int layer,
                                                                     SeqOrder order,
                                                                     const int32_t* __restrict__ len_in,
                                                                     const uint16_t* __restrict__ q,
                                                                     uint16_t* __restrict__ out, int stride_tokens,
                                                                     float scale_log2,
                                                                     const char* __restrict__ staging,
                                                                     int staging_tiles, float* __restrict__ split_out,
                                                                     PrefillGrid grid) {
  // LDS: the K halves of four tiles (filled by loads that go from memory straight into LDS, two tiles ahead)
  // and the V halves of two (through registers: V is converted on the way); MIX: the local results, every lane its own.  With
  // two column groups these leave room for two K halves, which use up the 160 KiB of a CU: tiles are then asked for one ahead.
  constexpr int kKeySlots = MIX && NG == 2 ? 2 : 4;
  __shared__ uint4 sm_k[kKeySlots == 2 ? 1 : kKeySlots][kTileBytes / 32];
  __shared__ uint4 sm_k1[kKeySlots == 2 ? kTileBytes / 32 : 1];          // (an array of its own: the compiler would have reads of the
                                                                          // one slot wait for the loads into the other)
  __shared__ uint4 sm_v[2][kTileBytes / 32];
  __shared__ floatx4 sm_local[MIX ? kPrefillWaves : 1][MIX ? NG * 8 : 1][MIX ? 64 : 1];
  // Where a wavefront turns its outputs into rows: 4 KiB for each column group in its part of the local results, or, group by group,
  // in its eighth of the K halves (kKeySlots == 4).
  constexpr bool kOutInLocal = kKeySlots == 2;
  constexpr int kOutChunks = kOutInLocal ? 512 : 0;           // 16-byte units from one group's place to the next
  // Workgroups are handed out in the order of their index, and each XCD takes the items dealt to it (prefill_item) in
  // order: the long ones go first - the pairs of full heads before those of compressed heads, long
  // sequences before short ones, and within a pair the later query blocks (more keys under the
  // causal mask) before the earlier ones - so that the short ones fill the end.
  // Bound, for a short chunk: latency.  What it takes to find the workgroup's own is asked for in as few turns as there are dependent
  // loads, the arguments and then the sequence's tables, and in little code: it runs once, and a cold line of it costs as much as a
  // load.  The sequences' words of the arguments therefore come to the lanes of two registers, and are picked out of
  // them.  (Each argument waited for where it was first looked at, a dozen in a row, a search by halves and divisions: two prompts of 212
  // and 250 tokens, 32 query and 8 KV heads, 25.1 us; side by side, with a search in scalar registers, 24.6; like this 24.2.)
  // The empty statement uses the values, so that their loads are issued side by side here.
  PrefillItems items = grid.items;
  uint64_t head8[2] = {grid.head[0][0], grid.head[1][0]};
  const int lane0 = threadIdx.x & 63;
  const int32_t first_lo = grid.first[lane0], first_hi = grid.first[lane0 + 64];
  const int32_t seq_lo = order.seq[lane0], seq_hi = order.seq[lane0 + 64], tok_lo = order.tok[lane0], tok_hi = order.tok[lane0 + 64];
  asm volatile("" : "+s"(items.gx), "+s"(items.heads[0]), "+s"(items.heads[1]), "+s"(items.inv_heads[0]), "+s"(items.inv_heads[1]),
                    "+s"(items.inv_seq[0]), "+s"(items.inv_seq[1]), "+s"(head8[0]), "+s"(head8[1])
                  : "s"(dv.batch), "s"(dv.n_kv_heads), "s"(dv.store_off), "s"(len_in), "s"(order.in_args), "s"(grid.n_split),
                    "s"(stride_tokens), "s"(grid.heads_given), "s"(grid.inv_group));
  static_assert(kArgSeqs == 128 && kFirstEntries == kArgSeqs + 1);
  auto of_place = [](int32_t lo, int32_t hi, int place) { return __builtin_amdgcn_readlane(place < 64 ? lo : hi, place & 63); };
  int index, place, head, from_end, blocks, b, t, share = 0;      // t: chunk length of the sequence
  bool full;
  const int Z = kKeySlots == 2 ? 1 : grid.n_split;               // (the form of two column groups that blends is not divided)
  if (Z == 1) {
    full = prefill_item(blockIdx.x, items, index);
  } else {                                 // (plain order, the first share of everything, then the others of the heavy items)
    index = blockIdx.x;
    const int heavy = items.n_seqs * items.heads[0] * items.gx, all = heavy + items.n_seqs * items.heads[1] * items.gx;
    if (index >= all) {
      share = (index - all) / heavy;
      index -= all + share++ * heavy;
    }
    full = index < heavy;
    if (!full) index -= heavy;
  }
  if (items.ragged) {                      // (the order is in the arguments)
    const int heads = full ? items.heads[0] : items.heads[1];
    const int x = quotient(index, heads, full ? items.inv_heads[0] : items.inv_heads[1]);
    place = __popcll(__ballot(first_lo <= x)) + __popcll(__ballot(first_hi <= x)) - 1;
    const int at = of_place(first_lo, first_hi, place);
    blocks = (place + 1 < kArgSeqs ? of_place(first_lo, first_hi, place + 1) : grid.first[kArgSeqs]) - at;
    ragged_place(index, heads, at, blocks, head, from_end);
  } else {
    even_place(index, full, items, place, head, from_end);
    blocks = items.gx;
  }
  if (order.in_args) {
    b = of_place(seq_lo, seq_hi, place);
    t = of_place(tok_lo, tok_hi, place);
  } else {
    seq_in_order(dv, order, place, b, t);
  }
  const int h = __builtin_amdgcn_readfirstlane(head_of_class(dv, layer, grid, full ? head8[0] : head8[1], head, full));
  const int pair = b * dv.n_kv_heads + h;
  const int block_x = blocks - 1 - from_end;
  const int layer_head = layer * dv.n_kv_heads + h;
  int n_old = table_entry(len_in + b);     // positions cached before the chunk
  int64_t store_at = table_entry(dv.store_off + ((int64_t)layer * dv.batch + b) * dv.n_kv_heads + h);
  int64_t slots_at = table_entry(dv.slotpos_off + layer_head);
  int32_t v_wide = table_entry(dv.v_wide + layer);
  float gate = MIX ? table_entry(dv.gate + layer_head) : 1.f;
  asm volatile("" : "+s"(n_old), "+s"(store_at), "+s"(slots_at), "+s"(v_wide));
  if (MIX) asm volatile("" : "+s"(gate));
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int tid = threadIdx.x, lane = tid & 63;
  int hd = lane & 15;           // score layout: column; operand layouts: row / column
  int kb = lane >> 4;           // k-group of the operand layouts; slot quad of the score layout
  const int G = dv.group, S = dv.sink, R = dv.recent;
  constexpr int kWaveCols = 16 * NG;
  // Columns are at most 256 and groups at most 16, so that col / G is exact as a product with the reciprocal rounded up.
  const int inv_g = grid.inv_group;
  auto div_g = [&](int col) { return (col * inv_g) >> 16; };
  const int wg_positions = div_g(kPrefillWaves * kWaveCols);   // chunk positions per workgroup
  const int c_wg = block_x * wg_positions; // the workgroup's first chunk index
  if (c_wg >= t) return;
  const int c_last = (c_wg + wg_positions < t ? c_wg + wg_positions : t) - 1;   // its last one
  // share z of Z of a divided workgroup; the last share, the longest one (it also takes the masked tiles), is handed out first
  const int z = Z - 1 - share;
  const bool split = full && Z > 1;
  const bool wide = v_wide != 0;
  const bool mix = MIX && full && gate < 1.f;            // this head blends causal and local attention

  // This wavefront's columns: kWaveCols of the workgroup's flattened (position, head) pairs.
  const int col0 = wave * kWaveCols;
  const int c0 = c_wg + div_g(col0);                                      // first chunk index it touches
  const int c_hi_raw = c_wg + div_g(col0 + kWaveCols - 1);
  const int c_hi = c_hi_raw < c_last ? c_hi_raw : c_last;               // last one
  const bool busy = c0 <= c_last;                                        // it has at least one query
  Frag qb[NG][4];               // Q as the B operand of the score MFMA
  int qpos[NG];                 // absolute position of the lane's column, -1 = no such query
  int g_lo[NG], g_hi[NG];       // positions a group holds
  bool g_on[NG];
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    const int col = col0 + 16 * cg + hd;
    const int cl = div_g(col), hh = col - cl * G;
    const bool valid = c_wg + cl <= c_last;
    qpos[cg] = valid ? n_old + c_wg + cl : -1;
    const int64_t qrow = ((int64_t)b * dv.n_q_heads + h * G + hh) * stride_tokens + c_wg + cl;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 qv = make_uint4(0, 0, 0, 0);
      if (valid)
        qv = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(q) + (qrow * kHeadDim + s * 32 + kb * 8) * 2);
      qb[cg][s].u = qv;
    }
    const int cl_lo = div_g(col0 + 16 * cg), cl_hi = div_g(col0 + 16 * cg + 15);
    g_on[cg] = c_wg + cl_lo <= c_last;
    g_lo[cg] = n_old + c_wg + cl_lo;
    g_hi[cg] = n_old + (c_wg + cl_hi < c_last ? c_wg + cl_hi : c_last);
  }

  TileMap<PAGED> store;
  store.base = dv.kv_base + store_at;
  store.paged = PAGED && full;
  if (PAGED) {
    store.row = dv.block_table + (int64_t)b * dv.table_stride;
    store.page_bytes = dv.page_bytes;
    store.shift = dv.page_shift;
    store.mask = dv.page_mask;
    store.last = dv.table_stride - 1;
  }
  const char* stage = staging + (int64_t)pair * staging_tiles * kTileBytes;
  const int32_t* slot_pos = nullptr;
  if (!full) slot_pos = dv.slot_pos + slots_at + (int64_t)b * dv.window;

  // store slots that hold data: of a full head the chunk's too, of a compressed one what was cached before it
  const int n_st = full ? n_old + t : (n_old < dv.window ? n_old : dv.window);
  const int sink_in_chunk = S - n_old;       // chunk indices below this are sink positions

  // Hot tiles (same for all wavefronts of the workgroup): tiles in which every slot counts for every
  // query of the workgroup.  Full head: the store's tiles up to the workgroup's first query.
  // Compressed head: the store's complete sink tiles, and the staging
  // tiles wholly before the first query that also lie wholly inside the recent band of the last one
  // (a chunk is usually longer than the band, so these are most of what such a head attends over).
  // A blending head's first pass (kLocal): of the tiles up to the first query the complete sink tiles and those
  // wholly inside the recent band of the last one; its second pass (kRest): the tiles wholly behind the
  // sinks and wholly before the band of the first query.  (A softmax scale that is not positive, unusual, takes the
  // general loop throughout.)
  const bool hot = scale_log2 > 0.f;
  const int q_first = n_old + c_wg;                      // position of the workgroup's first query
  const int band_first = c_last - R + 1;                 // first chunk index that the last query's band holds

  // General tiles of this wavefront: store tiles [0, n_store), then staging tiles [0, n_stage), without those that are hot or
  // of no use to it.
  const int band_lo = c0 - R + 1;            // first chunk index inside the recent band of the wavefront's first query
  const int sink_tiles = sink_in_chunk > 0 ? (sink_in_chunk + kTile - 1) / kTile : 0;            // staging tiles with sink positions
  const int band_tile = band_lo > 0 ? band_lo / kTile : 0;                                       // the band's first staging tile

  // What a pass takes.  kWhole: a head that does not blend, its one pass.
  enum { kLocal, kRest, kWhole };
  int hs_lo, hs_hi;                          // hot store tiles [hs_lo, hs_hi)
  int hb_lo, hb_hi;                          // kLocal: further ones, those of the band
  int stg_lo, stg_hi;                        // hot staging tiles [stg_lo, stg_hi)
  int n_store, n_stage;                      // general tiles: ranges, ...
  int skip_lo = 0, skip_hi = 0;              // ... store tiles (beside the hot ones) and ...
  int skip_stg_lo = 0, skip_stg_hi = 0;      // ... staging tiles that it passes over
  auto plan_pass = [&](int pass) {
    hs_lo = hs_hi = hb_lo = hb_hi = stg_lo = stg_hi = 0;
    if (!full) {
      n_stage = c_hi / kTile + 1;
      if (hot) {
        hs_hi = (S < n_st ? S : n_st) / kTile;
        stg_hi = c_wg / kTile;                           // staging tiles wholly before the first query
        stg_lo = band_first > 0 ? (band_first + kTile - 1) / kTile : 0;
        if (stg_lo > stg_hi) stg_lo = stg_hi;
      }
      // the ring matters only while the wavefront's first query still reaches positions before the chunk
      const int reach = c0 < R ? n_st : (S < n_st ? S : n_st);
      n_store = (reach + kTile - 1) / kTile;
      skip_stg_lo = sink_tiles;
      skip_stg_hi = band_tile;
      return;
    }
    n_store = (n_old + c_hi) / kTile + 1;
    n_stage = 0;
    const int seen = hot ? (q_first + 1) / kTile : 0;    // store tiles that the first query sees whole
    if (!MIX || pass == kWhole) {
      hs_hi = seen;
      return;
    }
    const int sinks_up = (S + kTile - 1) / kTile;
    if (pass == kLocal) {
      const int band = n_old + band_lo;                  // first position of the wavefront's band
      const int band_whole = n_old + band_first > 0 ? (n_old + band_first + kTile - 1) / kTile : 0;
      hs_hi = S / kTile < seen ? S / kTile : seen;
      hb_hi = seen;
      hb_lo = band_whole > hs_hi ? band_whole : hs_hi;
      if (hb_lo > hb_hi) hb_lo = hb_hi;
      skip_lo = sinks_up;                                // between the sinks and the band
      skip_hi = band > 0 ? band / kTile : 0;
    } else {
      const int rest = n_old + c_hi - R;                 // last position outside the band of the wavefront's last query
      const int rest_tiles = rest >= 0 ? rest / kTile + 1 : 0;
      if (rest_tiles < n_store) n_store = rest_tiles;
      if (hot) {
        const int before = q_first - R + 1;              // first position of the first query's band
        hs_lo = sinks_up;
        hs_hi = before > 0 ? before / kTile : 0;
        if (hs_hi < hs_lo) hs_hi = hs_lo;
      }
      skip_lo = 0;                                       // nothing but sinks
      skip_hi = S / kTile < n_store ? S / kTile : n_store;
    }
  };
  // The first general tile at or behind x.  Ranges are hopped over, not walked: at 16 384 cached tokens the walk over a full
  // head's 512 hot tiles took longer than the tiles here.
  auto next_needed = [&](int x) {
    if (MIX && x >= skip_lo && x < skip_hi) x = skip_hi;
    if (x >= hs_lo && x < hs_hi) x = hs_hi;
    if (MIX && x >= skip_lo && x < skip_hi) x = skip_hi;
    if (MIX && x >= hb_lo && x < hb_hi) x = hb_hi;
    if (x < n_store) return x;
    int j = x - n_store;
    if (j >= skip_stg_lo && j < skip_stg_hi) j = skip_stg_hi;
    if (j >= stg_lo && j < stg_hi) j = stg_hi;
    return j + n_store;
  };
  auto address = [&](int x) -> const char* {
    return x < n_store ? store.at(x) : stage + (int64_t)(x - n_store) * kTileBytes;
  };

  Frag ones;
  ones.u = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);      // eight bf16 1.0
  GroupState st[NG];
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    set_reference(st[k], -INFINITY, 1.f);
    st[k].l = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) st[k].o[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // The softmax scale rides in the exponent's multiply-add.  A negative one (unusual) would turn the
  // running maximum into a minimum, and zero times the -inf of a masked score is not a number, so
  // those two are applied to the scores up front (general loop) instead.
  const float exp_scale = scale_log2 > 0.f ? scale_log2 : 1.f;
  const float inv_scale = grid.inv_scale;

  // One pass, or two of a blending head (of a divided workgroup, the last share takes what is local).
  int pass = !mix ? kWhole : split && z != Z - 1 ? kRest : kLocal;
  auto walk = [&](auto local_tag) {
  constexpr bool LOCAL_PASS = decltype(local_tag)::value;
  plan_pass(pass);
  const int hot_store = hs_hi - hs_lo, hot_band = MIX ? hb_hi - hb_lo : 0;
  const int n_plain_all = hot_store + hot_band + stg_hi - stg_lo;
  // (a divided workgroup: share z of Z of them; the last share also takes the general tiles)
  const bool divide = split && pass != kLocal;
  const int plain_lo = divide ? (int)((int64_t)n_plain_all * z / Z) : 0;
  const int n_plain = divide ? (int)((int64_t)n_plain_all * (z + 1) / Z) - plain_lo : n_plain_all;
  auto plain_address = [&](int i0) -> const char* {
    const int i = i0 + plain_lo;
    if (MIX && i >= hot_store && i < hot_store + hot_band) return store.at(hb_lo + i - hot_store);
    return i < hot_store ? store.at(hs_lo + i) : stage + (int64_t)(stg_lo + i - hot_store - hot_band) * kTileBytes;
  };
  const int total = busy && (!split || z == Z - 1) ? n_store + n_stage : 0;

  // ---- hot loop: the whole workgroup, tiles through LDS ---------------------------------------
  // Thread i moves 16 bytes of the tile's K half and 16 of its V half.  The loop exists in two forms.
  // The usual one (HALF) puts V into LDS as fp16 and sends the weights to the matrix cores as one
  // fp16 operand.  The other one, for a layer whose v_wide flag is up (some V value beyond the fp16
  // range has been appended since the cache was last empty; unusual) and for the local pass of a blending head, takes V as
  // stored, with two-part bf16 weights.
  // (MIX: the second wavefront of every SIMD goes first where both could issue, which keeps the two out of step: one's exponentials beside
  // the other's products.  8 x 1000 .. 4000 tokens that blend 663 -> 659 us; in the one-group form one of 2670 tokens in chunks of 512 241.5 ->
  // 239.1, 8 x 291 .. 868 79.7 -> 78.0, 5 x 2735 .. 3469 734 -> 728.  The two-group form of plain heads: 0.3 % slower with it.)
  auto hot_loop = [&](auto half_tag) {
    // (It stays raised behind the loop, through the general tiles and the output.)
    if ((MIX || NG == 1) && wave >= kPrefillWaves / 2) __builtin_amdgcn_s_setprio(1);
    constexpr bool HALF = decltype(half_tag)::value;
    uint4 next_v = make_uint4(0, 0, 0, 0);      // the next tile's V as fp16, when the loop body has converted it already
    bool next_ready = false;
    auto put = [&](int x, const uint4& v16) {
      if (HALF) {
        sm_v[x & 1][tid] = next_ready ? next_v : bf16x8_to_f16x8(v16);
        next_ready = false;
      } else {
        sm_v[x & 1][tid] = v16;
      }
    };
    // Buffer loads: the tile's address travels in scalar registers (a descriptor made per tile) and the
    // per-thread offset is one fixed vector register, so no vector address registers are written while
    // earlier loads are still in flight (which the compiler answers with a wait for all of them).
    const int thread_off = tid * 16;
    // The K half goes from memory straight into LDS (lane i of a wavefront fills bytes 16 i .. 16 i + 15 behind
    // the wavefront's base, which is the tile's own order): no registers, no LDS store instruction.  Both
    // halves of a tile are asked for two tiles ahead; the compiler makes every wavefront wait for its loads into
    // LDS before the next barrier (the K half therefore has one iteration to arrive), the V half, which
    // passes through registers to be converted, is waited for where it is used, an iteration later.
    auto resource = [&](int x) {
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(plain_address(x)), 0, kTileBytes, 0x00020000);
    };
    auto fetch_k = [&](const __amdgpu_buffer_rsrc_t& rsrc, uint4* slot) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(slot + wave * 64), 16, thread_off, 0, 0, 0);
    };
    auto fetch_v = [&](const __amdgpu_buffer_rsrc_t& rsrc, uint4& v16) {
      const u32x4 vv = __builtin_amdgcn_raw_buffer_load_b128(rsrc, thread_off, 8192, 0);
      v16 = make_uint4(vv[0], vv[1], vv[2], vv[3]);
    };
    Frag ones_op = ones;
    if (HALF) ones_op.u = make_uint4(0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u);    // eight fp16 1.0
    // One tile.  c1 holds this thread's 16 bytes of V of tile x + 1, asked for an iteration ago; the loads of
    // tile x + 2 are issued here, K into LDS, V into f1.  Two iterations ahead, in two register sets that
    // swap roles: the workgroups of a pair walk its tiles at about the same time, so most of these loads find
    // their line still on its way from HBM, and one iteration (about a microsecond) does not cover that.  (Two key slots: tile
    // x + 1, V into c1 too.)
    auto step = [&](auto odd_tag, int x, uint4& c1, uint4& f1) {
      constexpr bool ODD = decltype(odd_tag)::value;
      if (kKeySlots == 2) __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt 0: this wavefront's part of tile x's K half is in LDS
      __syncthreads();          // tile x is complete in its buffers; nobody reads the buffers written next any more
      const uint4* kbuf = kKeySlots == 2 ? (ODD ? sm_k1 : sm_k[0]) : sm_k[x & (kKeySlots - 1)];
      const uint4* vbuf = sm_v[x & 1];
      TileRegs tr;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)                      // (also by a wavefront without queries: no branch here)
#pragma unroll
        for (int s = 0; s < 4; ++s) tr.k[hf][s].u = kbuf[(hf * 4 + s) * 64 + lane];
      auto read_v = [&]() {
#pragma unroll
        for (int j = 0; j < 8; ++j) tr.v[j].u = vbuf[j * 64 + lane];
      };
      if (kKeySlots == 4) read_v();             // (two slots: behind the scores, for the registers)
      // (past the end: the last tile again, unused)
      if constexpr (kKeySlots == 4) {
        const __amdgpu_buffer_rsrc_t rsrc = resource(x + 2 < n_plain ? x + 2 : n_plain - 1);
        fetch_k(rsrc, sm_k[(x + 2) & 3]);
        fetch_v(rsrc, f1);
      } else {                                   // (the other key slot was last read before this barrier)
        const __amdgpu_buffer_rsrc_t rsrc = resource(x + 1 < n_plain ? x + 1 : x);
        fetch_k(rsrc, ODD ? sm_k[0] : sm_k1);
        fetch_v(rsrc, c1);
      }
      if (busy) {
        float sc[NG][8], mx[NG];
        bool grow = false;
#pragma unroll
        for (int cg = 0; cg < NG; ++cg) {
          raw_scores(tr, qb[cg], sc[cg]);
          // (every lane holds its column's reference: the test needs the lane's own scores only)
          mx[cg] = max8(sc[cg]);
          grow |= mx[cg] > st[cg].thr;
        }
        if (kKeySlots == 2) {
          __builtin_amdgcn_sched_barrier(0);
          read_v();
        }
        if (__any(grow)) {
          // a maximum moved by more than the slack (rare): new references, accumulators rescaled
#pragma unroll
          for (int cg = 0; cg < NG; ++cg) {
            const float m_new = fmaxf(st[cg].m, column_max(mx[cg]) * exp_scale);
            const float alpha = st[cg].m == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(st[cg].m - m_new);
            set_reference(st[cg], m_new, inv_scale);
            rescale(st[cg], alpha);
          }
        }
        if constexpr (HALF && NG == 2) {
          // Two column groups, written out in issue order: a wavefront's own vector instructions run
          // beside its matrix instructions (those of another wavefront of the SIMD do not), so the
          // exponentials of the second group sit between the matrix instructions of the first, and the
          // fp16 conversion of the next tile's V between those of the second.  The scheduling barriers
          // keep the compiler from gathering each kind again.
          const float ref0 = st[0].ref, ref1 = st[1].ref;
          float p[8];
          Frag ph0, ph1;
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0][e], exp_scale, -ref0));
          half_weights(p, ph0);
          __builtin_amdgcn_sched_barrier(0);
          st[0].l = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones_op.h, ph0.h, st[0].l, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[1][j], exp_scale, -ref1));
            __builtin_amdgcn_sched_barrier(0);
            st[0].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr.v[j].h, ph0.h, st[0].o[j], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          half_weights(p, ph1);
          __builtin_amdgcn_sched_barrier(0);
          st[1].l = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones_op.h, ph1.h, st[1].l, 0, 0, 0);
          uint32_t hw[4];
          const uint32_t gw[4] = {c1.x, c1.y, c1.z, c1.w};
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if (j < 4) hw[j] = bf16x2_to_f16x2(gw[j]);
            __builtin_amdgcn_sched_barrier(0);
            st[1].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr.v[j].h, ph1.h, st[1].o[j], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          next_v = make_uint4(hw[0], hw[1], hw[2], hw[3]);
          next_ready = true;
        } else if constexpr (HALF && NG == 1) {
          // One column group: the fp16 conversion of the next tile's V sits between the matrix instructions.
          const float ref0 = st[0].ref;
          float p[8];
          Frag ph0;
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0][e], exp_scale, -ref0));
          half_weights(p, ph0);
          __builtin_amdgcn_sched_barrier(0);
          st[0].l = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones_op.h, ph0.h, st[0].l, 0, 0, 0);
          uint32_t hw[4];
          const uint32_t gw[4] = {c1.x, c1.y, c1.z, c1.w};
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if (j < 4) hw[j] = bf16x2_to_f16x2(gw[j]);
            __builtin_amdgcn_sched_barrier(0);
            st[0].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr.v[j].h, ph0.h, st[0].o[j], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          next_v = make_uint4(hw[0], hw[1], hw[2], hw[3]);
          next_ready = true;
        } else if constexpr (!HALF && NG == 2) {
          // (the same for two-part weights)
          const float ref0 = st[0].ref, ref1 = st[1].ref;
          float p[8];
          Frag hi, lo;
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0][e], exp_scale, -ref0));
          split_weights(p, hi, lo);
          __builtin_amdgcn_sched_barrier(0);
          st[0].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, hi.v, st[0].l, 0, 0, 0);
          st[0].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, lo.v, st[0].l, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[1][j], exp_scale, -ref1));
            __builtin_amdgcn_sched_barrier(0);
            st[0].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, hi.v, st[0].o[j], 0, 0, 0);
            st[0].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, lo.v, st[0].o[j], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          split_weights(p, hi, lo);
          st[1].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, hi.v, st[1].l, 0, 0, 0);
          st[1].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, lo.v, st[1].l, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            st[1].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, hi.v, st[1].o[j], 0, 0, 0);
            st[1].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, lo.v, st[1].o[j], 0, 0, 0);
          }
        } else
#pragma unroll
        for (int cg = 0; cg < NG; ++cg) {
          const float m_ref = st[cg].ref;
          float p[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[cg][e], exp_scale, -m_ref));
          if (HALF) {
            Frag ph;
            half_weights(p, ph);
            st[cg].l = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones_op.h, ph.h, st[cg].l, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 8; ++j)
              st[cg].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr.v[j].h, ph.h, st[cg].o[j], 0, 0, 0);
          } else {
            Frag phi, plo;
            split_weights(p, phi, plo);
            st[cg].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, phi.v, st[cg].l, 0, 0, 0);
            st[cg].l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_op.v, plo.v, st[cg].l, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              st[cg].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, phi.v, st[cg].o[j], 0, 0, 0);
              st[cg].o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr.v[j].v, plo.v, st[cg].o[j], 0, 0, 0);
            }
          }
        }
      }
      put(x + 1, c1);           // (after the last tile: a copy of it into the buffer nobody reads any more)
    };
    uint4 a1, b1;
    fetch_k(resource(0), sm_k[0]);
    fetch_v(resource(0), a1);
    put(0, a1);
    if (kKeySlots == 4) fetch_k(resource(1 < n_plain ? 1 : 0), sm_k[kKeySlots == 4 ? 1 : 0]);
    if (kKeySlots == 4) fetch_v(resource(1 < n_plain ? 1 : 0), a1);
    for (int x = 0; x < n_plain; x += 2) {
      step(std::false_type{}, x, a1, b1);
      if (x + 1 < n_plain) step(std::true_type{}, x + 1, kKeySlots == 2 ? a1 : b1, a1);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt 0: no load into LDS is left in flight behind the loop
  };
  if (n_plain > 0) {
    if constexpr (LOCAL_PASS) hot_loop(std::false_type{});
    else if (!wide) hot_loop(std::true_type{});
    else hot_loop(std::false_type{});
    if (!kOutInLocal && !LOCAL_PASS) __syncthreads();          // the outputs take the place of the K halves
  }
  if (!busy) return;

  // ---- general loop: this wavefront alone, tiles straight from memory -------------------------
  // One tile: mask the scores of each column group and fold the tile into its softmax state.
  // Bound: vector instructions (the matrix work of a tile and group is 26 instructions of 16 clocks, and two wavefronts
  // share a SIMD).  So the mask of a tile is chosen once per group, the same in all lanes: none, one comparison per slot
  // (causal diagonal, end of the store), two (the band's edge), and only a tile whose slots are in no order of positions
  // (a compressed head's ring) or that holds the end of the sinks looks every position up.  With the hops above, against every
  // position looked up and compared three ways: 16 x 16 384 tokens in chunks of 2048 (28 query, 4 KV heads, 2 full)
  // 16.2 -> 15.2 ms, one sequence of 32 500 4.53 -> 4.11 ms, blending heads (8 x 1000 .. 4000) 1157 -> 1020 us.
  auto process = [&](TileRegs& tr, int x, const char* refill) {
    const bool from_store = x < n_store;
    const int tile = from_store ? x : x - n_store;
    const int held = from_store ? n_st : t;                     // slots of this source that hold a position
    const bool complete = tile * kTile + kTile <= held;         // every slot of the tile does
    const bool ring = from_store && !full;                      // the slot table says which positions the slots hold
    const int base = from_store ? tile * kTile : n_old + tile * kTile;      // position of slot 0 (not `ring`)
    const int slot0 = tile * kTile + kb * 4;                    // the lane's slots: slot0 + offset(e)
    auto offset = [](int e) { return (e >> 2) * 16 + (e & 3); };
    if (from_store && !complete) {
      // slots of the store that were never written may hold anything: clear their V operands
      uint32_t msk[4];
#pragma unroll
      for (int jw = 0; jw < 4; ++jw)
        msk[jw] = (offset(2 * jw) < held - slot0 ? 0x0000ffffu : 0u) | (offset(2 * jw + 1) < held - slot0 ? 0xffff0000u : 0u);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        tr.v[j].u.x &= msk[0]; tr.v[j].u.y &= msk[1]; tr.v[j].u.z &= msk[2]; tr.v[j].u.w &= msk[3];
      }
    }
    // positions this tile can hold (store tiles of a compressed head: anything before the chunk)
    const int p_first = ring ? 0 : base;
    const int p_last = ring ? n_old - 1 : base + kTile - 1;
    const bool local = !full || LOCAL_PASS;                     // only local positions count; or
    const bool rest = MIX && !LOCAL_PASS && pass == kRest;                     // only those that are not; or all
    auto masked = [&](int cg, const float (&raw)[8], float (&sc)[8]) {
      const int i = qpos[cg];
      if (ring || ((local || rest) && p_first < S && p_last >= S)) {
        int p[8];
        if (ring) {
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = slot_pos[min(slot0 + offset(e), held - 1)];    // (all asked for side by side)
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = base + kb * 4 + offset(e);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int near = (p[e] < S) | (i - p[e] < R);
          const int on = (slot0 + offset(e) < held) & (p[e] <= i) & (MIX ? (local & near) | (rest & (near ^ 1)) : near);
          sc[e] = on ? raw[e] : -INFINITY;
        }
        return;
      }
      const int own = i - base - kb * 4;                        // offset of the query's own position, ...
      const int end = rest ? own - R : own;                     // ... of the last one that counts
      const int top = complete ? end : min(end, held - 1 - slot0);
      if (local && p_first >= S && g_hi[cg] - p_first >= R) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sc[e] = offset(e) <= top && offset(e) > own - R ? raw[e] : -INFINITY;
      } else if (!complete || p_last > (rest ? g_lo[cg] - R : g_lo[cg])) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sc[e] = offset(e) <= top ? raw[e] : -INFINITY;
      } else {
        // (columns that stand for no query compute on zeros and are never written out)
#pragma unroll
        for (int e = 0; e < 8; ++e) sc[e] = raw[e];
      }
    };
    // the scores of every group that sees the tile; then the K registers take the next tile, and behind the last products
    // the V registers do
    bool sees[NG];
    float raw[NG][8];
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) {
      // (not: wholly above the causal diagonal, or wholly before the recent band; of the rest: wholly sinks or in the band)
      sees[cg] = g_on[cg] && p_first <= (rest ? g_hi[cg] - R : g_hi[cg]) &&
                 (local ? p_first < S || p_last >= g_lo[cg] - R + 1 : !rest || p_last >= S);
      if (!sees[cg]) continue;
      raw_scores(tr, qb[cg], raw[cg]);
      if (!hot) {
#pragma unroll
        for (int e = 0; e < 8; ++e) raw[cg][e] *= scale_log2;
      }
    }
    load_k_cached(tr, refill, lane);
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) {
      if (!sees[cg]) continue;
      float sc[8];
      masked(cg, raw[cg], sc);
      group_update(tr, sc, exp_scale, inv_scale, st[cg], ones);
    }
    load_v_cached(tr, refill, lane);
  };
  {
    TileRegs tr;
    int x = next_needed(0);
    if (x < total) {
      const char* base = address(x);
      load_k_cached(tr, base, lane);
      load_v_cached(tr, base, lane);
      while (x < total) {
        // (behind the last tile it is asked for once more: no branch around the loads, so that nothing waits for the newest)
        const int nx = next_needed(x + 1);
        if (nx < total) base = address(nx);
        process(tr, x, base);
        x = nx;
      }
    }
  }

  };
  if constexpr (MIX) {
    if (pass == kLocal) {
      walk(std::true_type{});
      // what is local is complete: its result is put aside, and the rest goes on top of its accumulators
      pass = kRest;
      if (busy) {
#pragma unroll
        for (int cg = 0; cg < NG; ++cg) {
          const float inv = 1.f / st[cg].l[0];
#pragma unroll
          for (int j = 0; j < 8; ++j) sm_local[wave][cg * 8 + j][lane] = st[cg].o[j] * inv;
        }
      }
      __syncthreads();          // nobody reads the tile buffers any more
    }
    asm volatile("" : "+v"(tid));
    lane = tid & 63; hd = lane & 15; kb = lane >> 4;
  }
  walk(std::false_type{});
  if (!busy) return;            // no barrier lies ahead

  // Accumulators and outputs leave through LDS: a lane holds four values in a row of its own column, and 16 neighbouring lanes
  // belong to 16 rows, so they are turned into whole rows first, 16 lanes each.  (Stored from where they are, every
  // instruction is 64 requests of 8 or 16 bytes: the launch over 16 chunks of 300 tokens, 32 query and 8 KV heads, 49.1 us, now
  // 44.9; 14 of 142 .. 289 35.2, now 31.2; a prompt of 2670 in chunks of 512, divided, 241 us in all, now 236; blending, 8 x 1000 ..
  // 4000, 666, now 648.)  16-byte chunk c of row r lies at chunk c ^ r, which spreads both sides over all banks.  (Values keep their
  // type on the way: cast to integers here, the accumulators were copied between registers in every step of the hot loop, 8 %.)
  u32x4* rows = kOutInLocal ? reinterpret_cast<u32x4*>(sm_local[MIX ? wave : 0]) : reinterpret_cast<u32x4*>(&sm_k[0][0]) + wave * 256;
  if (split) {
    float* slot = split_out + ((int64_t)index * Z + z) * kSplitSlotFloats;
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      const int col = col0 + 16 * k + hd;                // the lane's own column
      if (kb == 0) {
        slot[kSplitCols * kHeadDim + col] = st[k].m;
        slot[kSplitCols * (kHeadDim + 1) + col] = st[k].l[0];
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {             // 64 of a row's 128 values at a time
#pragma unroll
        for (int j = 0; j < 4; ++j) reinterpret_cast<floatx4*>(rows)[hd * 16 + ((j * 4 + kb) ^ hd)] = st[k].o[half * 4 + j];
        wave_exchange();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = i * 4 + kb;
          *reinterpret_cast<u32x4*>(slot + (col0 + 16 * k + row) * kHeadDim + half * 64 + hd * 4) = rows[row * 16 + (hd ^ row)];
        }
        wave_exchange();
      }
      if (MIX && mix && z == Z - 1) {          // the local results, as columns 128 and up (one column group)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          *reinterpret_cast<floatx4*>(slot + (kSplitCols / 2 + col) * kHeadDim + j * 16 + kb * 4) = sm_local[MIX ? wave : 0][MIX ? k * 8 + j : 0][MIX ? lane : 0];
      }
    }
    return;
  }
  // out[b][head][c][d] = O / l (blended with the local result for a gated head)
  const uintptr_t out_bits = reinterpret_cast<uintptr_t>(out);               // (a caller's may start at any element)
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    u32x4* mine = rows + cg * kOutChunks;
    const float inv = 1.f / st[cg].l[0];
    u32x2 four[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      floatx4 res = st[cg].o[j] * inv;
      if (MIX && mix) res = gate * res + (1.f - gate) * sm_local[MIX ? wave : 0][MIX ? cg * 8 + j : 0][MIX ? lane : 0];
      four[j] = u32x2{bf16_pair(res[0], res[1]), bf16_pair(res[2], res[3])};
    }
    wave_exchange();
#pragma unroll
    for (int j = 0; j < 8; ++j) reinterpret_cast<u32x2*>(mine + hd * 16 + ((j * 2 + (kb >> 1)) ^ hd))[kb & 1] = four[j];
    wave_exchange();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 4 + kb, col = col0 + 16 * cg + row;
      const int cl = div_g(col), hh = col - cl * G;
      const u32x4 w = mine[row * 16 + (hd ^ row)];
      uint16_t* dst = out + (((int64_t)b * dv.n_q_heads + h * G + hh) * stride_tokens + c_wg + cl) * kHeadDim + hd * 8;
      if (c_wg + cl > c_last) continue;
      if ((out_bits & 15) == 0) {
        *reinterpret_cast<u32x4*>(dst) = w;
      } else if ((out_bits & 7) == 0) {
        reinterpret_cast<u32x2*>(dst)[0] = u32x2{w[0], w[1]};
        reinterpret_cast<u32x2*>(dst)[1] = u32x2{w[2], w[3]};
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] = (uint16_t)(w[e >> 1] >> (e & 1) * 16);
      }
    }
  }
}

// Combines the shares of a divided workgroup: weights 2^(m_z - max m) on each share's accumulators and
// normaliser (every share's weights carry the same 2^kWeightShift, which cancels).  A share that saw no
// key has m = -inf and counts for nothing; the last share always holds the query's own position.
// MIX: a block has 128 columns, and a blending head's local results are columns 128 and up of its last share.
template <bool MIX>
__global__ __launch_bounds__(kSplitCols) void prefill_merge_kernel(DeviceView dv, int layer, SeqOrder order, const float* __restrict__ split_out,
                                                                   int Z, uint16_t* __restrict__ out, int stride_tokens,
                                                                   PrefillGrid grid) {
  const int place = quotient(blockIdx.y, grid.items.heads[0], grid.items.inv_heads[0]);
  int b, t;
  seq_in_order(dv, order, place, b, t);
  const int h = head_of_class(dv, layer, grid, grid.head[0][0], blockIdx.y - place * grid.items.heads[0], true);
  const int G = dv.group;
  const int wg_positions = (MIX ? kSplitCols / 2 : kSplitCols) / G;
  const int c_wg = (gridDim.x - 1 - blockIdx.x) * wg_positions;
  if (c_wg >= t) return;
  const float gate = MIX ? dv.gate[layer * dv.n_kv_heads + h] : 1.f;
  const bool mix = MIX && gate < 1.f;
  const int c_last = (c_wg + wg_positions < t ? c_wg + wg_positions : t) - 1;
  const float* slot0 = split_out + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * Z * kSplitSlotFloats;
  // eight columns per workgroup, four per thread: the loads behind the four outputs are independent, so
  // their latencies overlap, and there are still thousands of workgroups
  const int d = threadIdx.x & (kHeadDim - 1);
  constexpr int kPer = kMergeColsPerGroup / 2;
  int col[kPer];
  bool on[kPer];
  float local[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    col[i] = blockIdx.z * kMergeColsPerGroup + 2 * i + (threadIdx.x >> 7);
    on[i] = c_wg + col[i] / G <= c_last;
    local[i] = mix && on[i] ? slot0[(int64_t)(Z - 1) * kSplitSlotFloats + (kSplitCols / 2 + col[i]) * kHeadDim + d] : 0.f;
  }
  float M[kPer], num[kPer], den[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    M[i] = -INFINITY;
    num[i] = den[i] = 0.f;
  }
  for (int zz = 0; zz < Z; ++zz) {
    const float* sl = slot0 + (int64_t)zz * kSplitSlotFloats;
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (on[i]) M[i] = fmaxf(M[i], sl[kSplitCols * kHeadDim + col[i]]);
  }
  for (int zz = 0; zz < Z; ++zz) {
    const float* sl = slot0 + (int64_t)zz * kSplitSlotFloats;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (!on[i]) continue;
      const float m = sl[kSplitCols * kHeadDim + col[i]];
      const float w = m == -INFINITY ? 0.f : exp2f(m - M[i]);
      num[i] += w * sl[col[i] * kHeadDim + d];
      den[i] += w * sl[kSplitCols * (kHeadDim + 1) + col[i]];
    }
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (!on[i]) continue;
    const int cl = col[i] / G, hh = col[i] - cl * G;
    const int64_t orow = ((int64_t)b * dv.n_q_heads + h * G + hh) * stride_tokens + c_wg + cl;
    const float r = num[i] / den[i];
    out[orow * kHeadDim + d] = f32_to_bf16_rne(mix ? gate * r + (1.f - gate) * local[i] : r);
  }
}

}  // namespace

hipError_t launch_prefill_mfma(const DeviceView& dv, int layer, bool narrow, bool mix, const SeqCounts& seqs, const SeqOrder& order, int n_seqs,
                               const int32_t* len_in, int32_t* len_out, const void* q, const void* k, const void* v, void* out, int stride_tokens,
                               int max_tokens, float scale_log2, char* staging, int staging_tiles, int n_split, float* split_out,
                               int dealt_rows, const uint8_t* mask_row, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (n_split < 1 || !split_out || (mix && !narrow)) n_split = 1;
  const int per_block = kPrefillWaves * 16 * (narrow ? 1 : 2) / dv.group;     // chunk positions per workgroup
  const int gx = (max_tokens + per_block - 1) / per_block;
  PrefillGrid grid = {};
  int32_t n_heads[2] = {0, 0};
  grid.heads_given = dv.n_kv_heads <= kPrefillArgHeads;
  uint64_t full_heads = 0;
  for (int i = 0; i < dv.n_kv_heads; ++i) {
    const int cls = mask_row[i] ? 0 : 1;
    if (grid.heads_given) full_heads |= (uint64_t)(cls == 0) << i;
    if (grid.heads_given) grid.head[cls][n_heads[cls] >> 3] |= (uint64_t)i << ((n_heads[cls] & 7) * 8);
    ++n_heads[cls];
  }
  grid.n_split = n_split;
  grid.inv_group = (65536 + dv.group - 1) / dv.group;
  grid.inv_scale = scale_log2 > 0.f ? 1.f / scale_log2 : 1.f;
  const int64_t items = plan_prefill_items(per_block, n_seqs, order.in_args && n_split == 1 ? order.tok : nullptr, gx, n_heads, dealt_rows,
                                           &grid.items, grid.first);
  const int tiles = (max_tokens + kTile - 2) / kTile + 1;      // (a full head's chunk may start anywhere in a tile)
  hipLaunchKernelGGL(place_chunk_kernel, dim3(tiles, dv.n_kv_heads, dv.batch), dim3(kBlock), 0, stream, dv, layer, seqs, len_in, len_out,
                     (const uint16_t*)k, (const uint16_t*)v, stride_tokens, staging, staging_tiles, full_heads);
  if (hipError_t e = hipGetLastError()) return e;
  const int64_t heavy_rows = (int64_t)n_seqs * n_heads[0];
  const dim3 blocks((uint32_t)(items + (n_split - 1) * heavy_rows * gx)), block(kPrefillBlock);
#define RLKV_LAUNCH(PG, NGR, MX)                                                                                          \
  hipExtLaunchKernelGGL((prefill_mfma_kernel<PG, NGR, MX>), blocks, block, 0, stream, ev_start, ev_stop, 0, dv, layer, order, len_in, \
                        (const uint16_t*)q, (uint16_t*)out, stride_tokens, scale_log2, (const char*)staging,       \
                        staging_tiles, split_out, grid)
  // (Layers that do not blend in an instance of their own in either form: the one-group form, which used to carry the blending code
  // along, 8 x 291 .. 868 tokens 77.9 -> 76.2 us, 5 x 2735 .. 3469 728 -> 706, one of 2670 in chunks of 512 239.1 -> 240.3.)
#define RLKV_FORM(PG, NGR) do { if (mix) RLKV_LAUNCH(PG, NGR, true); else RLKV_LAUNCH(PG, NGR, false); } while (0)
#define RLKV_PICK(PG) do { if (narrow) RLKV_FORM(PG, 1); else RLKV_FORM(PG, 2); } while (0)
  if (dv.page_shift >= 0) RLKV_PICK(true); else RLKV_PICK(false);
#undef RLKV_PICK
#undef RLKV_FORM
#undef RLKV_LAUNCH
  if (hipError_t e = hipGetLastError()) return e;
  if (n_split > 1 && heavy_rows > 0) {
    const dim3 mgrid(gx, (uint32_t)heavy_rows, kSplitCols / (narrow ? 2 : 1) / kMergeColsPerGroup), mblock(kSplitCols);
    if (narrow)
      hipLaunchKernelGGL(prefill_merge_kernel<true>, mgrid, mblock, 0, stream, dv, layer, order, (const float*)split_out, n_split,
                         (uint16_t*)out, stride_tokens, grid);
    else
      hipLaunchKernelGGL(prefill_merge_kernel<false>, mgrid, mblock, 0, stream, dv, layer, order, (const float*)split_out, n_split,
                         (uint16_t*)out, stride_tokens, grid);
  }
  return hipGetLastError();
}

}  // namespace rlkv
