// Internal definitions shared by the host API and the gfx950 kernels of librlkv.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "rlkv.h"

namespace rlkv {

constexpr int kTile = 32;          // tokens per scheduling tile (and per MFMA step)
constexpr int kHeadDim = 128;      // the only head_dim the kernels are written for
constexpr int kMaxGroup = 16;      // query heads per KV head
constexpr int kMaxWorkgroups = 2048;  // upper bound of the split-K grid (sizes the scratch)
constexpr int kBlock = 256;        // threads per workgroup (4 wavefronts)
constexpr int kRound = 4;          // tiles per scheduling unit (what a row-major workgroup works at a time up to group 8, half of that of a tiled one)
constexpr int kPairOverheadUnits = 1;  // units at the head of every pair that carry no tiles (a label for its start)
constexpr int kRoundCost = 2;          // cost model of the share partition, in half rounds: one round of tiles ...
constexpr int kPairStartCost = 3;      // ... and the start of a pair (pipeline restart on a new store, Q load,
                                       // merge, output write): about 1.5 rounds, from per-workgroup timestamps
constexpr int kWorklistSlack = 32; // tokens a work list stays valid for after it was built

// Work-list records, written by the host (share_plan.hip, ensure_worklist) and read by the attention and merge
// kernels with wave-uniform (scalar) loads.  A workgroup's record embeds the record of its
// first pair, so one load level separates the kernel start from the first K/V tile load.
// The list of a layer is one block of device memory, [ListHeader][WgDesc x n_wg][PairDesc x n_pairs], written by
// one kernel (launch_fetch) that reads a pinned staging slot of the same layout.
struct ListHeader {      // 64 bytes
  int32_t grow;          // tokens every active sequence has gained since the list was planned.  A new list brings
                         // 0; a fused step advances it by 1 (the merge kernel behind it, or, where there is
                         // none, the attention kernel itself), a uniform multi-token append by its
                         // token count, so that a decode launch needs no per-step argument and a captured step can
                         // be replayed
  int32_t pad[15];
};
struct PairDesc {        // 40 bytes
  int64_t koff;          // byte offset of the pair's K store from kv_base
  int32_t cap;           // token capacity of the store (the V store starts cap rows later)
  int32_t n_build;       // cached tokens of the sequence when the list was built
  int32_t unit_start;    // first scheduling unit of the pair in the end-to-end numbering
  int32_t unit_end;      // one past its last unit.  The first kPairOverheadUnits units of a pair hold
                         // no tiles; every later unit is WgDesc::round_tiles consecutive tiles of its store
  int32_t wg_first;      // first workgroup that holds units of the pair; its partial slots are wg + pair index
  int32_t ring;          // -1 = full head; of a compressed one its number among the compressed (layer, head)s, which is
                         // where its slot positions are: slot_pos + (ring * batch + sequence) * window
  float gate;            // Eq. 1 gate of a full head: out = gate * full + (1 - gate) * local; 1 = plain
  int32_t n_seg;         // workgroups that hold units of the pair (wg_first .. wg_first + n_seg - 1)
};
struct WgDesc {          // 64 bytes: one line, one scalar load
  int32_t first_pair;    // pair that holds the workgroup's first tile
  int32_t u_begin, u_end;  // the workgroup's share of units [u_begin, u_end); empty if u_begin >= u_end
  int32_t seq;           // sequence and head of that pair
  PairDesc first;        // copy of pair_desc[first_pair]
  int32_t head;
  int32_t round_tiles;   // tiles of a unit (kRound, or half of it: short fp32 lists)
};
static_assert(sizeof(ListHeader) == 64 && sizeof(PairDesc) == 40 && sizeof(WgDesc) == 64, "the kernels load these word by word");

// Everything a kernel needs to find its data; passed by value as a kernel argument.
struct DeviceView {
  int32_t n_layers, n_q_heads, n_kv_heads, group, batch;
  int32_t sink, recent, window;   // window = sink + recent
  int32_t window_pad;             // window rounded up to a whole tile
  int32_t dtype, kernel;
  int32_t row_bytes;              // head_dim * element size
  int32_t n_pairs;                // batch * n_kv_heads
  int32_t n_wg;                   // grid size of the split-K kernel

  const uint8_t* full_mask;       // [n_layers][n_kv_heads]
  uint8_t* active;                // [batch] 1 = the slot takes part in uniform appends and in decode
  float* gate;                    // [n_layers][n_kv_heads] Eq. 1 gates (1 = plain full attention)
  const int64_t* store_off;       // [n_layers][batch][n_kv_heads] byte offset of the K store
  const int32_t* cap_pad;         // [batch] padded token capacity of a full store
  const int64_t* slotpos_off;     // [n_layers][n_kv_heads] element offset into slot_pos, -1 = full
  int32_t* len;                   // [2][n_layers][batch] cached tokens, double buffered: a kernel that
                                  // appends reads one copy and writes the other, so no workgroup
                                  // can see a length another one has already advanced
  int32_t* slot_pos;              // per compressed (layer, head): [batch][window]
  int32_t* v_wide;                // [n_layers] 1 once a V value of magnitude >= 65536 (or Inf / NaN) has gone into the
                                  // layer's stores or staging (tiled layout): prefill then takes V as bf16
  int32_t* append_cnt;            // [2][batch] per-sequence token counts; sequence order of a prefill (batches beyond kArgSeqs)
  char* list_base;                // [n_layers] work-list blocks of list_stride bytes (see ListHeader)
  int64_t list_stride;
  int32_t list_pair_off;          // byte offset of the PairDesc array inside a block
  float* part_o;                  // [n_wg + n_pairs][group][head_dim]
  float* part_m;                  // [n_wg + n_pairs][group]  (log2 domain maxima)
  float* part_l;                  // [n_wg + n_pairs][group]
  int64_t part_set_o, part_set_ml; // element offsets of the second partial set (local attention of gated heads)
  int32_t* arrived;               // [n_layers][n_pairs][kMaxGroup / 2] workgroups that have left their partials of a pair's
                                  // two heads, 0 between launches
  char* kv_base;                  // start of the K/V stores

  // Paged full heads (Sec. 4.3).  store_off of a full head is then the offset of its pool, the
  // same for every sequence, and tile t of sequence b lives at
  //   pool + block_table[b][t >> page_shift] * page_bytes + (t & page_mask) * kTileBytes.
  int32_t page_shift;             // log2(tiles per page); -1 = contiguous stores
  int32_t page_mask;              // tiles per page - 1
  int32_t table_stride;           // block-table entries per sequence
  int64_t page_bytes;             // bytes of one page (K and V)
  int32_t* block_table;           // [batch][table_stride] page index, shared by all layers and heads
};

// Block-table entries that change, passed by value to a one-block kernel (no host-to-device copy
// on the append path).
constexpr int kTableUpdateMax = 96;
struct TableUpdates {
  int32_t n;
  int32_t index[kTableUpdateMax];   // element index into block_table
  int32_t value[kTableUpdateMax];   // page
};

// Per-sequence token counts of a ragged append or a prefill chunk, and the prefill's sequence order: by value in the
// kernel arguments, which costs the stream nothing.  (A copy through pinned memory took 10 us of it per call: 4.2 us of
// copy and a 5.6 us gap behind it.)  A batch beyond kArgSeqs has them written to dv.append_cnt by a kernel first.
constexpr int kArgSeqs = 128;
struct SeqCounts {
  int32_t in_args;                  // 1: the arrays below hold them, 0: dv.append_cnt does
  int32_t tok[kArgSeqs];            // [sequence]
};
// The same in the order in which a prefill's grid takes the sequences (a workgroup asks for both words at once).
struct SeqOrder {
  int32_t in_args;
  int32_t seq[kArgSeqs];            // [place in the order]
  int32_t tok[kArgSeqs];
};
// (the same in all lanes; readfirstlane because the compiler loads through a pointer that is one or the other, takes the
// result for a lane's own, and everything computed from it with it: 12 % on the blending prefill)
__device__ inline int tokens_of_seq(const DeviceView& dv, const SeqCounts& seqs, int b) {
  return __builtin_amdgcn_readfirstlane(seqs.in_args ? seqs.tok[b] : dv.append_cnt[b]);
}
__device__ inline void seq_in_order(const DeviceView& dv, const SeqOrder& order, int i, int& b, int& tokens) {
  if (order.in_args) {
    b = order.seq[i];
    tokens = order.tok[i];
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+s"(b), "+s"(tokens));          // (both asked for here: not through a pointer that is this one or the other)
#endif
  } else {
    b = dv.append_cnt[dv.batch + i];
    tokens = dv.append_cnt[b];
  }
  b = __builtin_amdgcn_readfirstlane(b);
  tokens = __builtin_amdgcn_readfirstlane(tokens);
}

// ---- store addressing ------------------------------------------------------------
// Row-major layout (VALU kernel): row `slot` of K (or V) at slot * row_bytes.
//
// Tiled layout (MFMA kernel, bf16): the store is cut into tiles so that lane l of a
// wavefront reading 16 bytes at tile_base + step * 1024 + l * 16 receives exactly its
// MFMA operand:
//   K, per 16 slots (4 KiB, two per tile):  [chunk = d / 8 : 16][slot % 16 : 16][d % 8 : 8]
//      -> step s in 0..3 covers chunks 4s..4s+3; lane l = (chunk % 4) * 16 + slot % 16
//         holds row slot%16, k-group chunk%4 of a 16x16x32 A operand.
//   V, per 32 slots (8 KiB):  [dblk = d / 16 : 8][kb : 4][d % 16 : 16][e : 8]
//      with slot % 32 = half * 16 + kb * 4 + r and e = half * 4 + r
//      -> step dblk; lane l = kb * 16 + d % 16 holds column d%16, k-group kb of a
//         16x16x32 B operand whose k index runs over the 32 slots of the tile in the
//         same order the score tile leaves them in the accumulator registers.
// K and V tiles of the same 32 slots sit next to each other (16 KiB: K then V), so the 16
// loads a wavefront issues per tile fall into one contiguous block.  Rows are brought into this order by rows_to_tile
// (tile_rows.h) and by the append of a fused step (decode_mfma.hip).
constexpr int kTileBytes = 16384;

// bf16 bits whose value lies beyond the fp16 range (exponent field >= 127 + 16; Inf and NaN included)
__host__ __device__ inline bool bf16_beyond_fp16(uint32_t bits) { return (bits & 0x7f80u) >= 0x4780u; }

// The parts of a layer's work-list block.
__host__ __device__ inline ListHeader* list_header(const DeviceView& dv, int layer) {
  return reinterpret_cast<ListHeader*>(dv.list_base + layer * dv.list_stride);
}
__host__ __device__ inline WgDesc* wg_desc_of(const DeviceView& dv, int layer) {
  return reinterpret_cast<WgDesc*>(dv.list_base + layer * dv.list_stride + sizeof(ListHeader));
}
__host__ __device__ inline PairDesc* pair_desc_of(const DeviceView& dv, int layer) {
  return reinterpret_cast<PairDesc*>(dv.list_base + layer * dv.list_stride + dv.list_pair_off);
}

// The list of a launch is not written while the launch runs, so it is read through the constant address space: scalar loads, in a
// kernel that stores too (else the compiler takes it for possibly changed, loads it through vector registers and waits at
// once, for every load before it as well).
#define RLKV_CONST const __attribute__((address_space(4)))
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x8 __attribute__((ext_vector_type(8), aligned(8)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));
template <typename T>
__device__ __forceinline__ T load_const(const void* p) { return *(RLKV_CONST T*)(uintptr_t)p; }
__device__ __forceinline__ PairDesc pair_from_words(const i32x8& a, int gate, int n_seg) {
  PairDesc d;
  d.koff = ((int64_t)a[1] << 32) | (uint32_t)a[0];
  d.cap = a[2]; d.n_build = a[3]; d.unit_start = a[4]; d.unit_end = a[5]; d.wg_first = a[6]; d.ring = a[7];
  d.gate = __builtin_bit_cast(float, gate); d.n_seg = n_seg;
  return d;
}
__device__ __forceinline__ PairDesc load_pair(const char* pairs, int pi) {
  const char* at = pairs + (int64_t)pi * (int)sizeof(PairDesc);
  const i32x8 a = load_const<i32x8>(at);
  const i32x2 b = load_const<i32x2>(at + 32);
  return pair_from_words(a, b[0], b[1]);
}
__device__ __forceinline__ WgDesc load_wg(const char* list, int wg) {
  const i32x16 r = load_const<i32x16>(list + sizeof(ListHeader) + (int64_t)wg * (int)sizeof(WgDesc));
  WgDesc d;
  d.first_pair = r[0]; d.u_begin = r[1]; d.u_end = r[2]; d.seq = r[3];
  const i32x8 a = {r[4], r[5], r[6], r[7], r[8], r[9], r[10], r[11]};
  d.first = pair_from_words(a, r[12], r[13]);
  d.head = r[14]; d.round_tiles = r[15];
  return d;
}

// Lengths of `layer` in copy `parity` (0 / 1).
__host__ __device__ inline int32_t* len_of(const DeviceView& dv, int parity, int layer) {
  return dv.len + ((int64_t)parity * dv.n_layers + layer) * dv.batch;
}

// ---- launchers (defined next to their kernels) -------------------------------------
// `len_in` is the current copy of the layer's lengths; kernels that append write the
// advanced lengths to `len_out` (the other copy).  A uniform append also adds its token count to the
// layer's ListHeader::grow.  `seqs` non-null: a ragged append (n_tokens_uniform unused).
hipError_t launch_append(const DeviceView& dv, int layer, const int32_t* len_in, int32_t* len_out,
                         const void* k, const void* v, int n_tokens_uniform, int stride_tokens, const SeqCounts* seqs,
                         int max_tokens, hipStream_t stream);
// Appends a chunk's K/V to the compressed heads of a layer of the tiled layout (behind launch_prefill_mfma, which has appended the
// full heads' and written the lengths).  mask_row (host, [n_kv_heads]): the layer's mask.
hipError_t launch_append_rings(const DeviceView& dv, int layer, const int32_t* len_in, const void* k, const void* v, int stride_tokens,
                               const SeqCounts& seqs, int max_tokens, const uint8_t* mask_row, hipStream_t stream);
// Copies `bytes` (a multiple of 8) from pinned host memory to the device by a kernel that reads them over the bus.
hipError_t launch_fetch(void* dst, const void* pinned_src, size_t bytes, hipStream_t stream);
// Writes n values of host memory to `dst` through kernel arguments.
hipError_t launch_write_values(int32_t* dst, const int32_t* values, int n, hipStream_t stream);
hipError_t launch_reset(const DeviceView& dv, int seq, int64_t slot_pos_elems, hipStream_t stream);
hipError_t launch_table_update(const DeviceView& dv, const TableUpdates& up, hipStream_t stream);
// Host-side plan of the shares (share_plan.hip): rounds[p] = rounds of tiles of pair p (0 = none).
// Fills wg_begin[0 .. n_wg] (share w = units [wg_begin[w], wg_begin[w + 1])), seg_first[p] / seg_count[p]
// (the workgroups that hold units of pair p); returns the number of workgroups used.
// `singly`: one round per workgroup (which the grid must be able to take), whatever else.
int plan_shares(const int32_t* rounds, int n_pairs, int n_wg, int32_t* wg_begin, int32_t* seg_first,
                int32_t* seg_count, bool singly = false);
// The plan of a list of whole pairs, one workgroup each (n_used of them have rounds; at most n_wg do): pairs spread evenly over
// the shares, so that few pairs still meet all XCDs.
void plan_whole_pairs(const int32_t* rounds, int n_pairs, int n_wg, int32_t* wg_begin, int32_t* seg_first,
                      int32_t* seg_count);
// Whether a list of whole pairs is the faster one for sequences of these lengths (see share_plan.hip).
bool wants_whole_pairs(int kernel, int dtype, int group, bool gated, bool step, int n_wg, int n_kv_heads, int n_full, int window,
                       int batch, const int32_t* lengths, const uint8_t* active, bool merged_inside);
bool list_is_whole(int kernel, int dtype, int group, bool gated, bool step, int n_wg, int n_kv_heads, int n_full, int window,
                   int batch, const int32_t* lengths, const uint8_t* active);
// ev_start / ev_stop (both or neither): events that receive the kernel's own begin and end
// timestamps (the dispatch's completion signal), for the measurement aid.
// `gated`: some full head of the layer has a gate below 1 (two passes for those heads).
// k_new / v_new non-null: fused single-token append (rows [batch][n_kv_heads][1][head_dim]); the advanced
// lengths are written to both copies of the length table.
// (The row-major kernel's form that blends does layers without blending heads as well: a recorded launch takes it, since gates may be set
// between replays.)
// `grow` (lists of whole pairs, and with `merge_here`): tokens since the layer's list was planned, as the host knows them; a fused
// launch then also writes the advanced growth counter.  `merge_here`: the last workgroup of a pair merges its partials, no merge launch
// follows.  -1 (a launch that may be replayed, or whose count the host does not know): read from the
// list's header, and a fused launch must be followed by the merge kernel with advance = 1.
hipError_t launch_decode_valu(const DeviceView& dv, int layer, bool gated, const void* q, void* out, float scale_log2,
                              const void* k_new, const void* v_new, int grow, bool merge_here, hipStream_t stream, hipEvent_t ev_start,
                              hipEvent_t ev_stop);
// `in_turn`: shares go to the XCDs in turn instead of in contiguous runs (a list of shares at most half of which hold units).
hipError_t launch_decode_mfma(const DeviceView& dv, int layer, bool gated,
                              const void* q, void* out, float scale_log2, const void* k_new, const void* v_new,
                              int grow, bool merge_here, bool in_turn, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop);
// merge_words (host, [n_pairs], optional): per pair (first partial slot << 12) | partials, as planned for the
// work list now on the device; with it and at most kMergeArgPairs pairs the merge kernel takes these from its
// arguments instead of from the pair records (not for a layer with gates: their records carry more).
// most_partials: of any pair of the list (0 where the launch may run under another list; the kernel's form only).
// advance: tokens to add to the layer's ListHeader::grow (1 behind a fused append + decode launch).
constexpr int kMergeArgPairs = 512;
constexpr int kMergeFew = 32;             // partials of a pair that the merge kernel takes in one go
hipError_t launch_combine(const DeviceView& dv, int layer, void* out, hipStream_t stream, int advance,
                          const uint32_t* merge_words, int most_partials);
// Prefill attention of one chunk (counts in `seqs`, the same in the grid's order in `order`, lengths before the chunk in len_in):
// appends the chunk's K/V of the full heads and stages those of the compressed heads as tiles in `staging` (staging_tiles tiles per
// pair), writes the advanced lengths to len_out, then attends.  Where the layer has compressed heads, launch_append_rings with the
// same chunk follows.
// `narrow`: the kernel form with one column group of queries per wavefront instead of two.  `mix`: some full head of the layer
// blends (Eq. 1: causal and local attention of a full head with a gate below 1).
// `n_split` > 1: the unmasked tiles of every full head's workgroup are divided among
// n_split workgroups, which leave their shares in `split_out` (kPrefillSplitSlotBytes per divided
// workgroup; at most kPrefillSplitSlots: full heads of the sequences that have a chunk x blocks x n_split) for a merge
// kernel that follows.  `n_seqs`: sequences that have a chunk, the first ones of the order.
constexpr int kPrefillSplitSlots = 1024;
constexpr int kPrefillArgHeads = 64;      // KV heads of a layer whose class lists travel in the prefill kernels' arguments
constexpr size_t kPrefillSplitSlotBytes = 256 * (size_t)(kHeadDim + 2) * sizeof(float);
hipError_t launch_prefill_mfma(const DeviceView& dv, int layer, bool narrow, bool mix, const SeqCounts& seqs, const SeqOrder& order, int n_seqs,
                               const int32_t* len_in, int32_t* len_out, const void* q, const void* k, const void* v, void* out, int stride_tokens,
                               int max_tokens, float scale_log2, char* staging, int staging_tiles, int n_split, float* split_out,
                               int dealt_rows, const uint8_t* mask_row /* host, [n_kv_heads]: the layer's mask */,
                               hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop);
// The items of an undivided launch (prefill_deal.h) with `per_block` chunk positions to a block: `tokens` [n_seqs] the chunk lengths
// in the grid's order, or null (not at hand: every sequence has gx blocks); dealt_rows: heavy rows that may go one row
// per XCD (rlkv_plan_prefill_rows).  Fills items and, where items->ragged is 1, first [kFirstEntries]; returns the number of items.
struct PrefillItems;
int64_t plan_prefill_items(int per_block, int n_seqs, const int32_t* tokens, int gx, const int32_t (&n_heads)[2], int dealt_rows,
                           PrefillItems* items, int32_t* first);

// Fewest 32-key tiles a share of a divided prefill workgroup has, where cfg.prefill_min_share_tiles does not say: in the
// form with two column groups per wavefront, in the single-group form, and in that form where heads blend.
constexpr int kShareTiles = 80, kShareTilesNarrow = 26, kShareTilesBlend = 40;
bool plan_blend_narrow(int n_compute_units, int group, int n_full_heads, int batch, const int32_t* n_tokens);
int plan_narrow_split(int n_compute_units, int group, int n_full_heads, int batch, const int32_t* n_tokens,
                      const int32_t* cached, int min_share_tiles);

// Measurement aid: reads `bytes` (whole 16 KiB blocks) of `buf` once with `workgroups` workgroups.
hipError_t launch_stream_read(const void* buf, size_t bytes, void* sink, int workgroups, hipStream_t stream);

// x % d for 0 <= x < 2^31 and 1 <= d by a product: inverse_of(d) is short of 2^32 / d by at most 1, so the quotient it gives is short by
// at most 1.  (A division by a value the compiler does not know is 40 instructions at the start of a launch, whose code is fetched as
// it runs: a step of one fp32 sequence of 1030 tokens, 32 on 8 heads, 8.10 -> 7.86 us.)
inline uint32_t inverse_of(int d) { return 0xffffffffu / (uint32_t)d; }
__host__ __device__ inline int remainder_of(int x, int d, uint32_t inverse) {
  const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)x * inverse) >> 32), rest = (uint32_t)x - q * (uint32_t)d;
  return (int)(rest >= (uint32_t)d ? rest - (uint32_t)d : rest);
}

// ---- small device helpers -----------------------------------------------------------
__device__ inline float bf16_bits_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
__device__ inline uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

}  // namespace rlkv
