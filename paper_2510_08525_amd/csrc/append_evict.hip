// Append + evict: writes the new K/V rows of one layer into the head-mixed cache.
//
// Full heads store position p at row p.  Compressed heads are a fixed-size store of
// `sink` never-evicted slots followed by a ring of `recent` slots (paper Sec. 4.3: fixed
// size circular buffer, sink + local; App. B: only the first-S and recent-R tokens are
// kept): position p < S lives in slot p, position p >= S in slot S + (p - S) mod R, where
// it overwrites position p - R.
//
// The kernel is destination driven: every workgroup owns a tile of slots, asks for each
// "which appended position ends up in this slot?" (the largest one that maps to it), and
// copies that row only (tiled layout: through LDS, tile_rows.h).  A multi-token append therefore writes survivors only and gives
// the same store as the same tokens appended one at a time, whatever the write order.
#include <string.h>
#include <type_traits>

#include "rlkv_internal.h"
#include "tile_rows.h"

namespace rlkv {
namespace {

struct TileRange { int first, count; };

__device__ inline TileRange tiles_of(int slot_lo, int slot_hi /* exclusive */) {
  if (slot_hi <= slot_lo) return {0, 0};
  const int t0 = slot_lo / kTile, t1 = (slot_hi - 1) / kTile;
  return {t0, t1 - t0 + 1};
}

// Appended position that ends in `slot` after the append, or -1 if the slot is untouched.
__device__ inline int source_position(bool full, int slot, int len_old, int len_new, int S, int R) {
  int p;
  if (full || slot < S) {
    p = slot;
  } else {
    const int r = slot - S;
    if (r >= R) return -1;                       // padding slot behind the ring
    const int last = len_new - 1 - S;            // ring index space of the newest position
    if (last < r) return -1;
    p = S + r + R * ((last - r) / R);            // largest p < len_new with (p - S) % R == r
  }
  return (p >= len_old && p < len_new) ? p : -1;
}

// The compressed heads of a layer, in the arguments of an append that is for them only (n < 0: not given, all heads).
struct NoRings {};
struct RingHeads {
  int32_t n;
  int32_t head[kPrefillArgHeads];
};

// RINGS: compressed heads only (ragged); the full heads and the lengths have been seen to.
template <int KERNEL, typename T, bool RINGS>
__global__ __launch_bounds__(kBlock) void append_kernel(DeviceView dv, int layer, const int32_t* __restrict__ len_in,
                                                        int32_t* __restrict__ len_out, const T* __restrict__ k_new,
                                                        const T* __restrict__ v_new, int n_uniform,
                                                        int stride_tokens, int ragged, SeqCounts seqs,
                                                        std::conditional_t<RINGS, RingHeads, NoRings> rings) {
  int b, h;
  bool given = false;                  // the head comes from the list: it is a compressed one
  if constexpr (RINGS) {
    given = rings.n >= 0;
    b = blockIdx.z;
    h = given ? rings.head[blockIdx.y] : (int)blockIdx.y;
  } else {
    b = blockIdx.y / dv.n_kv_heads;
    h = blockIdx.y % dv.n_kv_heads;
  }
  const int job = blockIdx.x;
  const int S = dv.sink, R = dv.recent;
  // a uniform append skips inactive slots; a ragged append states its counts explicitly
  const int n_tok = ragged ? tokens_of_seq(dv, seqs, b) : (dv.active[b] ? n_uniform : 0);
  // lengths are double buffered: read the current copy, the block of (job 0, head 0) writes
  // the advanced length of its sequence to the other copy
  const int len_old = len_in[b];
  if (!RINGS && job == 0 && h == 0 && threadIdx.x == 0) len_out[b] = len_old + n_tok;
  // a uniform append keeps the layer's work list valid: every active sequence has grown by the same count
  if (!RINGS && !ragged && job == 0 && blockIdx.y == 0 && threadIdx.x == 0) list_header(dv, layer)->grow += n_uniform;
  const int len_new = len_old + n_tok;
  const bool full = !given && dv.full_mask[layer * dv.n_kv_heads + h] != 0;

  int tile = -1;
  if (n_tok > 0 && !(RINGS && full)) {
    if (full) {
      const TileRange t = tiles_of(len_old, len_new);
      if (job < t.count) tile = t.first + job;
    } else {
      // up to three slot ranges change: new sinks, and the ring range (which may wrap)
      const TileRange ta = tiles_of(len_old < S ? len_old : S, len_new < S ? len_new : S);
      const int p0 = len_old > S ? len_old : S;
      const int c = len_new - p0;                 // positions that go to the ring
      TileRange tb = {0, 0}, tc = {0, 0};
      if (c >= R) {
        tb = tiles_of(S, S + R);
      } else if (c > 0) {
        const int r0 = (p0 - S) % R;
        const int r1 = r0 + c;
        tb = tiles_of(S + r0, S + (r1 < R ? r1 : R));
        if (r1 > R) tc = tiles_of(S, S + r1 - R);
      }
      int j = job;
      if (j < ta.count) tile = ta.first + j;
      else if ((j -= ta.count) < tb.count) tile = tb.first + j;
      else if ((j -= tb.count) < tc.count) tile = tc.first + j;
    }
  }

  if (tile >= 0) {
    constexpr int kChunks = kHeadDim * sizeof(T) / 16;    // 16-byte chunks per row
    constexpr int kElems = 16 / sizeof(T);                // elements per chunk
    const int64_t koff = dv.store_off[((int64_t)layer * dv.batch + b) * dv.n_kv_heads + h];
    const int cap = full ? dv.cap_pad[b] : dv.window_pad;
    char* kst = dv.kv_base + koff;
    char* vst = kst + (int64_t)cap * dv.row_bytes;    // row-major layout only
    // tiled layout: start of this block's tile (through the block table for a paged full head)
    char* tile_base = kst + (int64_t)tile * kTileBytes;
    if (KERNEL == RLKV_KERNEL_MFMA && full && dv.page_shift >= 0)
      tile_base = kst + dv.block_table[(int64_t)b * dv.table_stride + (tile >> dv.page_shift)] * dv.page_bytes +
                  (int64_t)(tile & dv.page_mask) * kTileBytes;
    const int64_t src_head = ((int64_t)b * dv.n_kv_heads + h) * stride_tokens;
    int32_t* slot_pos = nullptr;
    if (!full) slot_pos = dv.slot_pos + dv.slotpos_off[layer * dv.n_kv_heads + h] + (int64_t)b * dv.window;

    if constexpr (KERNEL == RLKV_KERNEL_MFMA) {
      // which appended row ends in each slot: once per slot, then the rows go through LDS into the tile
      __shared__ TileRowsLds lds;
      __shared__ int32_t src[kTile];
      if (threadIdx.x < kTile) {
        const int slot = tile * kTile + threadIdx.x;
        const int p = source_position(full, slot, len_old, len_new, S, R);
        src[threadIdx.x] = p < 0 ? -1 : p - len_old;
        if (slot_pos && p >= 0) slot_pos[slot] = p;
      }
      __syncthreads();
      const bool wide = rows_to_tile<true>(lds, [&](int slot) { return src[slot]; }, [&](int slot) { return src[slot] < 0; },
                                           k_new + src_head * kHeadDim, v_new + src_head * kHeadDim, tile_base);
      if (wide) dv.v_wide[layer] = 1;        // the prefill kernel takes this layer's V as bf16 from now on
    } else {
      // K and V rows: one 16-byte chunk per unit
      for (int u = threadIdx.x; u < kTile * kChunks; u += kBlock) {
        const int slot = tile * kTile + u / kChunks, chunk = u % kChunks;
        const int p = source_position(full, slot, len_old, len_new, S, R);
        if (p < 0) continue;
        const int64_t src = ((src_head + (p - len_old)) * kHeadDim + chunk * kElems) * sizeof(T);
        const int64_t dst = (int64_t)slot * dv.row_bytes + chunk * 16;
        *reinterpret_cast<uint4*>(kst + dst) = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(k_new) + src);
        *reinterpret_cast<uint4*>(vst + dst) = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(v_new) + src);
        if (slot_pos && chunk == 0) slot_pos[slot] = p;
      }
    }
  }
}

__global__ void reset_kernel(DeviceView dv, int seq, int64_t slot_pos_elems) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n_len = (int64_t)2 * dv.n_layers * dv.batch;     // both copies
  if (i < n_len) {
    if (seq < 0 || i % dv.batch == seq) dv.len[i] = 0;
  }
  if (seq < 0 && i < dv.n_layers) dv.v_wide[i] = 0;     // an empty cache holds no value beyond the fp16 range
  if (i < slot_pos_elems) {
    // slot_pos is [compressed (layer, head)][batch][window]
    const int b = (int)((i / dv.window) % dv.batch);
    if (seq < 0 || b == seq) dv.slot_pos[i] = -1;
  }
}

__global__ void table_update_kernel(DeviceView dv, TableUpdates up) {
  const int i = threadIdx.x;
  if (i < up.n) dv.block_table[up.index[i]] = up.value[i];
}

// Work lists go from their pinned staging slot to the device by this kernel: it reads the slot over the bus with
// system-scope loads (nothing stale from a cache), all of a block's loads in flight before its stores.
// Bound: one bus latency.  The copy engine that hipMemcpyAsync picked for these sizes (15 .. 60 KiB) left the GPU idle for
// 27 .. 50 us around a copy of 5.8 us; this launch takes 4 us, 5 us after its event is recorded.
constexpr int kFetchWords = 8;      // 8-byte words per thread
__global__ __launch_bounds__(kBlock) void fetch_kernel(unsigned long long* __restrict__ dst, const unsigned long long* __restrict__ src,
                                                       int64_t n) {
  const int64_t base = (int64_t)blockIdx.x * kBlock * kFetchWords + threadIdx.x;
  unsigned long long w[kFetchWords];
#pragma unroll
  for (int i = 0; i < kFetchWords; ++i)
    if (base + i * kBlock < n) w[i] = __hip_atomic_load(src + base + i * kBlock, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
#pragma unroll
  for (int i = 0; i < kFetchWords; ++i)
    if (base + i * kBlock < n) dst[base + i * kBlock] = w[i];
}

constexpr int kValuesPerLaunch = 512;
struct ValueBlock { int32_t v[kValuesPerLaunch]; };
__global__ void write_values_kernel(int32_t* __restrict__ dst, ValueBlock values, int n) {
  const int i = threadIdx.x;
  if (i < n) dst[i] = values.v[i];
}

}  // namespace

hipError_t launch_fetch(void* dst, const void* pinned_src, size_t bytes, hipStream_t stream) {
  const int64_t n = (int64_t)(bytes / 8);
  const int64_t per_block = kBlock * kFetchWords;
  hipLaunchKernelGGL(fetch_kernel, dim3((unsigned)((n + per_block - 1) / per_block)), dim3(kBlock), 0, stream,
                     static_cast<unsigned long long*>(dst), static_cast<const unsigned long long*>(pinned_src), n);
  return hipGetLastError();
}

hipError_t launch_write_values(int32_t* dst, const int32_t* values, int n, hipStream_t stream) {
  for (int at = 0; at < n; at += kValuesPerLaunch) {
    const int m = n - at < kValuesPerLaunch ? n - at : kValuesPerLaunch;
    ValueBlock block = {};
    memcpy(block.v, values + at, (size_t)m * sizeof(int32_t));
    hipLaunchKernelGGL(write_values_kernel, dim3(1), dim3(kValuesPerLaunch), 0, stream, dst + at, block, m);
    if (hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

hipError_t launch_table_update(const DeviceView& dv, const TableUpdates& up, hipStream_t stream) {
  if (up.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(table_update_kernel, dim3(1), dim3(kTableUpdateMax), 0, stream, dv, up);
  return hipGetLastError();
}

hipError_t launch_append(const DeviceView& dv, int layer, const int32_t* len_in, int32_t* len_out,
                         const void* k, const void* v, int n_tokens_uniform, int stride_tokens, const SeqCounts* seqs,
                         int max_tokens, hipStream_t stream) {
  const SeqCounts none = {};
  const SeqCounts& sq = seqs ? *seqs : none;
  const int ragged = seqs != nullptr;
  // Tiles a pair can touch: a range of c >= 1 slots touches at most (c + 30) / 32 + 1 tiles;
  // a full head has one range, a compressed head up to three (new sinks, ring, wrapped
  // ring) whose sizes add up to at most max_tokens.  One token touches one tile.
  const int jobs = max_tokens <= 1 ? 1 : (max_tokens + 3 * (kTile - 2)) / kTile + 3;
  const dim3 grid(jobs, dv.n_pairs), block(kBlock);
  if (dv.dtype == RLKV_F32) {
    hipLaunchKernelGGL((append_kernel<RLKV_KERNEL_VALU, float, false>), grid, block, 0, stream, dv, layer,
                       len_in, len_out, (const float*)k, (const float*)v, n_tokens_uniform, stride_tokens, ragged, sq, NoRings{});
  } else if (dv.kernel == RLKV_KERNEL_MFMA) {
    hipLaunchKernelGGL((append_kernel<RLKV_KERNEL_MFMA, uint16_t, false>), grid, block, 0, stream, dv, layer,
                       len_in, len_out, (const uint16_t*)k, (const uint16_t*)v, n_tokens_uniform, stride_tokens, ragged, sq, NoRings{});
  } else {
    hipLaunchKernelGGL((append_kernel<RLKV_KERNEL_VALU, uint16_t, false>), grid, block, 0, stream, dv, layer,
                       len_in, len_out, (const uint16_t*)k, (const uint16_t*)v, n_tokens_uniform, stride_tokens, ragged, sq, NoRings{});
  }
  return hipGetLastError();
}

hipError_t launch_append_rings(const DeviceView& dv, int layer, const int32_t* len_in, const void* k, const void* v, int stride_tokens,
                               const SeqCounts& seqs, int max_tokens, const uint8_t* mask_row, hipStream_t stream) {
  RingHeads rings = {};
  int n = 0;
  for (int h = 0; h < dv.n_kv_heads; ++h) {
    if (mask_row[h]) continue;
    if (n < kPrefillArgHeads) rings.head[n] = h;
    ++n;
  }
  if (n == 0) return hipSuccess;
  rings.n = n <= kPrefillArgHeads ? n : -1;
  const int rows = n <= kPrefillArgHeads ? n : dv.n_kv_heads;
  // Tiles a compressed pair can touch (launch_append), and no more than its three ranges have.
  const int slots = max_tokens < dv.window ? max_tokens : dv.window;
  const int jobs = (slots + 3 * (kTile - 2)) / kTile + 3;
  hipLaunchKernelGGL((append_kernel<RLKV_KERNEL_MFMA, uint16_t, true>), dim3(jobs, rows, dv.batch), dim3(kBlock), 0, stream, dv, layer,
                     len_in, (int32_t*)nullptr, (const uint16_t*)k, (const uint16_t*)v, 0, stride_tokens, 1, seqs, rings);
  return hipGetLastError();
}

hipError_t launch_reset(const DeviceView& dv, int seq, int64_t slot_pos_elems, hipStream_t stream) {
  int64_t n = (int64_t)2 * dv.n_layers * dv.batch;
  if (slot_pos_elems > n) n = slot_pos_elems;
  if (n == 0) return hipSuccess;
  const int block = 256;
  hipLaunchKernelGGL(reset_kernel, dim3((unsigned)((n + block - 1) / block)), dim3(block), 0, stream, dv, seq,
                     slot_pos_elems);
  return hipGetLastError();
}

}  // namespace rlkv
