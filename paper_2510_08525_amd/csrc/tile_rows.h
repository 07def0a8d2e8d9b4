// Row-major K/V rows -> one 32-slot tile of the MFMA-operand layout (rlkv_internal.h), by one workgroup.  Used by the
// multi-token append and by the placing of a prefill chunk.
//
// Bound: HBM, 16 KiB read and 16 KiB written per tile.  Both sides of the copy want whole lines and the layouts differ
// (the tile's V is transposed in 2-byte elements), so a tile passes through LDS: rows come in with 16-byte loads, K and
// V of a row side by side, and the tile goes out with 16-byte stores, a contiguous kilobyte per wavefront.
// Measured: append of 32 prompts of 1000 .. 6000 tokens, 4 of 8 heads full, in chunks of 1024: 23.9 us per launch on
// average (3.8 TB/s read + written) against 44.7 us when V was gathered element by element from memory; the placing
// of a prefill chunk of 16 x 2048 tokens, 4 heads: 24.7 us (5.4 TB/s).
#pragma once

#include "rlkv_internal.h"

namespace rlkv {

constexpr int kTileRowStride = 272;      // bytes of a V row in LDS: 16 more than the row, so that the transposed reads of a
                                         // wavefront (4 k-groups 4 rows apart, 16 columns) fall into different banks
struct TileRowsLds {
  uint4 k[kTile * 16];                   // the tile's K image; the 16 units of a chunk rotated by the chunk (bank conflicts)
  alignas(16) char v[kTile * kTileRowStride];
};

__device__ __forceinline__ bool any_beyond_fp16(uint32_t two) { return bf16_beyond_fp16(two) || bf16_beyond_fp16(two >> 16); }

// (NT: past the caches.  An append's tiles are not read before the next decode step: import of 32 prompts 211.2 -> 208.6 us.  The
// tiles of a prefill chunk are read by the attention launch behind them.)
typedef uint32_t row_x4 __attribute__((ext_vector_type(4)));
template <bool NT> __device__ __forceinline__ uint4 row_load(const uint16_t* p) {
  if (!NT) return *reinterpret_cast<const uint4*>(p);
  const row_x4 v = __builtin_nontemporal_load(reinterpret_cast<const row_x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool NT> __device__ __forceinline__ void tile_store(char* p, const uint4& u) {
  if (!NT) { *reinterpret_cast<uint4*>(p) = u; return; }
  const row_x4 v = {u.x, u.y, u.z, u.w};
  __builtin_nontemporal_store(v, reinterpret_cast<row_x4*>(p));
}

// row_of(slot): the slot's source row, -1 = none.  keep(slot): the slot keeps what it holds (it has no source row); the others
// without one are written as zeros.  k_rows / v_rows: row 0 of the pair (row r at r * kHeadDim).  Returns whether this thread moved a V
// value beyond the fp16 range.
template <bool NT, typename RowOf, typename Keep>
__device__ __forceinline__ bool rows_to_tile(TileRowsLds& lds, const RowOf& row_of, const Keep& keep, const uint16_t* __restrict__ k_rows,
                                             const uint16_t* __restrict__ v_rows, char* __restrict__ tile_base) {
  constexpr int kUnits = kTile * 16 / kBlock;            // 16-byte units of K (and of V) per thread
  const int tid = threadIdx.x;
  const bool v_aligned = (reinterpret_cast<uintptr_t>(v_rows) & 15) == 0;    // (a caller's V may start at any element)
  uint4 kv[kUnits], vv[kUnits];
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {
    const int u = tid + i * kBlock, row = row_of(u >> 4), chunk = u & 15;
    kv[i] = vv[i] = make_uint4(0, 0, 0, 0);
    if (row >= 0) {
      kv[i] = row_load<NT>(k_rows + (int64_t)row * kHeadDim + chunk * 8);
      const uint16_t* v = v_rows + (int64_t)row * kHeadDim + chunk * 8;
      if (v_aligned) {
        vv[i] = row_load<NT>(v);
      } else {
        vv[i] = make_uint4(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16, v[4] | (uint32_t)v[5] << 16,
                           v[6] | (uint32_t)v[7] << 16);
      }
    }
  }
  bool wide = false;
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {
    const int u = tid + i * kBlock, slot = u >> 4, chunk = u & 15;
    lds.k[(slot >> 4) * 256 + chunk * 16 + ((slot + chunk) & 15)] = kv[i];
    *reinterpret_cast<uint4*>(lds.v + slot * kTileRowStride + chunk * 16) = vv[i];
    wide |= any_beyond_fp16(vv[i].x) || any_beyond_fp16(vv[i].y) || any_beyond_fp16(vv[i].z) || any_beyond_fp16(vv[i].w);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {                     // K: unit u of the tile = [half][chunk][slot % 16]
    const int u = tid + i * kBlock, hf = u >> 8, chunk = (u >> 4) & 15, s16 = u & 15;
    if (!keep(hf * 16 + s16))
      tile_store<NT>(tile_base + u * 16, lds.k[hf * 256 + chunk * 16 + ((s16 + chunk) & 15)]);
  }
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {                     // V: unit u = [d / 16][kb][d % 16], eight slots of one d
    const int u = tid + i * kBlock, kb = (u >> 4) & 3, d = (u >> 6) * 16 + (u & 15);
    uint32_t val[8];
    unsigned have = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int slot = (e >> 2) * 16 + kb * 4 + (e & 3);
      val[e] = *reinterpret_cast<const uint16_t*>(lds.v + slot * kTileRowStride + d * 2);
      have |= keep(slot) ? 0u : 1u << e;
    }
    char* dst = tile_base + kTileBytes / 2 + u * 16;
    if (have == 0xffu) {
      tile_store<NT>(dst, make_uint4(val[0] | val[1] << 16, val[2] | val[3] << 16, val[4] | val[5] << 16, val[6] | val[7] << 16));
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (have & (1u << e)) reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)val[e];
    }
  }
  return wide;
}

}  // namespace rlkv
