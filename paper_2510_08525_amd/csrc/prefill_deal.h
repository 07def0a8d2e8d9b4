// Which (sequence, head, query block) a workgroup of a prefill attention launch works on, given its linear index.
// Shared by the kernel and the host-side planning entry points (which exist so that this arithmetic can be
// checked without a GPU).
#pragma once
#include <hip/hip_runtime.h>

namespace rlkv {

// n / d for 0 <= n < 2^31, inv = quotient_inverse(d): the product is at most n / d and less than 1/2 + 1/2 below it, so one
// correction makes it exact.  (Six scalar instructions; a division is about thirty vector ones, one behind the other.)
__host__ __device__ inline uint32_t quotient_inverse(int d) { return 0xffffffffu / (uint32_t)(d > 0 ? d : 1); }
__host__ __device__ inline int quotient(int n, int d, uint32_t inv) {
  const int q = (int)(((uint64_t)(uint32_t)n * inv) >> 32);
  return n - q * d >= d ? q + 1 : q;
}

// The items of a launch: the heavy ones (full heads of the sequences that have a chunk) and the light ones (compressed heads),
// each class numbered sequence by sequence (long to short), within a sequence head by head (a row: the query blocks of one
// sequence and head), within a row block by block.  Sequences have up to `gx` blocks; only blocks that hold queries are items
// (unless `gx` is taken for all, `ragged` 0), because the hardware deals workgroups not only to the 8 XCDs but also to the
// 4 shader engines of each strictly in turn, and an engine whose turn it is keeps the others waiting: with 488 of 928
// workgroups empty, engines of 8 CUs had 12 to 18 that were not, three rounds of work instead of two.
struct PrefillItems {
  int32_t gx;
  int32_t dealt[2];      // [heavy, light] rows, from the first on, that go one row per XCD: a multiple of 8, of gx blocks each
  int32_t rest;          // heavy items that do not
  int32_t heads[2];      // full, compressed heads of the layer
  int32_t n_seqs;        // sequences that have a chunk
  int32_t ragged;        // 1: a sequence's blocks are those `first` gives it; 0: all have gx (those without queries do nothing)
  uint32_t inv_gx, inv_heads[2], inv_seq[2];     // quotient_inverse of gx, heads and heads * gx
};
// Blocks of the sequences before each place in the order ([n_seqs + 1], then INT32_MAX), looked at where `ragged` is 1.
constexpr int kFirstEntries = 129;

// Workgroups are dealt to the 8 XCDs in turn by their linear index, and each XCD has an L2 of its own.  All the
// workgroups of a row read the same tiles, so whole rows are kept on one XCD where that leaves the XCDs equally loaded.
// Each XCD takes, in this order: its rows of the dealt heavy rows (row y on XCD y % 8); its eighth of the other heavy
// items, dealt one by one; its rows of the dealt light rows, likewise; its eighth of the other light items.  The two parts
// dealt one by one form one list dealt in turn, so every XCD ends up with exactly the workgroups the hardware hands it:
// a bijection for any counts.  Returns whether workgroup `lin` has a heavy item, and its number in the class.
__host__ __device__ inline bool prefill_item(int lin, const PrefillItems& p, int& index) {
  const int k = lin & 7;
  const int c_a = (p.dealt[0] >> 3) * p.gx, c_c = (p.dealt[1] >> 3) * p.gx;     // items of whole rows per XCD of either class
  const int c_b = (p.rest - k + 7) >> 3;                // how many of the heavy ones dealt one by one come to this XCD
  const int i = lin >> 3;
  const bool heavy = i < c_a + c_b;
  const int i_class = heavy ? i : i - c_a - c_b;        // the XCD's items of the class before it
  const bool by_rows = i_class < (heavy ? c_a : c_c);
  const int row = quotient(i_class, p.gx, p.inv_gx);
  const int of_rows = (row * 8 + k) * p.gx + (i_class - row * p.gx);
  const int one_by_one = heavy ? p.dealt[0] * p.gx + (i - c_a) * 8 + k
                               : p.dealt[1] * p.gx + (i - c_a - c_c) * 8 + k - p.rest;   // the dealt list goes on with the light items left over
  index = by_rows ? of_rows : one_by_one;
  return heavy;
}

// Item `index` of a class with `heads` heads a sequence: the sequence's place in the order, the head's number in its class and
// the block counted from the row's end (later query blocks have more keys under the causal mask and go first).
// Even launch: every sequence has gx blocks.
__host__ __device__ inline void even_place(int index, bool full, const PrefillItems& p, int& place, int& head, int& block) {
  const int per_seq = (full ? p.heads[0] : p.heads[1]) * p.gx;
  place = quotient(index, per_seq, full ? p.inv_seq[0] : p.inv_seq[1]);
  const int r = index - place * per_seq;
  head = quotient(r, p.gx, p.inv_gx);
  block = r - head * p.gx;
}
// Ragged launch: index / heads is a block of the sequence with first[place] <= it < first[place + 1]; `at` = first[place],
// `blocks` those of the sequence.  The head is a quotient below 2^16: in fp32, taken a little low (the reciprocal is good to
// 2^-22), it is the right one or one less.
__host__ __device__ inline void ragged_place(int index, int heads, int at, int blocks, int& head, int& block) {
  const int r = index - at * heads;
#ifdef __HIP_DEVICE_COMPILE__
  const float inv = __builtin_amdgcn_rcpf((float)blocks);
  head = __builtin_amdgcn_readfirstlane((int)((float)r * (inv * (1.f - 0x1p-20f))));
#else
  head = (int)((float)r * (1.f / (float)blocks * (1.f - 0x1p-20f)));
#endif
  block = r - head * blocks;
  if (block >= blocks) {
    ++head;
    block -= blocks;
  }
}

}  // namespace rlkv
