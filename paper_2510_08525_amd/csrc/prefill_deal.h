// Which (sequence, head, query block) a workgroup of a prefill attention launch works on, given its linear index.
// Shared by the kernel and the host-side planning entry points (which exist so that this arithmetic can be
// checked without a GPU).
#pragma once
#include <hip/hip_runtime.h>

namespace rlkv {

// The items of a launch: the heavy ones (full heads of the sequences that have a chunk) and the light ones (compressed heads),
// each class numbered sequence by sequence (long to short), within a sequence head by head (a row: the query blocks of one
// sequence and head), within a row block by block.  Sequences have up to `gx` blocks; only blocks that hold queries are items
// (unless `gx` is taken for all, see PrefillGrid::ragged), because the hardware deals workgroups not only to the 8 XCDs but also to the
// 4 shader engines of each strictly in turn, and an engine whose turn it is keeps the others waiting: with 488 of 928
// workgroups empty, engines of 8 CUs had 12 to 18 that were not, three rounds of work instead of two.
struct PrefillItems {
  int32_t gx;
  int32_t dealt[2];      // [heavy, light] rows, from the first on, that go one row per XCD: a multiple of 8, of gx blocks each
  int32_t rest;          // heavy items that do not
};

// Workgroups are dealt to the 8 XCDs in turn by their linear index, and each XCD has an L2 of its own.  All the
// workgroups of a row read the same tiles, so whole rows are kept on one XCD where that leaves the XCDs equally loaded.
// Each XCD takes, in this order: its rows of the dealt heavy rows (row y on XCD y % 8); its eighth of the other heavy
// items, dealt one by one; its rows of the dealt light rows, likewise; its eighth of the other light items.  The two parts
// dealt one by one form one list dealt in turn, so every XCD ends up with exactly the workgroups the hardware hands it:
// a bijection for any counts.  Returns whether workgroup `lin` has a heavy item, and its number in the class.
__host__ __device__ inline bool prefill_item(int lin, const PrefillItems& p, int& index) {
  const int k = lin & 7;
  int i = lin >> 3;
  const int c_a = (p.dealt[0] >> 3) * p.gx, c_c = (p.dealt[1] >> 3) * p.gx;     // items of whole rows per XCD of either class
  const int c_b = (p.rest - k + 7) >> 3;                // how many of the heavy ones dealt one by one come to this XCD
  if (i < c_a) { const int row = i / p.gx; index = (row * 8 + k) * p.gx + (i - row * p.gx); return true; }
  i -= c_a;
  if (i < c_b) { index = p.dealt[0] * p.gx + i * 8 + k; return true; }
  i -= c_b;
  if (i < c_c) { const int row = i / p.gx; index = (row * 8 + k) * p.gx + (i - row * p.gx); return false; }
  i -= c_c;
  index = p.dealt[1] * p.gx + (c_b + i) * 8 + k - p.rest;     // the dealt list goes on with the light items left over
  return false;
}

// Item `index` of a class with `heads` heads a sequence: the sequence's place in the order, the head's number in its class and
// the block counted from the row's end (later query blocks have more keys under the causal mask and go first).
// `first` [n_seqs + 1]: blocks of the sequences before each place; `ragged` 0: not looked at, every sequence has gx.
__host__ __device__ inline void prefill_place(int index, int heads, int gx, bool ragged, const int32_t* first, int n_seqs, int& place,
                                              int& head, int& block) {
  int at = 0, blocks = gx;
  if (ragged) {
    const int x = index / heads;                        // first[place] <= x < first[place + 1]
    int lo = 0, hi = n_seqs;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (first[mid] <= x) lo = mid; else hi = mid;
    }
    place = lo;
    at = first[lo];
    blocks = first[lo + 1] - at;
  } else {
    place = index / (heads * gx);
    at = place * gx;
  }
  const int r = index - at * heads;
  head = r / blocks;
  block = r - head * blocks;
}

}  // namespace rlkv
