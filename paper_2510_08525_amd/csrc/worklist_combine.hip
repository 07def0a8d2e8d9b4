// Split-K merge for decode attention over the head-mixed cache.
//
// A workgroup of the attention kernel whose share does not cover a whole pair leaves one partial
// (m, l, O) per pair it touches, in slot (workgroup index + pair index).  The workgroups of a pair
// are consecutive, and this kernel walks them in ascending order, so the result is deterministic.
#include <string.h>
#include <type_traits>

#include "share_merge.h"

namespace rlkv {
namespace {

// One block per (pair, query head of the group), one thread per output dimension.
//
// The kernel is a chain of memory latencies (words or record, partials, output) and little else: what it needs of the partials'
// place is in its first arguments, which are in registers when it starts (decode_mfma.hip), every load of a pair is asked for before
// anything is waited for, and the usual case, a handful of partials, has neither LDS nor a barrier.
//
// IN_ARGS (a layer without gates, at most kMergeArgPairs pairs): what the kernel needs of a pair's record
// - its first partial slot and its number of partials - comes as one word per pair among the kernel
// arguments instead of from the record in memory, which takes one memory latency out.
struct MergeWords {
  uint32_t w[kMergeArgPairs];     // (first slot << 12) | partials
};
struct NoWords {};
struct MergeRest {
  int64_t part_set_o, part_set_ml;
};
//
// MANY (some pair has more than kManyPartials): 32 loads of a pair with more than kFew partials are on their way at a time, the
// first 32 before anything else is waited for and each further batch before the one ahead of it is added up, where the
// usual form takes four at a time.  One pair of 65 536 rows in 256 partials: a decode call 28.1 -> 21.9 us; 64 partials:
// 18.4 -> 18.2 us; 40 partials in two sets (gates): 19.6 -> 22.9 us, hence the line.  A kernel of its own also because the
// registers cost the usual form 0.2 us a launch.
constexpr int kManyPartials = 64;
constexpr int kFew = kMergeFew;          // two DPP rows
static_assert(kFew == 32);

template <typename T, bool IN_ARGS, bool MANY>
__global__ __launch_bounds__(kHeadDim) void combine_kernel(const float* __restrict__ all_o, const float* __restrict__ all_m,
                                                           const float* __restrict__ all_l, T* __restrict__ out,
                                                           char* __restrict__ list, int G, int pair_off, int advance,
                                                           MergeRest r, std::conditional_t<IN_ARGS, MergeWords, NoWords> words) {
  __shared__ float sm_scale[kHeadDim];
  __shared__ float sm_red[2];
  const int pi = blockIdx.x, g = blockIdx.y, d = threadIdx.x;
  int nseg, wg_first, n_sets = 1;
  float gate = 1.f;
  if constexpr (IN_ARGS) {
    const uint32_t word = words.w[pi];
    nseg = (int32_t)(word & 0xfffu);
    wg_first = (int32_t)(word >> 12) - pi;
  } else {
    const PairDesc pd = load_pair(list + pair_off, pi);
    nseg = pd.n_seg;
    wg_first = pd.wg_first;
    gate = pd.gate;
    // a gated full head (Eq. 1) has two sets of partials: full attention and local attention
    if (pd.ring < 0 && gate < 1.f) n_sets = 2;
  }
  // behind a fused append + decode launch: the list's growth counter follows the lengths (no kernel reads it
  // while this one runs; the next launch that does comes after it on the stream).  An addition in memory: nothing comes back.
  if (advance != 0 && pi == 0 && g == 0 && d == 0)
    (void)__hip_atomic_fetch_add(reinterpret_cast<int32_t*>(list), advance, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (nseg <= 1) return;                // no units (inactive slot), or a single workgroup wrote the final output itself
  const int64_t slot0 = (int64_t)wg_first + pi;       // partial slots of this pair are consecutive
  const int64_t at = ((int64_t)pi * G + g) * kHeadDim + d;
  auto emit = [&](float v) {
    if constexpr (sizeof(T) == 4) out[at] = v;
    else out[at] = f32_to_bf16_rne(v);
  };
  if (nseg <= kFew) {
    // Lanes 0 .. nseg - 1 of either half hold the partials' (m, l), so that each wavefront has the weights by itself; same ascending
    // order of accumulation as the general path below.
    const int mine = d & (kFew - 1), from = mine < nseg ? mine : 0;
    float o[2][kFew], mw[2], lw[2];
    auto ask = [&](int set) {
      const int64_t ml = set * r.part_set_ml + (slot0 + from) * G + g;
      mw[set] = all_m[ml];
      lw[set] = all_l[ml];
      const float* po = all_o + set * r.part_set_o + (slot0 * G + g) * kHeadDim + d;
#pragma unroll
      for (int t = 0; t < kFew; t += 4) {
        if (t >= nseg) break;
#pragma unroll
        for (int j = t; j < t + 4; ++j) o[set][j] = po[(int64_t)(j < nseg ? j : 0) * G * kHeadDim];   // (weight 0 beyond nseg)
      }
    };
    auto merged = [&](int set) {
      const float m = mine < nseg ? mw[set] : -INFINITY;
      const float M = max32(m);
      const float sc = exp2_or_zero(m, M);
      const float L = sum32(product(sc, mine < nseg ? lw[set] : 0.f));
      float acc = 0.f;
#pragma unroll
      for (int t = 0; t < kFew; t += 4) {
        if (t >= nseg) break;
#pragma unroll
        for (int j = t; j < t + 4; ++j)
          acc = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), j)), o[set][j], acc);
      }
      // (beyond nseg partial 0 stood in with a weight of zero, which makes a NaN of an Inf: such sums are taken again, one by one)
      if (__builtin_expect(__any(acc != acc), 0)) {
        const float* po = all_o + set * r.part_set_o + (slot0 * G + g) * kHeadDim + d;
        acc = 0.f;
#pragma unroll 1
        for (int j = 0; j < nseg; ++j)
          acc = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), j)), po[(int64_t)j * G * kHeadDim], acc);
      }
      return quotients(floatx4{acc, acc, acc, acc}, L)[0];
    };
    ask(0);
    if (!IN_ARGS && n_sets == 2) {
      ask(1);
      const float full = merged(0);
      emit(blend(gate, full, merged(1)));
    } else {
      emit(merged(0));
    }
    return;
  }
  float res_all = 0.f;
  for (int set = 0; set < n_sets; ++set) {
    const float* part_m = all_m + set * r.part_set_ml;
    const float* part_l = all_l + set * r.part_set_ml;
    const float* part_o = all_o + set * r.part_set_o;
    __syncthreads();
    constexpr int kDeep = MANY ? 32 : 1;
    const float* po = part_o + (slot0 * G + g) * kHeadDim + d;
    float o[kDeep];
    auto load = [&](int first) {
#pragma unroll
      for (int j = 0; j < kDeep; ++j) o[j] = first + j < nseg ? po[(int64_t)(first + j) * G * kHeadDim] : 0.f;
    };
    if (MANY) load(0);
    // maximum over the partial maxima
    float M = -INFINITY;
    for (int i = d; i < nseg; i += kHeadDim) M = fmaxf(M, part_m[(slot0 + i) * G + g]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    if ((d & 63) == 0) sm_red[d >> 6] = M;
    __syncthreads();
    M = fmaxf(sm_red[0], sm_red[1]);
    float acc = 0.f, L = 0.f;
    for (int base = 0; base < nseg; base += kHeadDim) {       // chunks of 128 partials, ascending order
      __syncthreads();
      const int i = base + d;
      float sc = 0.f, ls = 0.f;
      if (i < nseg) {
        const float mw = part_m[(slot0 + i) * G + g];
        sc = mw == -INFINITY ? 0.f : exp2f(mw - M);
        ls = sc * part_l[(slot0 + i) * G + g];
      }
      sm_scale[d] = sc;
      // normaliser: fixed-order tree over the chunk
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) ls += __shfl_xor(ls, off);
      __syncthreads();
      if ((d & 63) == 0) sm_red[d >> 6] = ls;
      __syncthreads();
      L += sm_red[0] + sm_red[1];
      if constexpr (MANY) {
        for (int j0 = 0; j0 < kHeadDim && base + j0 < nseg; j0 += kDeep) {
          float now[kDeep];
#pragma unroll
          for (int j = 0; j < kDeep; ++j) now[j] = o[j];
          load(base + j0 + kDeep);
#pragma unroll
          for (int j = 0; j < kDeep; ++j) acc += sm_scale[j0 + j] * now[j];       // (scale and value are 0 beyond nseg)
        }
      } else {
        const int cnt = nseg - base < kHeadDim ? nseg - base : kHeadDim;
        const float* pb = po + (int64_t)base * G * kHeadDim;
        int j = 0;
        for (; j + 4 <= cnt; j += 4) {
          const float a0 = pb[(int64_t)(j + 0) * G * kHeadDim], a1 = pb[(int64_t)(j + 1) * G * kHeadDim];
          const float a2 = pb[(int64_t)(j + 2) * G * kHeadDim], a3 = pb[(int64_t)(j + 3) * G * kHeadDim];
          acc += sm_scale[j] * a0; acc += sm_scale[j + 1] * a1; acc += sm_scale[j + 2] * a2; acc += sm_scale[j + 3] * a3;
        }
        for (; j < cnt; ++j) acc += sm_scale[j] * pb[(int64_t)j * G * kHeadDim];
      }
    }
    const float res = acc / L;
    res_all = n_sets == 1 ? res : (set == 0 ? gate * res : res_all + (1.f - gate) * res);
  }
  emit(res_all);
}

}  // namespace

hipError_t launch_combine(const DeviceView& dv, int layer, void* out, hipStream_t stream, int advance,
                          const uint32_t* merge_words, int most_partials) {
  const dim3 grid(dv.n_pairs, dv.group), block(kHeadDim);
  char* list = dv.list_base + layer * dv.list_stride;
  const MergeRest r = {dv.part_set_o, dv.part_set_ml};
  const bool in_args = merge_words != nullptr && dv.n_pairs <= kMergeArgPairs;
#define RLKV_LAUNCH(T, IA, MN, W)                                                                                          \
  hipLaunchKernelGGL((combine_kernel<T, IA, MN>), grid, block, 0, stream, dv.part_o, dv.part_m, dv.part_l, (T*)out, list, \
                     dv.group, dv.list_pair_off, advance, r, W)
#define RLKV_PICK(T, IA, W) do { if (most_partials > kManyPartials) RLKV_LAUNCH(T, IA, true, W); else RLKV_LAUNCH(T, IA, false, W); } while (0)
  if (in_args) {
    MergeWords words;
    memcpy(words.w, merge_words, (size_t)dv.n_pairs * sizeof(uint32_t));
    if (dv.dtype == RLKV_F32) RLKV_PICK(float, true, words);
    else RLKV_PICK(uint16_t, true, words);
  } else {
    if (dv.dtype == RLKV_F32) RLKV_PICK(float, false, NoWords{});
    else RLKV_PICK(uint16_t, false, NoWords{});
  }
#undef RLKV_PICK
#undef RLKV_LAUNCH
  return hipGetLastError();
}

}  // namespace rlkv
