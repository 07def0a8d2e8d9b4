// Merging the partials (m, l, O) of a pair that several workgroups share: pieces of the merge kernel (worklist_combine.hip), and the
// merge inside an attention launch.  Both give the same bits.
//
// Inside the launch: every wavefront that writes partials - of two heads - leaves them by device-scope stores, which write through the L2
// of its XCD, and at the end of its workgroup, once they have arrived, adds one to the counter of those heads for each pair (two pairs at
// most: the one the workgroup's share begins in and the one it ends in).  The wavefront that completes a counter reads all partials
// of the pair's two heads by device-scope loads, merges them, and sets the counter back.  Nobody waits for anybody, there is no
// barrier, and no cache-wide write-back or invalidation.
// Bound: latencies; behind the last tile of 8 x 8192, clocks: the wavefronts' sums 1400, stores 1400, atomic 1000, loads and sums 2500.
// It replaces a launch that every call waited for; where that pays: merges_in_launch in rlkv_api.hip, with the figures.
#pragma once

#include <tuple>
#include <type_traits>

#include "mfma_tile.h"

namespace rlkv {

template <int CTRL>
__device__ __forceinline__ float row_ror(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// Maximum / sum over 32 lanes, in every lane of them.
__device__ __forceinline__ float max32(float x) {
  x = fmaxf(x, row_ror<0x128>(x));
  x = fmaxf(x, row_ror<0x124>(x));
  x = fmaxf(x, row_ror<0x122>(x));
  x = fmaxf(x, row_ror<0x121>(x));
  const TwoValues y = swap16(x);
  return fmaxf(y.a, y.b);
}
__device__ __forceinline__ float sum32(float x) {
  x += row_ror<0x128>(x);
  x += row_ror<0x124>(x);
  x += row_ror<0x122>(x);
  x += row_ror<0x121>(x);
  const TwoValues y = swap16(x);
  return y.a + y.b;
}
// A product that is rounded by itself wherever it is compiled.
__device__ __forceinline__ float product(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}
// Eq. 1: gate * full + (1 - gate) * local.
__device__ __forceinline__ float blend(float gate, float full, float local) { return fmaf(gate, full, product(1.f - gate, local)); }

// Device-scope accesses (sc1): past this XCD's L2, where another one's could be stale or unseen.  As buffer accesses, whose resource
// is the partials of one pair or workgroup: the lane's offset is computed once and a partial's place is a scalar.
constexpr int kThrough = 16;                                 // sc1 among the cache bits of a buffer access
__device__ __forceinline__ __amdgpu_buffer_rsrc_t partials_at(float* p, int64_t first, int count) {
  return __builtin_amdgcn_make_buffer_rsrc(p + first, 0, count * 4, 0x00020000);
}

// Where partials are, and how many workgroups have left theirs (null: a merge launch follows).
struct Partials {
  float *o, *m, *l;
  int64_t set_o, set_ml;         // offsets of the second set (local attention of blending heads)
  int32_t* arrived;              // [pairs][kMaxGroup / 2] of the layer, 0 between launches
};

__device__ __forceinline__ Partials partials_at(RLKV_CONST Partials& p) { return {p.o, p.m, p.l, p.set_o, p.set_ml, p.arrived}; }

// The arguments of an attention kernel beyond the 14 words that are in registers when it starts, asked for where this is called: left
// alone the compiler asks for all of them, and computes what depends on them or on the thread's number alone, in front of the first loads
// (of fp32 rows 470 instructions, 90 of them to keep scalars in lanes of vector registers).
constexpr int kLateArgumentsAt = 14 * 4;
template <typename Rest>
__device__ __forceinline__ RLKV_CONST Rest* late_arguments() {
  auto* p = (RLKV_CONST Rest*)((RLKV_CONST char*)__builtin_amdgcn_kernarg_segment_ptr() + kLateArgumentsAt);
  asm volatile("" : "+s"(p));
  return p;
}

// Where a kernel's last argument begins, and its type: of every kernel that reads it by late_arguments checked where it is launched.
template <typename Kernel> struct LastArgument;
template <typename... Args> struct LastArgument<void (*)(Args...)> {
  typedef std::tuple_element_t<sizeof...(Args) - 1, std::tuple<Args...>> type;
  static constexpr int begin() {
    int at = 0, next = 0;
    ((at = (next + (int)alignof(Args) - 1) / (int)alignof(Args) * (int)alignof(Args), next = at + (int)sizeof(Args)), ...);
    return at;
  }
};
template <typename Kernel, typename Rest>
constexpr bool late_arguments_are_last() {
  return std::is_same_v<typename LastArgument<Kernel>::type, Rest> && LastArgument<Kernel>::begin() == kLateArgumentsAt;
}

// Four columns of head g and partial `slot`; m and l by the thread that has the first four.
__device__ __forceinline__ void leave_partial(const Partials& p, int set, int slot, int G, int g, int d4, const floatx4& O, float M, float L) {
  const int64_t heads = set * p.set_ml + (int64_t)slot * G, values = set * p.set_o + (int64_t)slot * G * kHeadDim;
  if (p.arrived) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, O), partials_at(p.o, values, G * kHeadDim), (g * kHeadDim + d4 * 4) * 4, 0, kThrough);
    if (d4 == 0) {
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(M), partials_at(p.m, heads, G), g * 4, 0, kThrough);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(L), partials_at(p.l, heads, G), g * 4, 0, kThrough);
    }
  } else {
    *reinterpret_cast<floatx4*>(p.o + values + g * kHeadDim + d4 * 4) = O;
    if (d4 == 0) { p.m[heads + g] = M; p.l[heads + g] = L; }
  }
}

// A pair this workgroup has left partials of.
struct LeftPair {
  int pair, first_wg, n_seg;
  float gate;                    // below 1: two sets
};

// Four values over one divisor: the reciprocal, and one correction of each quotient, which is as close as a division; what is not finite
// is left as the reciprocal alone gives it.
__device__ __forceinline__ floatx4 quotients(const floatx4& a, float b) {
  const float y0 = __builtin_amdgcn_rcpf(b), y = fmaf(fmaf(-b, y0, 1.f), y0, y0);
  floatx4 q;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float first = product(a[e], y), better = fmaf(fmaf(-first, b, a[e]), y, first);
    q[e] = __builtin_isfinite(better) ? better : product(a[e], y0);
  }
  return q;
}

// The partials of a pair's heads 2 * duo and 2 * duo + 1 merged by one wavefront: emit(g, d4, four columns).  sm_w: scratch in LDS.
template <bool BLENDS, typename Emit>
__device__ __forceinline__ void merge_duo(const Partials& p, const LeftPair& w, int duo, int G, float (*sm_w)[kMergeFew], Emit emit) {
  constexpr int kDeep = BLENDS ? 8 : 16;                     // partials asked for at a time, of each set
  const int d4 = threadIdx.x & 31, head = duo * 2 + ((threadIdx.x >> 5) & 1);
  const int g = head < G ? head : G - 1;
  const int slot0 = w.first_wg + w.pair;                     // the pair's slots are consecutive
  const bool two = BLENDS && w.gate < 1.f;
  // lanes 0 .. n_seg - 1 of either half hold the partials' (m, l)
  const int ml_off = (d4 * G + g) * 4, o_off = (g * kHeadDim + d4 * 4) * 4;
  float mw[2], lw[2];
  u32x4 o[BLENDS ? 2 : 1][kDeep];
  auto ask_o = [&](int set, int from) {
    const __amdgpu_buffer_rsrc_t rsrc = partials_at(p.o, set * p.set_o + (int64_t)slot0 * G * kHeadDim, w.n_seg * G * kHeadDim);
#pragma unroll
    for (int t = 0; t < kDeep; t += 4) {
      if (from + t >= w.n_seg) break;
#pragma unroll
      for (int j = t; j < t + 4; ++j)                        // (weight 0 beyond n_seg)
        o[set][j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o_off, from + j < w.n_seg ? (from + j) * G * kHeadDim * 4 : 0, kThrough);
    }
  };
  auto ask = [&](int set) {
    const int64_t heads = set * p.set_ml + (int64_t)slot0 * G;
    mw[set] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(partials_at(p.m, heads, w.n_seg * G), ml_off, 0, kThrough));
    lw[set] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(partials_at(p.l, heads, w.n_seg * G), ml_off, 0, kThrough));
    ask_o(set, 0);
  };
  ask(0);
  if (two) ask(BLENDS ? 1 : 0);
  auto merged = [&](int set) {
    const float m = d4 < w.n_seg ? mw[set] : -INFINITY;
    const float M = max32(m);
    const float sc = exp2_or_zero(m, M);
    const float L = sum32(product(sc, d4 < w.n_seg ? lw[set] : 0.f));
    sm_w[g][d4] = sc;                                        // (read by the same 32 lanes)
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int from = 0; from < w.n_seg; from += kDeep) {
      if (from > 0) ask_o(set, from);
#pragma unroll
      for (int t = 0; t < kDeep; t += 4) {
        if (from + t >= w.n_seg) break;
        const floatx4 four = *reinterpret_cast<const floatx4*>(&sm_w[g][from + t]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaf(four[j], __uint_as_float(o[set][t + j][e]), acc[e]);
        }
      }
    }
    // (Beyond n_seg partial 0 stood in with a weight of zero, which makes a NaN of an Inf: such sums are taken again, one by one.  Zeros in
    // its place, or no loads, cost every call 0.1 us.)
    const float any = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    if (__builtin_expect(__any(any != any), 0)) {
      const __amdgpu_buffer_rsrc_t rsrc = partials_at(p.o, set * p.set_o + (int64_t)slot0 * G * kHeadDim, w.n_seg * G * kHeadDim);
      acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int i = 0; i < w.n_seg; ++i) {
        const u32x4 one = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o_off, i * G * kHeadDim * 4, kThrough);
        const float weight = sm_w[g][i];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(weight, __uint_as_float(one[e]), acc[e]);
      }
    }
    return quotients(acc, L);
  };
  floatx4 out = merged(0);
  if (two) {
    const floatx4 local = merged(BLENDS ? 1 : 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = blend(w.gate, out[e], local[e]);
  }
  if (head < G) emit(g, d4, out);
}

// The end of a workgroup of kThreads that has left partials of `n` pairs (0 .. 2; `left` in LDS): thread t wrote those of heads t / 32, t / 32 + kThreads
// / 32 and so on.
template <int kThreads, bool BLENDS, typename Emit>
__device__ __forceinline__ void finish_pairs(const Partials& p, const LeftPair* left, int n, int G, float (*sm_w)[kMergeFew], Emit emit) {
  if (n == 0) return;
  constexpr int kDuos = kMaxGroup / 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (wave * 2 >= G) return;
  asm volatile("" ::: "memory");           // (no store of a partial behind the wait)
  __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0): the partials of this wavefront have arrived where every XCD sees them
  asm volatile("" ::: "memory");
  for (int duo = wave; duo * 2 < G; duo += kThreads / 64) {
    int missing = 1;
    if (lane < n)
      missing = left[lane].n_seg - 1 -
                __hip_atomic_fetch_add(p.arrived + left[lane].pair * kDuos + duo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::: "memory");
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
      if (__builtin_amdgcn_readlane(missing, k) != 0) continue;
      LeftPair w = left[k];
      w = LeftPair{__builtin_amdgcn_readfirstlane(w.pair), __builtin_amdgcn_readfirstlane(w.first_wg),
                   __builtin_amdgcn_readfirstlane(w.n_seg), w.gate};
      if (lane == 0) __hip_atomic_store(p.arrived + w.pair * kDuos + duo, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      merge_duo<BLENDS>(p, w, duo, G, sm_w, [&](int g, int d4, const floatx4& v) { emit(w.pair, g, d4, v); });
    }
  }
}

}  // namespace rlkv
