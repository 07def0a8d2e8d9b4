// Split-K decode attention over row-major stores (fp32, and bf16 where it is asked for).
//
// For every (sequence, KV head) pair the kernel computes ordinary softmax attention of
// the G query heads of the group over the rows the store holds (paper Sec. 3.1 Eq. 1 with
// the gate at 0 or 1; Sec. 3.3: compressed heads run full attention over their
// compressed cache).  A store's valid rows are always the prefix [0, n_eff), and softmax
// attention does not depend on the order of the rows, so ring slots are read in slot
// order.
//
// Mapping: a wavefront works 16 rows at a time, two rows to a load of 32 lanes with 4 columns each, with v_mfma_f32_4x4x1_16b_f32, 16
// independent blocks (lane quads) of a 4 x 4 outer product each (products and sums in fp32), four query heads to a set:
//   scores   block b = columns 16 (b % 8) .. + 15 of rows 2n + b / 8; A = 4 rows of K (n = 0 .. 3 or 4 .. 7), B = 4 heads of Q, one
//            instruction per column.  As loaded, a quad's lanes hold neighbouring columns of one row (lanes of a quad in different rows
//            take a load four times as long); a 4 x 4 transpose inside the quad gives each of them a row.
//   output   blocks 0..7 = one row, 8..15 the next: A = V as loaded, B = the weights of 4 heads, one
//            instruction per column of a lane: lane l holds 16 sums of head l%4, of the even rows or of the odd ones
// The partial scores of the blocks are dealt out as they are summed: each quarter of the wavefront keeps 4 of the 16 rows.
// Groups of one and two heads would leave most of a 4 x 4 block empty: they take multiply-adds of the vector ALU on rows as loaded, every
// lane its four columns of every head, the scores summed over the lanes of a row and dealt out in the same way.  us a launch with the
// matrix cores / with these: bf16, 48 of up to 700 tokens, 8 heads on 8, decode 19.7 / 16.7, a step 22.2 / 19.1, with blending heads 37.1 / 30.4
// and 46.0 / 37.4; 16 on 8 20.1 / 18.5 and 22.7 / 21.0, blending 37.0 / 34.0 and 46.2 / 42.5; fp32, one of 1500, 8 on 8 6.7 / 6.2, blending
// 10.5 / 9.5; 16 of 700, 16 on 8 13.0 / 12.5.  At three heads the matrix cores had gained on the former vector kernel (bf16, 24 on 8, 16 of up
// to 4000, 23.0 / 19.7).  Error against 64 bits the same (40 inputs each of four shapes: 1.48 to 2.02e-7 / 1.48 to 1.97e-7).
// With the vector ALU alone a batch of 16 rows and 4 fp32 heads was 520 instructions and 3300 clocks, which two wavefronts of a SIMD
// do not share; now 2000, 512 of them of the matrix cores.  References of the running maxima are whole numbers, so that moving a sum
// from one to another rounds nothing: error against 64 bits over 13 fp32 shapes 1.4e-7 .. 3.1e-7, before 1.5e-7 .. 4.7e-7, and no
// shape's is larger.
// Measured, before / now, us: fp32, one sequence of 1000 tokens and 16 steps, 32 query and 8 KV heads, the launch by itself 7.3 / 6.1;
// 8 x 5000, 28 and 4 heads 38.3 / 30.2, 16 on 1 33.7 / 21.5, 32 and 8 56.2 / 53.0 (at the rate of the memory); one of 60, 16 on 1 14.9 / 8.3;
// bf16, 16 x 16 384, 28 and 4 144 / 109, 8 x 5000, 32 and 8 32.6 / 30.0.
// Short lists wait for the start: with the second pass of blending heads in a form of its own (GATED) and whatever the loads do not need
// behind them (late_arguments), 470 instructions between the record and the first row are 190; a launch after another of a step of one
// fp32 sequence, 32 and 8 heads, half compressed, 20 / 500 / 1030 tokens 5.6 / 7.6 / 8.1 -> 4.2 / 6.2 / 7.1 us, of a decode call 4.2 / 6.5 /
// 7.3 -> 3.5 / 6.0 / 6.9.
#include <type_traits>

#include "share_merge.h"

namespace rlkv {
namespace {

// Four columns of a row, as loaded.
template <typename T> struct Elem;
template <> struct Elem<float> {
  typedef u32x4 Four;
  __device__ static void unpack(const Four& r, float* f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(r[e]);
  }
};
template <> struct Elem<uint16_t> {
  typedef uint32_t Four __attribute__((ext_vector_type(2)));
  __device__ static void unpack(const Four& r, float* f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float((e & 1) ? r[e >> 1] & 0xffff0000u : r[e >> 1] << 16);
  }
};

// 4 x 4 transpose over the lanes of each quad: lane i of x[k] receives what lane k of x[i] held.
template <typename Four>
__device__ __forceinline__ void quad_transpose(Four* x, int lane) {
  const bool odd = lane & 1, high = lane & 2;
  // (every lane takes part in an exchange: the empty asm keeps it out of a branch of the lanes that use it)
  auto other = [](int v, auto ctrl) {
    int x = __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xf, 0xf, true);
    asm("" : "+v"(x));
    return x;
  };
  constexpr std::integral_constant<int, 0xb1> xor1;      // quad_perm [1,0,3,2]
  constexpr std::integral_constant<int, 0x4e> xor2;      // quad_perm [2,3,0,1]
#pragma unroll
  for (int w = 0; w < (int)(sizeof(Four) / 4); ++w) {
    int t[4];
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
      const int a = x[k][w], b = x[k + 1][w], ax = other(a, xor1), bx = other(b, xor1);
      t[k] = odd ? bx : a;
      t[k + 1] = odd ? b : ax;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int ax = other(t[k], xor2), bx = other(t[k + 2], xor2);
      x[k][w] = high ? bx : t[k];
      x[k + 2][w] = high ? t[k + 2] : ax;
    }
  }
}

__device__ __forceinline__ floatx4 mfma_4x4(float a, float b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

constexpr uint32_t kShapeGroup = 31;           // of `shape`
constexpr int waves_for(int heads) { return heads > 8 ? 4 : 8; }
template <typename T>
struct DecodeRest {
  T* out;
  float scale_log2;
  int32_t n_kv_heads;
  Partials part;
  int32_t pair_off, batch;
  int32_t *len0, *len1;          // both copies of the layer's lengths
  int32_t* slot_pos;
  uint32_t recent_inverse;       // inverse_of(recent)
};

// GATED: some full head may have a gate below 1.  HEADS: room for heads, 1 and 2 on the vector ALU, else sets of four.
// FUSED: the step's append as well, in the manner of decode_mfma_kernel: the wavefront that owns the batch of
// rows with the new slot writes the row, every byte by the lane that loads it.
// Of every tile two wavefronts take a batch of 16 rows each, one register image, K refilled behind the scores and V behind the
// products; eight wavefronts, two per SIMD, up to group 8, four beyond (Q and the sums of four sets take 128 registers).  The first arguments are in registers when the kernel starts (decode_mfma.hip).
template <typename T, int HEADS, bool FUSED, bool GATED>
__global__ __launch_bounds__(waves_for(HEADS) * 64, 1) void decode_valu_kernel(const char* __restrict__ list, char* __restrict__ kv_base,
                                                             const T* __restrict__ q, const T* __restrict__ k_new,
                                                             const T* __restrict__ v_new, uint32_t shape, int grow_known,
                                                             int window, int recent, DecodeRest<T> r) {
  using E = Elem<T>;
  typedef typename E::Four Four;
  constexpr int kWaves = waves_for(HEADS), kThreads = kWaves * 64;
  constexpr bool kVector = HEADS <= 2;          // (a set is one head then, the same in every lane)
  constexpr int NS = kVector ? HEADS : HEADS / 4;
  constexpr int kBatch = 16;                    // rows of a batch
  constexpr int kLoads = kBatch / 2;            // loads of K and of V in a batch, two rows each
  constexpr int kBatches = kTile / kBatch;      // batches of a tile, one wavefront each
  constexpr int kStride = kWaves / kBatches;    // tiles a workgroup works at a time
  constexpr int kRowBytes = kHeadDim * sizeof(T);

  __shared__ floatx4 sm_o[kWaves][HEADS][kHeadDim / 4];
  __shared__ float2 sm_ml[HEADS][kWaves];
  __shared__ alignas(16) float sm_w[HEADS][kMergeFew];        // (merge_duo reads four weights at a time)
  __shared__ LeftPair sm_left[2];                      // (in LDS only to spare registers)

  const int wg = blockIdx.x;
  const WgDesc wd = load_wg(list, wg);
  // tokens since the list was planned: known to the host, or asked for beside the record
  int grow = grow_known;
  if (grow_known < 0) grow = load_const<int32_t>(list);
  // (what the loads and scores need of the other arguments in the shadow of the record; global pointers: see decode_mfma.hip)
  typedef __attribute__((address_space(1))) T GlobalOut;
  typedef __attribute__((address_space(1))) int32_t GlobalInt;
  auto late_args = [] { return late_arguments<DecodeRest<T>>(); };
  asm volatile("" : "+s"(r.scale_log2));
  if (FUSED) asm volatile("" : "+s"(r.recent_inverse));

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

  const int hl = lane & 3;                             // head of a set
  const int half = lane >> 5, off = (lane & 31) * 4 * (int)sizeof(T);        // loads: row of two, and bytes
  const int s_row = ((lane >> 4) & 1) * 8 + half;      // scores: rows s_row + 2 u, u = 0 .. 3
  const int G = shape & kShapeGroup;
  auto emit = [&](GlobalOut* out, int pair, int g, int d4, const floatx4& v) {
    constexpr int kAlign = 4 * sizeof(T);                // (a caller's output may start at any element)
    const bool out_aligned = ((uintptr_t)out & (kAlign - 1)) == 0;
    GlobalOut* dst = out + ((int64_t)pair * G + g) * kHeadDim + d4 * 4;
    if constexpr (sizeof(T) == 4) {
      if (out_aligned) {
        *(__attribute__((address_space(1))) floatx4*)dst = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = v[e];
      }
    } else {
      const uint2 four = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
      if (out_aligned) {
        *(__attribute__((address_space(1))) i32x2*)dst = i32x2{(int)four.x, (int)four.y};
      } else {
        dst[0] = (T)four.x;
        dst[1] = (T)(four.x >> 16);
        dst[2] = (T)four.y;
        dst[3] = (T)(four.y >> 16);
      }
    }
  };
  const int sink = window - recent;
  const int row0 = (wave % kBatches) * kBatch;         // the wavefront's batch of a tile

  for (int u = u_begin; u < u_end;) {
    // segment = the units [u, seg_end) of pair pi = tiles [tile_lo, tile_hi) of its store
    const int ps = pd.unit_start, pe = pd.unit_end;
    const int seg_end = u_end < pe ? u_end : pe;
    // the first unit(s) of a pair carry no tiles (they stand for its fixed cost)
    const int r_lo = u - ps > kPairOverheadUnits ? u - ps - kPairOverheadUnits : 0;
    const int r_hi = seg_end - ps > kPairOverheadUnits ? seg_end - ps - kPairOverheadUnits : 0;
    const int tile_lo = r_lo * wd.round_tiles;
    const bool whole_pair = u == ps && seg_end == pe;

    const int n_old = pd.n_build + grow;
    const int n = FUSED ? n_old + 1 : n_old;
    const bool full = pd.ring < 0;
    const int n_eff = full ? n : (n < window ? n : window);
    char* kst = kv_base + pd.koff;
    char* vst = kst + (int64_t)pd.cap * kRowBytes;
    // the list was built with room to grow: tiles past the valid prefix are still empty
    const int tiles_valid = (n_eff + kTile - 1) / kTile;
    const int tile_hi = r_hi * wd.round_tiles < tiles_valid ? r_hi * wd.round_tiles : tiles_valid;
    const int tile_first = tile_lo + wave / kBatches;

    // This step's append: position n_old goes to slot_new (sink / ring / next row of a full head).  The row is asked for first and
    // written behind the loads of the wavefront's first batch.
    int slot_new = 0;
    bool mine = false;
    Four kn, vn;
    if (FUSED) {
      slot_new = (full || n_old < sink) ? n_old : sink + remainder_of(n_old - sink, recent, r.recent_inverse);
      const int tile_new = slot_new / kTile;
      mine = tile_new >= tile_lo && tile_new < tile_hi && (tile_new - tile_lo) % kStride == wave / kBatches &&
             slot_new % kTile / kBatch * kBatch == row0;
      if (mine) {
        kn = *reinterpret_cast<const Four*>(reinterpret_cast<const char*>(k_new) + (int64_t)pi * kRowBytes + off);
        vn = *reinterpret_cast<const Four*>(reinterpret_cast<const char*>(v_new) + (int64_t)pi * kRowBytes + off);
      }
    }
    // Q: the block's 16 columns of head hl of every set (past the group: its last head again; nobody reads what comes of it); on the
    // vector ALU the lane's four columns of every head
    float qf[NS][kVector ? 4 : 16];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if constexpr (kVector) {
        E::unpack(*reinterpret_cast<const Four*>(reinterpret_cast<const char*>(q) + ((int64_t)pi * HEADS + s) * kRowBytes + off), qf[s]);
        continue;
      }
      const int g = s * 4 + hl < G ? s * 4 + hl : G - 1;
      const Four* src = reinterpret_cast<const Four*>(reinterpret_cast<const char*>(q) + ((int64_t)pi * G + g) * kRowBytes) + ((lane >> 2) & 7) * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) E::unpack(src[k], qf[s] + 4 * k);
    }

    // Eq. 1 gate (GATED): a full head with gate < 1 takes a second, local pass over the tiles of this
    // segment that hold sink or recent positions; out = gate * full + (1 - gate) * local.
    const bool two_pass = GATED && full && pd.gate < 1.f;
    const int keep_lo = sink, keep_from = n - recent;              // local pass: row < S or row >= n - R
    const int sink_tiles = (keep_lo + kTile - 1) / kTile;
    const int recent_tile0 = keep_from > 0 ? keep_from / kTile : 0;
    constexpr int kPasses = (HEADS * kHeadDim / 4 + kThreads - 1) / kThreads;
    floatx4 held[kPasses];                                         // full-pass results of a whole-pair segment
#pragma unroll 1
    for (int pass = 0; pass < (two_pass ? 2 : 1); ++pass) {
      float m[NS], l[NS];
      // [set][column of four]: D row i = columns 4 * (4 * (block % 8) + i) + e; on the vector ALU [head][0], the lane's four columns
      floatx4 acc[NS][kVector ? 1 : 4];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        m[s] = -INFINITY;
        l[s] = 0.f;
#pragma unroll
        for (int e = 0; e < (kVector ? 1 : 4); ++e) acc[s][e] = floatx4{0.f, 0.f, 0.f, 0.f};
      }

      struct Rows { Four k[kLoads], v[kLoads]; };
      auto counts = [&](int tok) { return (tok < n_eff) & (!GATED | (pass == 0) | (tok < keep_lo) | (tok >= keep_from)); };   // (no short circuits)
      // rows are read once per step: stream them past the caches
      auto load = [&](Four (&dst)[kLoads], const char* st, int tile) {
        const char* base = st + (int64_t)tile * (kTile * kRowBytes);
        const int last = n_eff - 1 - tile * kTile;                       // stay inside the valid prefix
#pragma unroll
        for (int t = 0; t < kLoads; ++t) {
          const int row = row0 + t * 2 + half;
          dst[t] = __builtin_nontemporal_load(reinterpret_cast<const Four*>(base + (uint32_t)((row < last ? row : last) * kRowBytes + off)));
        }
      };
      auto work = [&](Rows& rw, int tile, auto scored) {
        const int tok0 = tile * kTile + row0;
        const bool ragged = tok0 + kBatch > n_eff || (GATED && pass == 1 && tok0 + kBatch > keep_lo && tok0 < keep_from);
        float sc[NS][4];                       // [set][u]: rows s_row + 2 u of the batch
        if constexpr (kVector) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float kf[2][4];
            E::unpack(rw.k[u], kf[0]);
            E::unpack(rw.k[4 + u], kf[1]);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              float x[2];
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                x[i] = kf[i][0] * qf[s][0];
#pragma unroll
                for (int e = 1; e < 4; ++e) x[i] = fmaf(kf[i][e], qf[s][e], x[i]);
              }
              const TwoValues y = deal16(x[0], x[1]);
              float z = y.a + y.b;
              z += row_ror<0x128>(z);
              z += row_ror<0x124>(z);
              z += row_ror<0x122>(z);
              z += row_ror<0x121>(z);
              sc[s][u] = z;
            }
          }
        } else
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          Four x[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) x[k] = rw.k[part * 4 + k];
          quad_transpose(x, lane);
          float kf[16];
#pragma unroll
          for (int k = 0; k < 4; ++k) E::unpack(x[k], kf + 4 * k);
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            floatx4 d[4];                      // (four sums of four columns: one chain loses more of the small products behind large ones)
#pragma unroll
            for (int k = 0; k < 4; ++k) d[k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int k = 0; k < 4; ++k) d[k] = mfma_4x4(kf[4 * k + e], qf[s][4 * k + e], d[k]);
            const floatx4 sum = (d[0] + d[1]) + (d[2] + d[3]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (part == 0) {
                sc[s][u] = sum[u];
              } else {
                const TwoValues y = deal16(sc[s][u], sum[u]);
                float z = y.a + y.b;
                z += row_ror<0x128>(z);
                z += row_ror<0x124>(z);
                sc[s][u] = z;
              }
            }
          }
        }
        scored();                        // K's registers are free from here on
        // The reference is a whole number (log2 domain): what moves a sum from one reference to another, here and in the merges, is a power
        // of two and rounds nothing.  The scale goes into the exponent's one rounding, up to references of 2^24.  From there on the products
        // are whole numbers, and a product before its rounding may lie beyond the reference by more than an exponential takes (128 from
        // 2^31 on), on either side: there the rounded products count, of which the largest is the reference.
        bool on[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) on[u] = !ragged || counts(tok0 + s_row + 2 * u);
        float p[NS][4];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          float mx = -INFINITY;
#pragma unroll
          for (int u = 0; u < 4; ++u) mx = fmaxf(mx, on[u] ? product(sc[s][u], r.scale_log2) : -INFINITY);
          const float m_new = fmaxf(m[s], __builtin_ceilf(column_max(mx)));     // (over the quarters, which hold other rows)
          const float m_ref = m_new == -INFINITY ? 0.f : m_new;
          const float alpha = __builtin_amdgcn_exp2f(m[s] - m_ref);   // 2^-inf = 0 for a fresh stream
          m[s] = m_new;
          float sum = 0.f, factor = r.scale_log2;
          const bool whole = fabsf(m_ref) >= 0x1p24f;
          if (__builtin_expect(__any(whole), 0)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) sc[s][u] = whole ? product(sc[s][u], r.scale_log2) : sc[s][u];
            factor = whole ? 1.f : r.scale_log2;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            p[s][u] = on[u] ? __builtin_amdgcn_exp2f(fmaf(sc[s][u], factor, -m_ref)) : 0.f;
            sum += p[s][u];
          }
          l[s] = l[s] * alpha + sum;
          if (__any(alpha != 1.f)) {
#pragma unroll
            for (int e = 0; e < (kVector ? 1 : 4); ++e) acc[s][e] *= alpha;
          }
        }
        // (a row that does not count may hold anything, and of a step be the one another wavefront is writing: nothing of it may reach a sum)
        if (ragged) {
#pragma unroll
          for (int t = 0; t < kLoads; ++t) {
            uint32_t keep = counts(tok0 + t * 2 + half) ? 0xffffffffu : 0u;
            asm("" : "+v"(keep));                       // (a mask in a vector register: eight comparisons in scalar ones are kept in lanes)
            rw.v[t] &= keep;
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float vf[2][4];
          E::unpack(rw.v[u], vf[0]);
          E::unpack(rw.v[4 + u], vf[1]);
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const TwoValues w = swap16(p[s][u]);       // rows 2u and 2u + 1 in the halves, then 8 + 2u and 9 + 2u
            if constexpr (kVector) {
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[s][0][e] = fmaf(vf[1][e], w.b, fmaf(vf[0][e], w.a, acc[s][0][e]));
              continue;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[s][e] = mfma_4x4(vf[0][e], w.a, acc[s][e]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[s][e] = mfma_4x4(vf[1][e], w.b, acc[s][e]);
          }
        }
      };
      // the tile at or behind `tile` (in this wavefront's steps) that this pass looks at
      auto settle = [&](int tile) {
        if (GATED && pass == 1 && tile >= sink_tiles && tile < recent_tile0) tile += (recent_tile0 - tile + kStride - 1) / kStride * kStride;   // hop over the evicted middle
        return tile;
      };
      int tile = settle(tile_first);
      if (tile < tile_hi) {
        Rows rw;
        load(rw.k, kst, tile);
        load(rw.v, vst, tile);
        if (FUSED && mine && (!GATED || pass == 0)) {
          // the row goes into the store and, where this is its batch, into the registers: a load behind the stores would be
          // another memory latency
          const int in = slot_new % kBatch;
          const bool lane_new = half == in % 2;
          if (tile == slot_new / kTile) {
            int at = lane_new ? in / 2 : -1;
            asm volatile("" : "+v"(at));                  // (eight comparisons here, not in front of the loads)
#pragma unroll
            for (int t = 0; t < kLoads; ++t) {
              const bool here = at == t;
#pragma unroll
              for (int w = 0; w < (int)(sizeof(Four) / 4); ++w) {
                rw.k[t][w] = here ? kn[w] : rw.k[t][w];
                rw.v[t][w] = here ? vn[w] : rw.v[t][w];
              }
            }
          }
          if (lane_new) {
            *reinterpret_cast<Four*>(kst + (int64_t)slot_new * kRowBytes + off) = kn;
            *reinterpret_cast<Four*>(vst + (int64_t)slot_new * kRowBytes + off) = vn;
          }
          auto* late = late_args();
          if (lane == 0 && !full) ((GlobalInt*)late->slot_pos)[((int64_t)pd.ring * late->batch + b) * window + slot_new] = n_old;
        }
        for (;;) {
          const int next = settle(tile + kStride);
          if (next >= tile_hi) break;
          work(rw, tile, [&] { load(rw.k, kst, next); });
          load(rw.v, vst, next);
          tile = next;
        }
        work(rw, tile, [] {});
      }

      // (what follows is computed behind the loads, see late_arguments)
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, hl = tid & 3;
      auto* late = late_args();
      const Partials part = partials_at(late->part);
      GlobalOut* out = (GlobalOut*)late->out;
      // The halves of a wavefront (even and odd rows; one reference) are added as their columns are dealt out over them.
      if (u != u_begin || (GATED && pass > 0)) __syncthreads();   // the previous merge has finished reading LDS
      if (pass == 0 && tid == 0 && !whole_pair) sm_left[n_left] = LeftPair{pi, pd.wg_first, pd.n_seg, two_pass ? pd.gate : 1.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const TwoValues l16 = swap16(l[s]);
        const TwoValues l32 = swap32(l16.a + l16.b);
        if constexpr (kVector) {
          if (lane == 0) sm_ml[s][wave] = make_float2(m[s], l32.a + l32.b);
          continue;
        }
        if (lane < 4) sm_ml[s * 4 + hl][wave] = make_float2(m[s], l32.a + l32.b);
        floatx4 o[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const TwoValues x = deal32(acc[s][e][i], acc[s][e][i + 2]);
            o[i][e] = x.a + x.b;
          }
        // (four columns to an entry: of the lane's block, i and, in the upper half, i + 2)
        const int at = ((lane >> 2) & 7) * 4 + (lane >> 5) * 2;
        sm_o[wave][s * 4 + hl][at] = o[0];
        sm_o[wave][s * 4 + hl][at + 1] = o[1];
      }
      if constexpr (kVector) {
        floatx4 o;                             // head 0 in the lower half, the last one in the upper
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const TwoValues x = deal32(acc[0][0][e], acc[NS - 1][0][e]);
          o[e] = x.a + x.b;
        }
        sm_o[wave][(lane >> 5) * (HEADS - 1)][lane & 31] = o;
      }
      __syncthreads();
      // merge the wavefronts, four outputs of a head per thread; emit the final output or a partial for the combine pass
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
          if (GATED && two_pass) {
            if (pass == 0) { held[it] = res; continue; }
            res = pd.gate * held[it] + (1.f - pd.gate) * res;
          }
          emit(out, pi, g, d4, res);
        } else {
          leave_partial(part, GATED ? pass : 0, wg + pi, G, g, d4, O, M, L);
        }
      }
    }   // pass
    auto* late = late_args();
    if (!whole_pair && late->part.arrived) ++n_left;
    // whoever owns tile 0 of head 0 publishes the new length, in both copies of the table (nobody reads either during this launch)
    if (FUSED && h == 0 && tile_lo == 0 && tid == 0) {
      ((GlobalInt*)late->len0)[b] = n;
      ((GlobalInt*)late->len1)[b] = n;
    }
    u = seg_end;
    auto step_on = [&]() { ++pi; if (++h == late->n_kv_heads) { h = 0; ++b; } };
    while (u < u_end) {
      step_on();
      pd = load_pair(list + late->pair_off, pi);
      if (pd.unit_end > u) break;                          // (pairs of inactive slots own no units)
    }
  }
  if (n_left > 0) {
    auto* late = late_args();
    finish_pairs<kThreads, GATED>(partials_at(late->part), sm_left, n_left, G, sm_w,
                                  [&](int pair, int g, int d4, const floatx4& v) { emit((GlobalOut*)late->out, pair, g, d4, v); });
  }
  if (advance) *reinterpret_cast<int32_t*>(const_cast<char*>(list)) = grow + 1;
}

template <typename T, bool FUSED, bool GATED>
hipError_t launch_t(const DeviceView& dv, int layer, const void* q, void* out, float scale_log2, const void* k_new,
                    const void* v_new, int grow, bool merge_here, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(dv.n_wg);
  const T *qp = (const T*)q, *kp = (const T*)k_new, *vp = (const T*)v_new;
  const int G = dv.group;
  const char* list = dv.list_base + layer * dv.list_stride;
  const uint32_t shape = (uint32_t)G;
  DecodeRest<T> r = {};
  r.out = (T*)out; r.scale_log2 = scale_log2; r.n_kv_heads = dv.n_kv_heads;
  r.part = {dv.part_o, dv.part_m, dv.part_l, dv.part_set_o, dv.part_set_ml, merge_here ? dv.arrived + (int64_t)layer * dv.n_pairs * (kMaxGroup / 2) : nullptr};
  r.pair_off = dv.list_pair_off; r.batch = dv.batch;
  r.len0 = len_of(dv, 0, layer); r.len1 = len_of(dv, 1, layer); r.slot_pos = dv.slot_pos;
  r.recent_inverse = inverse_of(dv.recent);
  // (without events: the plain launch, which a stream capture can record)
#define RLKV_LAUNCH_ROWS(HEADS)                                                                                         \
  do {                                                                                                               \
    static_assert(late_arguments_are_last<decltype(&decode_valu_kernel<T, HEADS, FUSED, GATED>), DecodeRest<T>>());     \
    if (e0 || e1)                                                                                                    \
      hipExtLaunchKernelGGL((decode_valu_kernel<T, HEADS, FUSED, GATED>), grid, dim3(waves_for(HEADS) * 64), 0, stream, e0, e1, 0, list, dv.kv_base, \
                            qp, kp, vp, shape, grow, dv.window, dv.recent, r);                                       \
    else                                                                                                             \
      hipLaunchKernelGGL((decode_valu_kernel<T, HEADS, FUSED, GATED>), grid, dim3(waves_for(HEADS) * 64), 0, stream, list, dv.kv_base, qp, kp, vp,   \
                         shape, grow, dv.window, dv.recent, r);                                                      \
  } while (0)
  if (G == 1) RLKV_LAUNCH_ROWS(1);
  else if (G == 2) RLKV_LAUNCH_ROWS(2);
  else if (G <= 4) RLKV_LAUNCH_ROWS(4);
  else if (G <= 8) RLKV_LAUNCH_ROWS(8);
  else RLKV_LAUNCH_ROWS(16);
#undef RLKV_LAUNCH_ROWS
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_valu(const DeviceView& dv, int layer, bool gated, const void* q, void* out, float scale_log2,
                              const void* k_new, const void* v_new, int grow, bool merge_here, hipStream_t stream, hipEvent_t ev_start,
                              hipEvent_t ev_stop) {
#define RLKV_PICK(T, F) \
  (gated ? launch_t<T, F, true> : launch_t<T, F, false>)(dv, layer, q, out, scale_log2, k_new, v_new, grow, merge_here, stream, ev_start, ev_stop)
  if (dv.dtype == RLKV_F32) return k_new ? RLKV_PICK(float, true) : RLKV_PICK(float, false);
  return k_new ? RLKV_PICK(uint16_t, true) : RLKV_PICK(uint16_t, false);
#undef RLKV_PICK
}

}  // namespace rlkv
