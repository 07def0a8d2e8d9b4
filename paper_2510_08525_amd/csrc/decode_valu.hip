// Split-K decode attention, vector-ALU variant (row-major stores; fp32 and bf16).
//
// For every (sequence, KV head) pair the kernel computes ordinary softmax attention of
// the G query heads of the group over the rows the store holds (paper Sec. 3.1 Eq. 1 with
// the gate at 0 or 1; Sec. 3.3: compressed heads run full attention over their
// compressed cache).  A store's valid rows are always the prefix [0, n_eff), and softmax
// attention does not depend on the order of the rows, so ring slots are read in slot
// order.
//
// Mapping: a wavefront reads whole rows with 128-bit loads, 16 lanes per row (a 256-byte bf16 row
// in one load, a 512-byte fp32 row in two); every lane keeps its 8 elements of Q for all heads of the group, so a
// K/V row is loaded once per group.  (32 lanes per fp32 row, 4 elements each, took twice the reductions, exponentials and
// batches per tile.  With one round of tiles per workgroup where the grid allows it, fp32 decode of one sequence of 1000 tokens:
// 15.7 -> 10.7 us a call, 8 of 5000: 43.2 -> 33.4 us; with the append in the same launch, a step of one sequence of 1000
// tokens: 18.2 -> 11.2 us.)
// Dot products are reduced across the lanes of a row with DPP row rotations; each group
// of lanes that shares a row index runs its own online softmax, and the streams are
// merged at the end of the segment (lane groups by shuffles, wavefronts through LDS).
#include "mfma_tile.h"

namespace rlkv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ inline float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

// Sum over the 16 lanes of a DPP row; every lane receives the total.
__device__ inline float row_sum16(float x) {
  x += dpp_mov<0x128>(x);  // row_ror:8
  x += dpp_mov<0x124>(x);  // row_ror:4
  x += dpp_mov<0x122>(x);  // row_ror:2
  x += dpp_mov<0x121>(x);  // row_ror:1
  return x;
}

// Element types.  `Q` is what a lane keeps of a query row (its column chunk) and `dot` the lane's part of
// <q, k> for one K row as loaded: fp32 multiplies and adds the unpacked elements; bf16 leaves both rows packed
// and takes two products per instruction (v_dot2c_f32_bf16: exact products, fp32 accumulation), which spares
// the unpacking of K and half of the multiply-adds - this kernel is bound by its vector instruction count.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kChunks = 2;            // 16-byte chunks of a row per lane
  struct Q { float f[8]; };
  __device__ static void unpack(const uint4 (&r)[2], float* f) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f[4 * i + 0] = __uint_as_float(r[i].x); f[4 * i + 1] = __uint_as_float(r[i].y);
      f[4 * i + 2] = __uint_as_float(r[i].z); f[4 * i + 3] = __uint_as_float(r[i].w);
    }
  }
  __device__ static Q query(const uint4 (&r)[2]) { Q q; unpack(r, q.f); return q; }
  __device__ static float dot(const Q& q, const uint4 (&k)[2]) {
    float kf[8];
    unpack(k, kf);
    // (a sum of its own per chunk: one chain over both loses more of the small products behind large ones)
    float d[2] = {0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e >> 2] = fmaf(q.f[e], kf[e], d[e >> 2]);
    return d[0] + d[1];
  }
};
template <> struct Elem<uint16_t> {
  static constexpr int kChunks = 1;
  struct Q { uint4 packed; };
  __device__ static void unpack(const uint4 (&rr)[1], float* f) {
    const uint4& r = rr[0];
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  }
  __device__ static Q query(const uint4 (&r)[1]) { return Q{r[0]}; }
  __device__ static float dot(const Q& q, const uint4 (&kk)[1]) {
    const uint4& k = kk[0];
    float d = 0.f;
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.packed.x), __builtin_bit_cast(bf16x2, k.x), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.packed.y), __builtin_bit_cast(bf16x2, k.y), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.packed.z), __builtin_bit_cast(bf16x2, k.z), d, false);
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.packed.w), __builtin_bit_cast(bf16x2, k.w), d, false);
    return d;
  }
};

// FUSED: the step's append as well, in the manner of decode_mfma_kernel: the wavefront that owns the tile with the new
// slot writes the row before it loads the tile, every 16 bytes by the lane that later loads them.
template <typename T, int GB, bool FUSED>
__global__ __launch_bounds__(kBlock, 1) void decode_valu_kernel(DeviceView dv, int layer,
                                                             const T* __restrict__ q, T* __restrict__ out,
                                                             float scale_log2, const T* __restrict__ k_new,
                                                             const T* __restrict__ v_new, int grow_known) {
  constexpr int LPR = 16;                       // lanes per row
  constexpr int EPL = kHeadDim / LPR;           // elements per lane
  constexpr int CH = Elem<T>::kChunks;          // 16-byte chunks they come in, 16 chunks apart
  constexpr int EPC = EPL / CH;                 // elements per chunk
  constexpr int RPL = 64 / LPR;                 // rows per wavefront load
  constexpr int U = 4;                          // row loads in flight per K and per V
  constexpr int kBatches = kTile / (RPL * U);

  __shared__ floatx4 sm_o[4][GB][kHeadDim / 4];
  __shared__ float sm_m[4][GB];
  __shared__ float sm_l[4][GB];

  const int wg = blockIdx.x;
  const WgDesc* __restrict__ wdp = wg_desc_of(dv, layer) + wg;
  // tokens since the list was planned: known to the host, or asked for beside the record
  const int grow = grow_known >= 0 ? grow_known : list_header(dv, layer)->grow;
  if (FUSED && grow_known >= 0 && blockIdx.x == 0 && threadIdx.x == 0)
    list_header(dv, layer)->grow = grow + 1;           // (no workgroup of this launch reads it)
  const int u_begin = wdp->u_begin, u_end = wdp->u_end;
  if (u_begin >= u_end) return;
  int pi = wdp->first_pair;
  PairDesc pd = wdp->first;
  const PairDesc* __restrict__ pairs = pair_desc_of(dv, layer);

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int c = lane % LPR, rg = lane / LPR;
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
    PairDesc pd_next = pd;
    if (seg_end < u_end) pd_next = pairs[pi + 1];     // (moved to scalar registers here, which waits for it)

    const int b = pi / dv.n_kv_heads, h = pi % dv.n_kv_heads;
    const int n_old = pd.n_build + grow;
    const int n = FUSED ? n_old + 1 : n_old;
    const bool full = pd.ring < 0;
    const int n_eff = full ? n : (n < dv.window ? n : dv.window);
    char* kst = dv.kv_base + pd.koff;
    char* vst = kst + (int64_t)pd.cap * dv.row_bytes;
    // the list was built with room to grow: tiles past the valid prefix are still empty
    const int tiles_valid = (n_eff + kTile - 1) / kTile;
    const int tile_hi = r_hi * kRound < tiles_valid ? r_hi * kRound : tiles_valid;

    if (FUSED) {
      // whoever owns tile 0 of head 0 publishes the new length, in both copies of the table (nobody reads
      // either during this launch)
      if (h == 0 && tile_lo == 0 && tid == 0) { len_of(dv, 0, layer)[b] = n; len_of(dv, 1, layer)[b] = n; }
      const int slot_new = (full || n_old < dv.sink) ? n_old : dv.sink + (n_old - dv.sink) % dv.recent;
      const int tile_new = slot_new / kTile;
      if (tile_new >= tile_lo && tile_new < tile_hi && ((tile_new - tile_lo) & 3) == wave) {
        if (rg == slot_new % RPL) {                        // the lanes that load row slot_new below
          const int64_t src = ((int64_t)b * dv.n_kv_heads + h) * dv.row_bytes + c * 16;
          const int64_t dst = (int64_t)slot_new * dv.row_bytes + c * 16;
          uint4 kn[CH], vn[CH];
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            kn[i] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(k_new) + src + i * LPR * 16);
            vn[i] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(v_new) + src + i * LPR * 16);
          }
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            *reinterpret_cast<uint4*>(kst + dst + i * LPR * 16) = kn[i];
            *reinterpret_cast<uint4*>(vst + dst + i * LPR * 16) = vn[i];
          }
        }
        if (lane == 0 && !full)
          dv.slot_pos[((int64_t)pd.ring * dv.batch + b) * dv.window + slot_new] = n_old;
      }
    }

    for (int gb = 0; gb < G; gb += GB) {
      const int gcount = G - gb < GB ? G - gb : GB;
      typename Elem<T>::Q qf[GB];
#pragma unroll
      for (int g = 0; g < GB; ++g) {
        uint4 r[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          r[i] = make_uint4(0, 0, 0, 0);                   // (no such head: zeros, in either element type)
          if (g < gcount) {
            const int64_t qrow = (int64_t)b * dv.n_q_heads + h * G + gb + g;
            r[i] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(q) + qrow * dv.row_bytes + (i * LPR + c) * 16);
          }
        }
        qf[g] = Elem<T>::query(r);
      }

      // Eq. 1 gate: a full head with gate < 1 takes a second, local pass over the tiles of this
      // segment that hold sink or recent positions; out = gate * full + (1 - gate) * local.
      const bool two_pass = full && pd.gate < 1.f;
      const int keep_lo = dv.sink, keep_from = n - dv.recent;        // local pass: row < S or row >= n - R
      const int sink_tiles = (keep_lo + kTile - 1) / kTile;
      const int recent_tile0 = keep_from > 0 ? keep_from / kTile : 0;
      constexpr int kPasses = (GB * kHeadDim / 4 + kBlock - 1) / kBlock;
      floatx4 held[kPasses];                                         // full-pass results of a whole-pair segment
      for (int pass = 0; pass < (two_pass ? 2 : 1); ++pass) {
      float m[GB], l[GB], acc[GB][EPL];
#pragma unroll
      for (int g = 0; g < GB; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
      }

      // The wavefront's rows in batches of U loads of K and of V.
      // fp32, and groups beyond 4: one loop, one copy of its body.  bf16 up to group 4: two register images that swap roles, a
      // batch asked for before the one ahead of it is worked on.  With the images everywhere the body stands four times,
      // 29 to 43 KB of code at group 8, and half the registers are reached through copies.  Two images / one loop (us per
      // call): bf16, 8 sequences of 5000 tokens, 32 query and 8 KV heads 22.1 / 27.6, group 16 (one sequence) 35.7 / 32.6; fp32,
      // group 16, 8 of 5000 95.6 / 84.8, one of 60 23.8 / 19.0; fp32, group 4: one of 1000 tokens, a fused step 11.8 / 11.2.
      struct Rows { uint4 k[U][CH], v[U][CH]; bool on[U]; };
      auto load = [&](Rows& r, int tile, int bt) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int tok = tile * kTile + (bt * U + u) * RPL + rg;
          // (no short circuits: they make a branch around every row's loads)
          r.on[u] = (tok < n_eff) & ((pass == 0) | (tok < keep_lo) | (tok >= keep_from));
          const int tc = r.on[u] ? tok : n_eff - 1;          // stay inside the valid prefix
          const int64_t off = (int64_t)tc * dv.row_bytes + c * 16;
          // rows are read once per step: stream them past the caches
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            const u32x4 kk = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kst + off + i * LPR * 16));
            const u32x4 vv = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vst + off + i * LPR * 16));
            r.k[u][i] = make_uint4(kk.x, kk.y, kk.z, kk.w);
            r.v[u][i] = make_uint4(vv.x, vv.y, vv.z, vv.w);
          }
        }
      };
      auto work = [&](Rows& r) {
        float s[U][GB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // (a row that does not count may be the one another wavefront is writing: nothing of it may reach a sum)
#pragma unroll
          for (int i = 0; i < CH; ++i)
            if (FUSED && !r.on[u]) r.v[u][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
          for (int g = 0; g < GB; ++g) {
            float d = Elem<T>::dot(qf[g], r.k[u]);
            d = row_sum16(d);
            s[u][g] = r.on[u] ? d * scale_log2 : -INFINITY;
          }
        }
        float p[U][GB];
#pragma unroll
        for (int g = 0; g < GB; ++g) {
          float mx = s[0][g];
#pragma unroll
          for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u][g]);
          const float m_new = fmaxf(m[g], mx);
          const float m_ref = m_new == -INFINITY ? 0.f : m_new;
          const float alpha = __builtin_amdgcn_exp2f(m[g] - m_ref);   // 2^-inf = 0 for a fresh stream
          m[g] = m_new;
          float ps_ = 0.f;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            p[u][g] = __builtin_amdgcn_exp2f(s[u][g] - m_ref);
            ps_ += p[u][g];
          }
          l[g] = l[g] * alpha + ps_;
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[g][e] *= alpha;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float vf[EPL];
          Elem<T>::unpack(r.v[u], vf);
#pragma unroll
          for (int g = 0; g < GB; ++g)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(p[u][g], vf[e], acc[g][e]);
        }
      };
      // the tile at or behind `tile` (in this wavefront's steps of 4) that this pass looks at
      auto settle = [&](int tile) {
        if (pass == 1 && tile >= sink_tiles && tile < recent_tile0) tile += (recent_tile0 - tile + 3) / 4 * 4;   // hop over the evicted middle
        return tile;
      };
      if constexpr (GB > 4 || sizeof(T) == 4) {
        for (int tile = settle(tile_lo + wave); tile < tile_hi; tile = settle(tile + 4)) {
#pragma unroll 1
          for (int bt = 0; bt < kBatches; ++bt) {
            Rows r;
            load(r, tile, bt);
            work(r);
          }
        }
      } else {
        int tile = settle(tile_lo + wave), bt = 0;
        auto step_on = [&]() { if (++bt == kBatches) { bt = 0; tile = settle(tile + 4); } };
        if (tile < tile_hi) {
          Rows ra, rb;
          load(ra, tile, bt);
          for (;;) {
            step_on();
            if (tile >= tile_hi) { work(ra); break; }
            load(rb, tile, bt);
            work(ra);
            step_on();
            if (tile >= tile_hi) { work(rb); break; }
            load(ra, tile, bt);
            work(rb);
          }
        }
      }

      // Merge of the wavefront's four lane groups (they hold the same columns), lane groups 16 apart first, then halves.  The columns
      // are dealt out as they are summed - of a pair of lanes either keeps one half of its columns - so that every lane ends up with
      // two whole sums.  (Every lane summing all eight of its columns by LDS permutes, and one output per thread and pass
      // below, took longer by 10 % of a 1000-token prompt and 16 fp32 steps, 205.7 -> 186.6 us; a fp32 decode call, gated, 28 query
      // and 4 KV heads, 7 x 104 tokens 19.3 -> 15.5 us, one of 33 464 tokens, 16 heads on 1, 41.4 -> 36.9 us; the same sums to the bit.)
      static_assert(EPL == 8 && LPR == 16);
      float part[GB][2];
#pragma unroll
      for (int g = 0; g < GB; ++g) {
        const TwoValues m16 = swap16(m[g]), l16 = swap16(l[g]);
        const float M16 = fmaxf(m16.a, m16.b);
        const float a16 = exp2_or_zero(m16.a, M16), b16 = exp2_or_zero(m16.b, M16);
        float four[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const TwoValues x = deal16(acc[g][e], acc[g][e + 4]);
          four[e] = x.a * a16 + x.b * b16;
        }
        const TwoValues m32 = swap32(M16), l32 = swap32(l16.a * a16 + l16.b * b16);
        m[g] = fmaxf(m32.a, m32.b);
        const float a32 = exp2_or_zero(m32.a, m[g]), b32 = exp2_or_zero(m32.b, m[g]);
        l[g] = l32.a * a32 + l32.b * b32;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const TwoValues x = deal32(four[e], four[e + 2]);
          part[g][e] = x.a * a32 + x.b * b32;
        }
      }
      __syncthreads();   // previous segment's readers are done with the LDS buffers
      {
        const int e = (rg & 1) * 4 + (rg >> 1) * 2;        // the lane's two columns are its group's e and e + 1
        const int at = (e / EPC * LPR + c) * EPC + e % EPC;
#pragma unroll
        for (int g = 0; g < GB; ++g) {
          *reinterpret_cast<float2*>(reinterpret_cast<float*>(sm_o[wave][g]) + at) = make_float2(part[g][0], part[g][1]);
          if (lane == 0) { sm_m[wave][g] = m[g]; sm_l[wave][g] = l[g]; }
        }
      }
      __syncthreads();
      // merge the four wavefronts, four outputs of a head per thread; emit the final output or a partial for the combine pass
      constexpr int kAlign = 4 * sizeof(T);                // (a caller's output may start at any element)
      const bool out_aligned = (reinterpret_cast<uintptr_t>(out) & (kAlign - 1)) == 0;
#pragma unroll
      for (int it = 0; it < kPasses; ++it) {
        const int idx = tid + it * kBlock, g = idx >> 5, d4 = idx & 31;
        if (g >= gcount) break;
        float M = sm_m[0][g];
#pragma unroll
        for (int w = 1; w < 4; ++w) M = fmaxf(M, sm_m[w][g]);
        floatx4 O = floatx4{0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float sc = exp2_or_zero(sm_m[w][g], M);
          O += sc * sm_o[w][g][d4];
          L += sc * sm_l[w][g];
        }
        if (whole_pair) {
          T* dst = out + ((int64_t)b * dv.n_q_heads + h * G + gb + g) * kHeadDim + d4 * 4;
          floatx4 r = O / L;
          if (two_pass) {
            if (pass == 0) { held[it] = r; continue; }
            r = pd.gate * held[it] + (1.f - pd.gate) * r;
          }
          if constexpr (sizeof(T) == 4) {
            if (out_aligned) {
              *reinterpret_cast<floatx4*>(dst) = r;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) dst[e] = r[e];
            }
          } else {
            const uint2 four = make_uint2(bf16_pair(r[0], r[1]), bf16_pair(r[2], r[3]));
            if (out_aligned) {
              *reinterpret_cast<uint2*>(dst) = four;
            } else {
              dst[0] = (T)four.x;
              dst[1] = (T)(four.x >> 16);
              dst[2] = (T)four.y;
              dst[3] = (T)(four.y >> 16);
            }
          }
        } else {
          const int64_t slot = (int64_t)wg + pi;
          *reinterpret_cast<floatx4*>(dv.part_o + pass * dv.part_set_o + (slot * G + gb + g) * kHeadDim + d4 * 4) = O;
          if (d4 == 0) {
            dv.part_m[pass * dv.part_set_ml + slot * G + gb + g] = M;
            dv.part_l[pass * dv.part_set_ml + slot * G + gb + g] = L;
          }
        }
      }
      }   // pass
    }
    u = seg_end;
    ++pi;
    pd = pd_next;
    if (u < u_end)
      while (pd.unit_end <= u) pd = pairs[++pi];       // pairs of inactive slots own no units
  }
}

template <typename T, bool FUSED>
hipError_t launch_t(const DeviceView& dv, int layer, const void* q, void* out, float scale_log2, const void* k_new,
                    const void* v_new, int grow, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(dv.n_wg), block(kBlock);
  const T *qp = (const T*)q, *kp = (const T*)k_new, *vp = (const T*)v_new;
  T* op = (T*)out;
  const int G = dv.group;
  // (without events: the plain launch, which a stream capture can record)
#define RLKV_LAUNCH_VALU(GB)                                                                                         \
  do {                                                                                                               \
    if (e0 || e1)                                                                                                    \
      hipExtLaunchKernelGGL((decode_valu_kernel<T, GB, FUSED>), grid, block, 0, stream, e0, e1, 0, dv, layer, qp,   \
                            op, scale_log2, kp, vp, grow);                                                           \
    else                                                                                                             \
      hipLaunchKernelGGL((decode_valu_kernel<T, GB, FUSED>), grid, block, 0, stream, dv, layer, qp, op, scale_log2, \
                         kp, vp, grow);                                                                              \
  } while (0)
  if (G <= 1) RLKV_LAUNCH_VALU(1);
  else if (G <= 2) RLKV_LAUNCH_VALU(2);
  else if (G <= 4) RLKV_LAUNCH_VALU(4);
  else if (G == 7) RLKV_LAUNCH_VALU(7);
  else RLKV_LAUNCH_VALU(8);
#undef RLKV_LAUNCH_VALU
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_valu(const DeviceView& dv, int layer, const void* q, void* out, float scale_log2,
                              const void* k_new, const void* v_new, int grow, hipStream_t stream, hipEvent_t ev_start,
                              hipEvent_t ev_stop) {
  if (dv.dtype == RLKV_F32)
    return k_new ? launch_t<float, true>(dv, layer, q, out, scale_log2, k_new, v_new, grow, stream, ev_start, ev_stop)
                 : launch_t<float, false>(dv, layer, q, out, scale_log2, k_new, v_new, grow, stream, ev_start, ev_stop);
  return k_new ? launch_t<uint16_t, true>(dv, layer, q, out, scale_log2, k_new, v_new, grow, stream, ev_start, ev_stop)
               : launch_t<uint16_t, false>(dv, layer, q, out, scale_log2, k_new, v_new, grow, stream, ev_start, ev_stop);
}

}  // namespace rlkv
