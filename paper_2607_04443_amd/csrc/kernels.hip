// gfx950 (MI355X, CDNA4) kernels of the performer unit attention.
//
//  kv_append       writes a segment's K/V into its cache pages; NORM_ROPE keys
//                  get per-head RMS-norm, the gamma weight and (t,h,w) rotary
//                  positions in fp32 before the bf16 store; V is stored
//                  transposed per page ([d][slot]).
//  unit_attn       video queries: flash attention over the visible pages with
//                  v_mfma_f32_16x16x32_bf16, K/V pages staged through a ring
//                  of LDS stages, softmax in the exp2 domain under a shift
//                  fixed in advance or a lazily raised running maximum.
//  audio_attn      the few audio queries: memory-bound split-KV, one wave per
//                  key range, v_mfma_f32_16x16x32_bf16 straight from registers.
//  combine         log-sum-exp merge of split-KV partials.
//
// The attention is the performer's per-step attention over its K/V cache
// (Wan-Streamer v0.2, Sec. 3); block-causal visibility (Fig. 1 caption) is
// resolved on the host into the list of visible pages.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <type_traits>
#include <utility>

#include "ws_kernels.hpp"

namespace ws {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kNegInf = -__builtin_inff();
// Largest logit bound (log2 units) used as a fixed softmax shift.
constexpr float kShiftBoundMax = 40.0f;
// Above it the video kernel's shift is a running maximum, raised when a logit
// exceeds it by more than this (so p <= 2^8).
constexpr float kRaiseAbove = 8.0f;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2 r = __builtin_convertvector((f32x2){lo, hi}, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max and sum over lanes l, l ^ 16 (kLane = 16) or l, l ^ 32 (v_permlane*_swap:
// no LDS round trip)
template <int kLane>
__device__ __forceinline__ float pair_max(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = kLane == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                             : __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int kLane>
__device__ __forceinline__ float pair_sum(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = kLane == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                             : __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// max over the wave (rotations within a row of 16, then the swaps)
template <int kRor>
__device__ __forceinline__ float ror_max(float v) {
  const int u = __float_as_int(v);
  return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(u, u, 0x120 + kRor, 0xf, 0xf, false)));
}
__device__ __forceinline__ float wave_max(float v) {
  return pair_max<32>(pair_max<16>(ror_max<1>(ror_max<2>(ror_max<4>(ror_max<8>(v))))));
}
// sum over the 16 lanes of a row, in every lane
template <int kRor>
__device__ __forceinline__ float ror_add(float v) {
  const int u = __float_as_int(v);
  return v + __int_as_float(__builtin_amdgcn_update_dpp(u, u, 0x120 + kRor, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_sum(float v) { return ror_add<1>(ror_add<2>(ror_add<4>(ror_add<8>(v)))); }
// |x|^2 of the lane's words, in fp32 products and sums
__device__ __forceinline__ float norm2_fma(u32x4 w) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = bf16_lo(w[i]), hi = bf16_hi(w[i]);
    s = fmaf(lo, lo, s);
    s = fmaf(hi, hi, s);
  }
  return s;
}
// the same by the dot product instruction, added to acc: for bounds only (its
// rounding and subnormals are the instruction's own)
__device__ __forceinline__ float norm2_words(u32x4 w, float acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t x = w[i];
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, x), acc, false);
  }
  return acc;
}

// (cos, sin) of rotary pair p (0..63) for a token at position pos (t, h, w).
__device__ __forceinline__ float2 rope_cs(const RopeTables& r, int p, int pt, int ph, int pw) {
  const int p0 = r.pairs[0], p01 = r.pairs[0] + r.pairs[1];
  if (p < p0) return r.tab[0][pt * r.pairs[0] + p];
  if (p < p01) return r.tab[1][ph * r.pairs[1] + (p - p0)];
  return r.tab[2][pw * r.pairs[2] + (p - p01)];
}

// Clamps a token's (t, h, w) into the table; flags a clamp.
__device__ __forceinline__ void clamp_pos(const RopeTables& r, int t, int h, int w, uint32_t* flags,
                                          int& pt, int& ph, int& pw) {
  const int ct = min(max(t, 0), r.max_pos[0] - 1);
  const int ch = min(max(h, 0), r.max_pos[1] - 1);
  const int cw = min(max(w, 0), r.max_pos[2] - 1);
  if ((ct != t) | (ch != h) | (cw != w)) atomicOr(flags, kFlagPositionClamped);
  pt = ct;
  ph = ch;
  pw = cw;
}

// Loads a token's (t, h, w), clamped into the table; flags a clamp.
__device__ __forceinline__ void load_pos(const RopeTables& r, const int32_t* positions, int tok,
                                         uint32_t* flags, int& pt, int& ph, int& pw) {
  clamp_pos(r, positions[3 * tok + 0], positions[3 * tok + 1], positions[3 * tok + 2], flags, pt, ph, pw);
}

typedef const __attribute__((address_space(4))) AppendSeg* const_append_seg;
typedef const __attribute__((address_space(4))) AppendArgs* const_append_args;

// The append launch's arguments, read in place from the kernel argument
// segment (the kernel's only argument is the AppendArgs): with run-time
// indexes into the by-value argument the compiler copies all of it to
// private memory.
__device__ __forceinline__ const_append_args append_args() {
  return (const_append_args)__builtin_amdgcn_kernarg_segment_ptr();
}

// Four rotary pairs (4 c .. 4 c + 3) of a token: their (cos, sin).  A pair's
// band is a select on its index, not a branch, so that the loads of several
// tokens are in flight together.
__device__ __forceinline__ void rope_pairs(const RopeTables& r, int c, const int (&pos)[3], float2 (&cs)[4]) {
  const int p0 = r.pairs[0], p01 = p0 + r.pairs[1];
  const float2* row[3] = {r.tab[0] + static_cast<int64_t>(pos[0]) * r.pairs[0],
                          r.tab[1] + static_cast<int64_t>(pos[1]) * r.pairs[1] - p0,
                          r.tab[2] + static_cast<int64_t>(pos[2]) * r.pairs[2] - p01};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = 4 * c + i;
    cs[i] = (p < p0 ? row[0] : p < p01 ? row[1] : row[2])[p];
  }
}

// RMS norm, gamma and rotation of one row's eight dims (x, dims 8 c .. of the 16
// lanes of the row), times scale, rounded once to bf16.
__device__ __forceinline__ u32x4 norm_rope_row(u32x4 x, const float (&g)[8], float eps, const float2 (&cs)[4],
                                               float scale) {
  const float inv = rsqrtf(row_sum(norm2_fma(x)) * (1.0f / kHeadDim) + eps);
  u32x4 y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float y0 = bf16_lo(x[i]) * inv * g[2 * i];
    const float y1 = bf16_hi(x[i]) * inv * g[2 * i + 1];
    y[i] = pack_bf16((y0 * cs[i].x - y1 * cs[i].y) * scale, (y0 * cs[i].y + y1 * cs[i].x) * scale);
  }
  return y;
}

// A segment's rows of one tile as the append's arithmetic takes them: 16 lanes
// per token row (lane c: dims 8 c ..), rows rr, rr + 16, rr + 32, rr + 48.
struct AppendRows {
  u32x4 x[4];
  int pos[4][3];
};
__device__ __forceinline__ void load_rows(const_append_seg sg, int tok0, int head, bool norm_rope, int c, int rr,
                                          AppendRows& r) {
  const uint16_t* src = sg->k;
  const int64_t tok_stride = sg->tok_stride;
  const int n_tokens = sg->n_tokens;
  const int32_t* positions = sg->positions;
  src += head * sg->head_stride + 8 * c;
  if (norm_rope) {
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
      const int tok = min(tok0 + pass * 16 + rr, n_tokens - 1);
#pragma unroll
      for (int b = 0; b < 3; ++b) r.pos[pass][b] = positions[3 * tok + b];
    }
  }
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int tok = tok0 + pass * 16 + rr;
    r.x[pass] = tok < n_tokens ? *reinterpret_cast<const u32x4*>(src + tok * tok_stride) : (u32x4){0u, 0u, 0u, 0u};
  }
}
__device__ __forceinline__ void load_gamma(const_append_seg sg, int c, float (&g)[8]) {
  const float* gamma = sg->gamma;
  const float4 g0 = *reinterpret_cast<const float4*>(gamma + 8 * c);
  const float4 g1 = *reinterpret_cast<const float4*>(gamma + 8 * c + 4);
  g[0] = g0.x; g[1] = g0.y; g[2] = g0.z; g[3] = g0.w;
  g[4] = g1.x; g[5] = g1.y; g[6] = g1.z; g[7] = g1.w;
}
// store(pass, slot, words) for the tile's 64 rows: normed, rotated and scaled
// (two rows' table entries in flight at a time, which keeps the registers to
// six blocks per CU), or scaled only.
template <class F>
__device__ __forceinline__ void rotate_rows(const RopeTables& rope, uint32_t* flags, const_append_seg sg, int tok0,
                                            float scale, int c, int rr, AppendRows& r, F&& store) {
  float g[8];
  load_gamma(sg, c, g);
  const float eps = sg->eps;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    float2 cs[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // (a row past the end holds the last token's positions)
      int (&p)[3] = r.pos[2 * half + k];
      int q[3];
      clamp_pos(rope, p[0], p[1], p[2], flags, q[0], q[1], q[2]);
      rope_pairs(rope, c, q, cs[k]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int pass = 2 * half + k, slot = pass * 16 + rr;
      store(pass, slot, norm_rope_row(r.x[pass], g, eps, cs[k], scale));
    }
  }
}

// Query preparation, one block of an append launch: tokens 64 chunk ..
// 64 chunk + 63 of query set si, one head, 16 threads per token row as in
// the key path below.  Q'' = RoPE(RMSNorm(Q) * gamma, positions) * scale *
// log2(e) (mode 3) or Q * scale * log2(e) (mode 2), in fp32, rounded once to
// bf16: the attention kernels' own query prologue, done once per step
// instead of once per workgroup that reads the queries.
__device__ __forceinline__ void prepare_queries(const RopeTables& rope, uint32_t* flags, const_append_seg sg,
                                                int chunk, int head) {
  const int n_tokens = sg->n_tokens;
  const bool norm_rope = (sg->mode & 1) != 0;
  const float scale = sg->scale_log2;
  const int t = threadIdx.x, c = t & 15, rr = t >> 4;
  const int tok0 = chunk * kPageTokens;
  AppendRows r;
  load_rows(sg, tok0, head, norm_rope, c, rr, r);
  uint16_t* const dst = sg->q_out + head * sg->out_head_stride + 8 * c;
  const int64_t out_tok_stride = sg->out_tok_stride;
  auto put = [&](int, int slot, u32x4 y) {
    const int tok = tok0 + slot;
    if (tok < n_tokens) *reinterpret_cast<u32x4*>(dst + tok * out_tok_stride) = y;
  };
  if (norm_rope) {
    rotate_rows(rope, flags, sg, tok0, scale, c, rr, r, put);
  } else {
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
      u32x4 y;
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = pack_bf16(bf16_lo(r.x[pass][i]) * scale, bf16_hi(r.x[pass][i]) * scale);
      put(pass, pass * 16 + rr, y);
    }
  }
}

// ------------------------------------------------------------------------- //
// kv_append: one (item, head) tile of an append launch, an item being a K/V
// page or a 64-token chunk of a query set of one of up to
// AppendArgs::kMaxSegs segments.  256 threads; vt and wave_norm2 are the
// block's LDS, free again when the call returns.
//
// What bounds it: memory (a step of 924 queries and 1,180 new tokens over 40
// heads moves 67 MB, 10 us at the rate of a large copy) and, before that, the
// chain position -> table entry -> rotation of each row.  So a tile's loads are
// all issued first, its table entries two rows ahead by a select instead of a
// branch per band, and row sums are DPP rotations instead of LDS permutes.
// V is transposed through LDS: rows of 128 d, the 16-byte chunk d / 8 of row r
// at position (d / 8) ^ (r / 8), so that the 32-bit reads of a d pair over the
// eight row groups hit different banks; two rows of V^T per thread halve the
// LDS reads.  Measured (that step / its queries alone / 12 heads, 256
// queries and 320 tokens): 17.1 / 7.8 / 7.1 us before, 14.4 / 7.6 / 5.2 us.
// With registers for six blocks per CU it spills (25.7 us); grids of 3, 5 and 8
// blocks per CU take 15.6, 16.1 and 15.9 us for the first, 4 takes 14.9 in the
// same run.
// ------------------------------------------------------------------------- //
__device__ __forceinline__ void append_tile(const_append_args A, int item, int head, uint16_t (*vt)[kHeadDim],
                                            float* wave_norm2) {
  const const_append_seg sg = A->seg + A->blk_seg[item];
  RopeTables rope;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    rope.tab[b] = A->rope.tab[b];
    rope.max_pos[b] = A->rope.max_pos[b];
    rope.pairs[b] = A->rope.pairs[b];
  }
  uint32_t* const flags = A->flags;
  if (sg->mode & kAppendQuery) {
    prepare_queries(rope, flags, sg, A->blk_page[item], head);
    return;
  }
  const int num_heads = A->num_heads;
  const int page = A->pages[item];
  const int64_t tok_stride = sg->tok_stride;
  const int n_tokens = sg->n_tokens;
  const bool norm_rope = sg->mode == 1;
  const int tok0 = A->blk_page[item] * kPageTokens;
  const int64_t tile = (static_cast<int64_t>(page) * num_heads + head) * kPageHeadElems;
  uint16_t* kdst = A->kpool + tile;
  uint16_t* vdst = A->vpool + tile;
  const int t = threadIdx.x, c = t & 15, rr = t >> 4;

  // all loads of the tile are issued up front: positions, K rows, V rows
  AppendRows r;
  load_rows(sg, tok0, head, norm_rope, c, rr, r);
  const uint16_t* const src_v = sg->v + head * sg->head_stride + 8 * c;
  u32x4 vx[4];
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int tok = tok0 + pass * 16 + rr;
    vx[pass] = tok < n_tokens ? *reinterpret_cast<const u32x4*>(src_v + tok * tok_stride) : (u32x4){0u, 0u, 0u, 0u};
  }

  // K: alongside, the largest squared norm of the stored rows of the tile.  It
  // only bounds scores (the softmax shift), so the dot product instruction does:
  // exact products, fp32 sums; squares it may flush (|k| < 1.1e-19) could move
  // a bound by less than 32 for the largest |q| whose square is finite.
  float norm2 = 0.f;
  auto put = [&](int, int slot, u32x4 y) {
    *reinterpret_cast<u32x4*>(kdst + k_tile_index(slot, 8 * c)) = y;
    norm2 = fmaxf(norm2, row_sum(norm2_words(y, 0.f)));
  };
  if (norm_rope) {
    // empty slots hold zeros whatever gamma and eps are
    rotate_rows(rope, flags, sg, tok0, 1.0f, c, rr, r, [&](int pass, int slot, u32x4 y) {
      put(pass, slot, tok0 + slot < n_tokens ? y : (u32x4){0u, 0u, 0u, 0u});
    });
  } else {
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) put(pass, pass * 16 + rr, r.x[pass]);
  }
  norm2 = pair_max<32>(pair_max<16>(norm2));
  if ((t & 63) == 0) wave_norm2[t >> 6] = norm2;
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int row = pass * 16 + rr;
    *reinterpret_cast<u32x4*>(&vt[row][8 * (c ^ (row >> 3))]) = vx[pass];
  }
  __syncthreads();
  // thread: d pair d2 (two rows of V^T), slots 8 tc .. 8 tc + 7
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ch = t + 256 * i, tc = ch & 7, d = 2 * (ch >> 3);
    uint32_t w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      w[j] = *reinterpret_cast<const uint32_t*>(&vt[8 * tc + j][8 * ((d >> 3) ^ tc) + (d & 7)]);
    u32x4 lo, hi;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lo[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x05040100u);
      hi[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x07060302u);
    }
    *reinterpret_cast<u32x4*>(vdst + v_tile_index(8 * tc, d)) = lo;
    *reinterpret_cast<u32x4*>(vdst + v_tile_index(8 * tc, d + 1)) = hi;
  }
  if (t == 0)
    A->knorm2[static_cast<int64_t>(page) * num_heads + head] =
        fmaxf(fmaxf(wave_norm2[0], wave_norm2[1]), fmaxf(wave_norm2[2], wave_norm2[3]));
}

// The launch: a grid of a few blocks per CU that loop over the launch's
// (item, head) tiles, consecutive tiles being the heads of one item.  (One
// block per tile made the launch as long as dispatching its ~1,400 short
// blocks: their average life was about an eighth of the launch.)
__global__ __launch_bounds__(256) void kv_append_kernel(const AppendArgs args) {
  (void)args;  // read in place, through append_args()
  __shared__ __attribute__((aligned(16))) uint16_t vt[kPageTokens][kHeadDim];
  __shared__ float wave_norm2[4];
  const const_append_args A = append_args();
  const int heads = A->num_heads;
  const int n_tiles = A->n_blocks * heads;
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    append_tile(A, tile / heads, tile % heads, vt, wave_norm2);
    __syncthreads();  // vt and wave_norm2 are rewritten by the next tile
  }
}

// ------------------------------------------------------------------------- //
// unit_attn (video): query tiles of 256, 192 or 128 rows on 4 waves (one per
// SIMD) of 64, 48 or 32 queries, a last tile of at most 128 rows on waves of
// 32; 64-key pages through LDS.
//
// Per wave and page, with lane l = 16 g + i (i = query column of a 16-query
// subtile, g = lane group) and v_mfma_f32_16x16x32_bf16:
//   S^T[16 keys][16 q]  = K Q''^T    4 key tiles x 4 k-steps per subtile
//   O^T[16 d][16 q]    += V^T P^T    8 d tiles x 2 key chunks of 32
//   l[q]               += 1 P^T      2 key chunks (the row sums, on the matrix
//                                    pipe: over the same bf16 P as O)
// Row m = 4 g' + r of key tile t holds key 32 (t/2) + 8 g' + 4 (t%2) + r
// (audio_key below), so registers r of tiles 2c and 2c + 1 in lane group g are
// keys 32 c + 8 g + 0..7: directly the B operand of the P*V MFMA of chunk c.
//
// What bounds it: at the long windows the chip's power limit, then the matrix
// pipe.  The MFMA shape, the operand reuse and the row sums follow from that.
// Measured on the page loop alone (256 CUs, random operands, no page loads):
//   32x32x16 MFMAs, 8 waves x 32 rows               1.455 us per page
//   32x32x16 MFMAs, 4 waves x 64 rows               1.43  us
//   16x16x32 MFMAs, 8 waves x 32 rows               1.33-1.41 us
//   16x16x32 MFMAs, 4 waves x 64 rows, v_dot2 sums  1.30-1.40 us
//   16x16x32 MFMAs, 4 waves x 64 rows, MFMA sums    1.23-1.27 us
// (16x16x32 sustains 2170-2240 TFLOP/s on random register operands, 32x32x16
// 1950; 64 rows per wave halve the LDS operand reads; a row-sum MFMA costs
// less than the 16 v_dot2 it replaces.)
// ------------------------------------------------------------------------- //

// f(Const<0>), ..., f(Const<N - 1>), unrolled by construction.
template <int N>
struct Const {
  static constexpr int value = N;
};
template <class F, int... Is>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, Is...>) {
  (f(Const<Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Row m (lane index i) of key tile t: the key it holds.
__device__ __forceinline__ int audio_key(int t, int m) {
  return 32 * (t >> 1) + 8 * (m >> 2) + 4 * (t & 1) + (m & 3);
}

// LDS stages of the video kernel (a ring of five pages, 160 KB: the previous
// page, whose V^T the pipelined schedule still reads, the current page, the
// next page, already complete so that its first operands can be read before
// the page barrier, and the two after it in flight), filled by direct
// global->LDS loads (global_load_lds_dwordx4: lane l of a wave writes 16
// bytes at base + 16 l).  A stage is a K tile, then a V tile:
//   K    [64 rows][16 chunks]: row 16 t + m holds key audio_key(t, m); its
//        logical chunk c (dims 8c..8c+7) sits at position c ^ m.
//   V^T  [128 d][8 chunks]: logical chunk c (keys 8c..8c+7) of row d sits at
//        position c ^ ((d >> 1) & 7).
// Either way the 16 lanes of a lane group read 16 distinct 16-byte bank groups.
constexpr int kStages = 5;
constexpr uint32_t kStageBytes = 2 * kPageHeadElems * 2;
constexpr uint32_t kStageV = kPageHeadElems * 2;  // offset of the V tile
__shared__ __attribute__((aligned(1024))) uint16_t g_stages[kStages * 2 * kPageHeadElems];

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Read-only for a whole launch: accessed through the constant address space
// so that uniform reads become scalar loads.
typedef const __attribute__((address_space(4))) int2* const_page_list;

// The call's visible page list: in device memory, or in the kernel
// arguments themselves (the kernel's only argument is the AttnArgs, at the
// start of the kernel argument segment; addressing it through the segment
// pointer keeps the compiler from copying the argument to private memory).
__device__ __forceinline__ const_page_list page_list(const AttnArgs& a) {
  if (a.pages) return (const_page_list)a.pages;
  const __attribute__((address_space(4))) char* seg =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  return (const_page_list)(seg + offsetof(AttnArgs, inline_pages));
}

// LDS byte offset of a pointer into a __shared__ object.
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p));
}
// 16 bytes at an LDS byte offset.
__device__ __forceinline__ bf16x8 lds_read16(uint32_t off) {
  return as_bf16x8(*(const __attribute__((address_space(3))) u32x4*)off);
}

__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// The video kernel's MFMAs.  The S tiles sit in vector registers (the softmax
// reads them; the build asks for that form of the MFMA builtins), O and l in
// accumulation registers, by inline asm: the compiler's own choice puts all
// of them in one bank, and every exponential or every O update then goes
// through a copy.  The compiler does not see the matrix pipe's latency behind
// the asm: O and l are read or written by other instructions only across
// mfma_drain(), and a P word or another vector operand is written at least
// two instructions ahead of the asm that reads it.
__device__ __forceinline__ void mfma_s(f32x4& d, bf16x8 a, bf16x8 b, const f32x4& c) {
  d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ void mfma_o(f32x4& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
// The first product into an accumulator (C = 0).
__device__ __forceinline__ void mfma_o_first(f32x4& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(d) : "v"(a), "v"(b));
}
// An accumulator times a factor, in place: multiplied in plain code it would
// move to vector registers, and the page loop around the branch with it.
__device__ __forceinline__ void scale_acc(f32x4& d, float f) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float x = d[r], t;
    asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                 : "+a"(x), "=&v"(t)
                 : "v"(f));
    d[r] = x;
  }
}
// A value the compiler cannot carry over from an earlier computation: the
// epilogue recomputes its addresses instead of keeping them live across the
// page loop.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
// Waits until every MFMA issued so far has written its result (and, between a
// vector write and a following MFMA, until the write is visible to it).
__device__ __forceinline__ void mfma_drain() {
  sched_fence();
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  sched_fence();
}

// What one page's iteration addresses, computed a little at a time during the
// iteration before it, so that the page boundary holds nothing but the
// barrier.
struct PageCtx {
  uint32_t k[4];        // LDS offsets of this lane's operand reads: K, per k-step (key tile t: + 4096 t)
  uint32_t v;           // V^T chunk 0 (d tile dt: + 2048 dt)
  uint32_t vp;          // V^T chunk 1 of the page before
  const uint16_t* ldk;  // the loads to issue, of the page three ahead: K and V tile,
  const uint16_t* ldv;
  uint32_t lds;         // and their LDS offset
};

// A workgroup's share of one query tile's (head, page) units, lo .. lo + n - 1
// in head-major order: one continuous stream of pages through the LDS ring,
// whatever heads it crosses.  A unit's list entry is its tile index
// (page * H + head) and the page's valid tokens; each lane holds the entries
// of two units out of a window of 128, read with v_readlane, so that the page
// loop has no scalar load to wait for (scalar loads and LDS reads share a
// counter that only a full wait can order).
struct VideoStream {
  const_page_list pages;
  FastDiv div_pages;
  int num_heads, n_pages, page0, lo, n;
  int lane;
  uint32_t ent[2];        // entries of units 64 k + lane of the window (tile index << 7 | valid tokens)
  int raw_head[2], raw_page[2], raw_valid[2];  // what ent is made of
  float kn2[2];           // key-norm maxima (squared) of the first window's units
  const uint16_t* kpool;
  const uint16_t* vpool;
  uint32_t dma_k, dma_v;  // this lane's source byte offsets within a tile (block 0)
  uint32_t k_read, v_read;  // this lane's operand read offsets within a stage (k-step 0, chunk 0)
  uint32_t lds0;          // LDS offset of the wave's first block in stage 0
  int at;                 // stream index of the current page
  uint32_t stage;         // its stage's LDS offset
  uint32_t valid;         // valid tokens of pages at .. at + 3, a byte each
  PageCtx c;              // the current page's context
};

// (Past the end: the last unit's entry.  No lane-dependent branch here or
// anywhere else inside the page loops' regions: with one, the compiler
// serialises the uniform branches around it and keeps the accumulators of both
// sides.)
__device__ __forceinline__ uint32_t stream_entry(const VideoStream& s, int k) {
  const uint32_t x = s.lo + min(k, s.n - 1), head = fast_div(x, s.div_pages);
  const int pi = s.page0 + static_cast<int>(x - head * s.n_pages);
  return ((s.pages[pi].x * s.num_heads + head) << 7) | static_cast<uint32_t>(s.pages[pi].y);
}
// The first window: its list entries requested, then combined.
__device__ __forceinline__ void stream_request(VideoStream& s) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint32_t x = s.lo + min(64 * k + s.lane, s.n - 1), head = fast_div(x, s.div_pages);
    const int pi = s.page0 + static_cast<int>(x - head * s.n_pages);
    s.raw_head[k] = head;
    s.raw_page[k] = s.pages[pi].x;
    s.raw_valid[k] = s.pages[pi].y;
  }
}
__device__ __forceinline__ void stream_combine(VideoStream& s) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
    s.ent[k] = ((s.raw_page[k] * s.num_heads + s.raw_head[k]) << 7) | static_cast<uint32_t>(s.raw_valid[k]);
}
// Entry of stream index k (uniform, inside the window).
__device__ __forceinline__ uint32_t stream_peek(const VideoStream& s, int k) {
  const uint32_t e0 = __builtin_amdgcn_readlane(s.ent[0], k & 63), e1 = __builtin_amdgcn_readlane(s.ent[1], k & 63);
  return (k & 64) ? e1 : e0;
}
// Moves the window when the page to look up next, at + 4, enters a new half:
// it replaces the half that lies two behind.
__device__ __forceinline__ void stream_reach(VideoStream& s) {
  const int k = s.at + 4;
  if ((k & 63) == 0 && k >= 128) {
    uint32_t e = stream_entry(s, k + s.lane);
    asm volatile("" : "+v"(e));  // waited for here, not at every later use
    if (k & 64) s.ent[1] = e; else s.ent[0] = e;
  }
}
constexpr uint32_t kRingBytes = kStages * kStageBytes;
__device__ __forceinline__ uint32_t ring_add(uint32_t stage, uint32_t k) {
  const uint32_t x = stage + k * kStageBytes;
  return x >= kRingBytes ? x - kRingBytes : x;
}

// One direct load: each lane's 16 bytes at sbase + voff go to LDS at
// lds + kLdsAdd + 16 * lane.  Written as inline asm: with the compiler's own
// LDS-DMA intrinsic in flight, every later LDS read waits for lgkmcnt(0),
// which serializes the MFMA operand reads.  Completion is tracked by the
// explicit vmcnt waits below.  M0 is the asm's own: nothing the compiler
// emits in this kernel keeps a value in it.
template <uint32_t kLdsAdd>
__device__ __forceinline__ void dma16(const uint16_t* sbase, uint32_t voff, uint32_t lds) {
  // both are wave-uniform by construction; make that visible to the compiler
  // (readfirstlane returns int: widen through uint32_t, never sign-extend)
  lds = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(lds));
  const uint64_t b = reinterpret_cast<uint64_t>(sbase);
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32)));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b)));
  sbase = reinterpret_cast<const uint16_t*>((static_cast<uint64_t>(hi) << 32) | lo);
  asm volatile(
      "s_add_u32 m0, %2, %3\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(sbase), "s"(lds), "i"(kLdsAdd)
      : "memory", "scc");
}

// The direct loads of one page: 32 blocks of 1 KB, 8 per wave (block 4 i +
// wave of each tile, i = 0..3).  Block b of K is rows 4 b .. 4 b + 3, i.e.
// rows 4 wave .. of key tile i (keys 32 (i / 2) + 4 (i % 2) + 8 wave ..); block
// b of V^T is rows d = 8 b .. 8 b + 7.
constexpr int kDmaPerPage = 8;  // direct loads per wave and page
template <int kPart>            // 0..3: K blocks, 4..7: V blocks
__device__ __forceinline__ void issue_load(const VideoStream& s, const PageCtx& c) {
  if constexpr (kPart < 4) {
    constexpr uint32_t src = 2u * k_tile_index(32 * (kPart >> 1) + 4 * (kPart & 1), 0);
    dma16<4096u * kPart>(c.ldk, s.dma_k + src, c.lds);
  } else {
    constexpr uint32_t src = 2u * v_tile_index(0, 32 * (kPart - 4));
    dma16<kStageV + 4096u * (kPart - 4)>(c.ldv, s.dma_v + src, c.lds);
  }
}
__device__ __forceinline__ void issue_page(const VideoStream& s, const PageCtx& c) {
  static_for<kDmaPerPage>([&](auto i) __attribute__((always_inline)) { issue_load<decltype(i)::value>(s, c); });
}
// The load part of a context: the page with entry e into ring stage `stage`.
__device__ __forceinline__ void set_load(const VideoStream& s, uint32_t e, uint32_t stage, PageCtx& c) {
  const uint64_t off = static_cast<uint64_t>(e >> 7) << 14;  // 16 KB tiles
  c.ldk = reinterpret_cast<const uint16_t*>(reinterpret_cast<uint64_t>(s.kpool) + off);
  c.ldv = reinterpret_cast<const uint16_t*>(reinterpret_cast<uint64_t>(s.vpool) + off);
  c.lds = __builtin_amdgcn_readfirstlane(s.lds0 + stage);
}

// Waits for this wave's direct loads of every page but the one issued last
// (loads retire in order).  The barrier that follows then makes every wave's
// share visible.
__device__ __forceinline__ void wait_dma_all_but_last_page() {
  static_assert(kDmaPerPage == 8, "vmcnt encoding below");
  __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8), expcnt(7), lgkmcnt(15)
}
__device__ __forceinline__ void wait_dma_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)
// The page barrier alone: no wait for the LDS reads in flight, which belong
// to a page that stays.
__device__ __forceinline__ void page_barrier() {
  sched_fence();
  asm volatile("s_barrier" ::: "memory");
  sched_fence();
}

template <class T>
__device__ __forceinline__ void pin_s(T& x) { asm volatile("" : "+s"(x)); }
template <class T>
__device__ __forceinline__ void pin_v(T& x) { asm volatile("" : "+v"(x)); }

// The rest of a context: operand reads of the page in ring stage `stage`.
__device__ __forceinline__ void set_reads(const VideoStream& s, uint32_t stage, PageCtx& c) {
#pragma unroll
  for (int n = 0; n < 4; ++n) c.k[n] = (s.k_read + stage) ^ (64u * n);
  c.v = s.v_read + stage;
  c.vp = (s.v_read + ring_add(stage, kStages - 1)) ^ 64u;
}

// Starts the stream: key norms of its first window, the loads of its first
// three pages, and the context of its first page.  (Past a stream's end the
// last page is loaded once more, into a stage nothing reads.)
__device__ __forceinline__ void stream_start(const AttnArgs& a, VideoStream& s) {
  stream_combine(s);
#pragma unroll
  for (int k = 0; k < 2; ++k) s.kn2[k] = a.knorm2[s.ent[k] >> 7];  // (past the end: the last unit's)
  if (s.n == 0) return;
  s.valid = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t e = stream_peek(s, min(k, s.n - 1));
    s.valid |= (e & 127u) << (8 * k);
    set_load(s, e, k * kStageBytes, s.c);
    if (k < 3) issue_page(s, s.c);
  }
  set_reads(s, 0, s.c);
}

// A wave's query rows: kQT subtiles of 16.
template <int kQT>
struct VideoState {
  f32x4 o[8][kQT];    // O^T[16 dt + 4 g + r][q]  (accumulation registers)
  f32x4 l[kQT];       // row sums, the same in every register and lane group
  f32x4 s_init[kQT];  // -m in every register: the S tiles start at the exp2 argument
  float m[kQT];       // softmax shift of row q
  bf16x8 q[kQT][4];   // Q''[q][32 s + 8 g .. + 8]
  // across pages
  f32x4 s3[kQT];      // S tile 3 of the previous page
  u32x4 p1[kQT];      // P words of its chunk 1 (tile 2's done)
  bf16x8 ring[4];     // operands in flight (slot = step % 4)
  // rows under a running maximum
  bool any_lazy;      // some row of the wave is one
  uint32_t raised;    // subtiles whose O and l wait to be scaled (bit j) ...
  float scale[kQT];   // ... by this, row q
  u32x4 ones;         // bf16 ones (an opaque value: not rematerialised in front of an MFMA)
};
// Operand reads are issued this many steps ahead.  (Six, through eight
// registers, gives the narrower waves nothing: they are not latency-bound.)
constexpr int kRingAhead = 3;

// The queries live in accumulation registers (an MFMA reads its operands from
// either bank), which leaves the vector registers to the softmax.
template <int kQT>
__device__ __forceinline__ void pin_queries(VideoState<kQT>& st) {
#pragma unroll
  for (int j = 0; j < kQT; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) asm volatile("" : "+a"(st.q[j][t]));
}

// Two adjacent exponentials to one word of P.
// The pins here and at the exponentials and S tiles keep them where they are
// scheduled: the compiler would sink them past the branches of a page tail.
__device__ __forceinline__ void put_word(u32x4& p, int word, float lo, float hi) {
  uint32_t w = pack_bf16(lo, hi);
  pin_v(w);
  p[word] = w;
}

// O and l of the rows raised at the last check, scaled to their new m.  No MFMA
// on them may be under way (the page loop: the last one was issued eight steps
// before).
template <int kQT>
__device__ __forceinline__ void scale_raised(VideoState<kQT>& st) {
  if (st.raised == 0) return;
  sched_fence();
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    if (st.raised >> j & 1) {
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) scale_acc(st.o[dt][j], st.scale[j]);
      scale_acc(st.l[j], st.scale[j]);
    }
  }
  st.raised = 0;
  asm volatile("s_nop 7" ::: "memory");
  sched_fence();
}

// One page, software-pipelined across pages so that the softmax work is
// spread over the MFMA steps.  Iteration p (page p from the current stage,
// V^T of page p - 1 from the one before it): 32 steps of one LDS operand read
// (kRingAhead steps ahead, through a ring of four registers that runs on
// across the page barrier) and kQT MFMAs, one per subtile:
//   steps  0- 7  S tiles 0 and 1 of p       exponentials of tile 3 of p - 1
//   steps  8-15  P*V of p - 1, chunk 1      tile 0 of p (from step 10)
//   steps 16-23  S tiles 2 and 3 of p       tile 1 of p
//   steps 24-31  P*V of p, chunk 0          tile 2 of p (from step 26)
// The subtiles' exponentials run in streams of two subtiles, one exponential per
// stream and step (two in steps 10, 11, 26 and 27), each issued behind an MFMA
// of its own (an exponential takes 8 of the 16 cycles of an MFMA, a pack 4)
// and packed behind the next one, and each slot ends in a scheduling fence,
// so that the emitted order is the program order.  Every P word is complete
// before the P*V step that reads it.  Steps 0-7 also issue the direct loads
// of page p + 3 into the stage freed by page p - 2; at the end of the page
// each wave waits for its loads of page p + 2, so every load has two pages to
// land and the next page is complete a page before it is used.  One barrier
// per page.
// kFirst: a range's first page: no page p - 1.
//
// Rows under a running maximum (st.any_lazy; after the first page the kLazy
// form of the loop): the range's first 32 keys set a row's m to their maximum.
// From then on the largest S (a difference to m) of every chunk is taken in the
// steps that have no exponential (8 and 9, 24 and 25) and compared ahead of
// the chunk's exponentials; where it exceeds kRaiseAbove, the row takes it as
// its new m, and what O and l hold by then is scaled to it between the P*V of
// the chunk before and the chunk's own (after step 23, and after step 7 of the
// next page: their MFMAs are long done by then, and no P word is rounded
// twice).  Every choice is the row's own, so a row's result does not depend on
// the rows that share its wave, and a row under a fixed shift never exceeds it.
// A raised row's largest weight is exactly 1 instead of rounded like the others,
// which keeps the error of sharp attention down; a threshold of 4 gives more
// such rows and more raises (9% slower), one of 16 fewer (0.3% more error).
// Measured, 40 heads, 920 rows, 139 pages, us a step at query norm weights 1
// (no such row), 3, 4 and 7: 157, 190, 207, 223; without raises the loop takes
// 170.  (A shift fixed at 16 below the logit bound took 154 up to 4, but rounded
// the largest weight, and out of its reach, from 5 on, the range ran unpipelined
// under a running maximum: 344 to 455.)
template <int kQT, bool kFirst, bool kLazy>
__device__ __forceinline__ void video_iter(VideoState<kQT>& st, VideoStream& s) {
  const int n_valid = static_cast<int>(s.valid & 0xffu);
  const bool tail = n_valid < kPageTokens;
  const PageCtx c = s.c;
  PageCtx nx;
  pin_queries(st);
  pin_v(st.ones);
  page_barrier();
  // operand of step n
  auto oread = [&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    if constexpr (n >= 32) return lds_read16(nx.k[n - 32]);
    else if constexpr (n < 8) return lds_read16(c.k[n & 3] + 4096u * (n >> 2));
    else if constexpr (n < 16) return lds_read16(c.vp + 2048u * (n - 8));
    else if constexpr (n < 24) return lds_read16(c.k[n & 3] + 4096u * (2 + ((n - 16) >> 2)));
    else return lds_read16(c.v + 2048u * (n - 24));
  };
  if constexpr (kFirst) {
    static_for<kRingAhead>([&](auto n) __attribute__((always_inline)) { st.ring[decltype(n)::value] = oread(n); });
  }
  f32x4 sa[4][kQT];
  u32x4 p0[kQT], p1n[kQT];
  float cm[kQT], top;  // largest S of the lane's keys of a chunk, and of all subtiles
  // exponential x of a stream: tile x / 8, subtile (x / 4) % 2, register x % 4
  // (the last stream of an odd kQT has one subtile)
  constexpr int kStreams = (kQT + 1) / 2;
  float e[kStreams][32];

  auto exp_x = [&](auto kc_, auto xc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc_)::value, x = decltype(xc)::value;
    constexpr int t = x >> 3, j = 2 * k + ((x >> 2) & 1), r = x & 3;
    if constexpr (j >= kQT) {
    } else if constexpr (t == 3) {
      if constexpr (!kFirst) { e[k][x] = fast_exp2(st.s3[j][r]); pin_v(e[k][x]); }
    } else {
      e[k][x] = fast_exp2(sa[t][j][r]);
      pin_v(e[k][x]);
    }
  };
  auto pack_x = [&](auto kc_, auto xc) __attribute__((always_inline)) {  // words of exponentials x, x + 1 (x even)
    constexpr int k = decltype(kc_)::value, x = decltype(xc)::value;
    constexpr int t = x >> 3, j = 2 * k + ((x >> 2) & 1), word = 2 * (t & 1) + ((x & 3) >> 1);
    if constexpr (j >= kQT) {
    } else if constexpr (t == 3) {
      if constexpr (!kFirst) put_word(st.p1[j], word, e[k][x], e[k][x + 1]);
    } else if constexpr (t == 2) {
      put_word(p1n[j], word, e[k][x], e[k][x + 1]);
    } else {
      put_word(p0[j], word, e[k][x], e[k][x + 1]);
    }
  };
  // the largest S of chunk a (tiles a, a + 1) in this lane
  auto take_max = [&](auto jc, auto ac) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value, a = decltype(ac)::value;
    const f32x4 &x = sa[a][j], &y = sa[a + 1][j];
    cm[j] = fmaxf(fmaxf(fmaxf(fmaxf(x[0], x[1]), x[2]), fmaxf(fmaxf(x[3], y[0]), y[1])), fmaxf(y[2], y[3]));
    pin_v(cm[j]);
  };
  auto take_top = [&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    top = j == 0 ? cm[0] : fmaxf(top, cm[j]);
    pin_v(top);
  };
  auto take_all = [&](auto ac) __attribute__((always_inline)) {
    static_for<kQT>([&](auto jc) __attribute__((always_inline)) {
      take_max(jc, ac);
      take_top(jc);
    });
  };
  // New maxima for the rows of a chunk that exceed theirs by too much.
  auto raise = [&](auto ac) __attribute__((always_inline)) {
    constexpr int a = decltype(ac)::value;
    st.raised = 0;
#pragma unroll
    for (int j = 0; j < kQT; ++j) {
      const float row = pair_max<32>(pair_max<16>(cm[j]));
      if (__any(row > kRaiseAbove)) {
        const float up = row > kRaiseAbove ? row : 0.f;  // (0: nothing of the row changes)
        st.raised |= 1u << j;
        st.scale[j] = fast_exp2(-up);
        st.m[j] += up;
        const float neg = -st.m[j];
        st.s_init[j] = (f32x4){neg, neg, neg, neg};
        sa[a][j] -= up;
        sa[a + 1][j] -= up;
      }
    }
  };
  // a page tail's work on the chunk of tiles a and a + 1, and its maxima
  auto check_chunk = [&](auto ac) __attribute__((always_inline)) {
    constexpr int a = decltype(ac)::value;
    if (tail) {
      // logits of slots at or past n_valid become -inf, so they weigh exactly
      // 0 (a correction subtracted from the row sum afterwards would cancel
      // for rows whose logits all sit far below the shift)
      const int lim = n_valid - 8 * (opaque(s.lane) >> 4);
#pragma unroll
      for (int t = a; t < a + 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int j = 0; j < kQT; ++j)
            sa[t][j][r] = 32 * (t >> 1) + 4 * (t & 1) + r >= lim ? kNegInf : sa[t][j][r];
      if constexpr (kLazy) take_all(ac);
    }
    if constexpr (kFirst) {
      if (st.any_lazy) {
        take_all(ac);
        if constexpr (a == 0) {
#pragma unroll
          for (int j = 0; j < kQT; ++j) {
            // (a page's first chunk has a valid key; clamped all the same)
            const float row = fmaxf(pair_max<32>(pair_max<16>(cm[j])), -3.0e38f);
            const float up = st.m[j] < 0.f ? row : 0.f;  // (m < 0: not set yet)
            st.m[j] = st.m[j] < 0.f ? row : st.m[j];
            const float neg = -st.m[j];
            st.s_init[j] = (f32x4){neg, neg, neg, neg};
            sa[0][j] -= up;
            sa[1][j] -= up;
          }
        } else {
          raise(ac);
        }
      }
    } else if constexpr (kLazy) {
      if (__any(top > kRaiseAbove)) raise(ac);
    }
    sched_fence();
  };

  // the next page's context, one small piece per step
  int look = 0;
  uint32_t ent = 0, st_next = 0;
  auto next_ctx = [&](auto oc) __attribute__((always_inline)) {
    constexpr int o = decltype(oc)::value;
    if constexpr (o == 12) { look = min(s.at + 4, s.n - 1); pin_s(look); }
    if constexpr (o == 13) { ent = __builtin_amdgcn_readlane(s.ent[0], look & 63); pin_s(ent); }
    if constexpr (o == 14) {
      const uint32_t e1 = __builtin_amdgcn_readlane(s.ent[1], look & 63);
      ent = (look & 64) ? e1 : ent;
      pin_s(ent);
    }
    if constexpr (o == 15) { st_next = ring_add(s.stage, 1); pin_s(st_next); }
    if constexpr (o == 16) {
      nx.ldk = reinterpret_cast<const uint16_t*>(reinterpret_cast<uint64_t>(s.kpool) + (static_cast<uint64_t>(ent >> 7) << 14));
      pin_s(nx.ldk);
    }
    if constexpr (o == 17) {
      nx.ldv = reinterpret_cast<const uint16_t*>(reinterpret_cast<uint64_t>(s.vpool) + (static_cast<uint64_t>(ent >> 7) << 14));
      pin_s(nx.ldv);
    }
    if constexpr (o == 18) { nx.lds = s.lds0 + ring_add(st_next, 3); pin_s(nx.lds); }
    if constexpr (o == 19) { nx.k[0] = s.k_read + st_next; pin_v(nx.k[0]); }
    if constexpr (o == 20) { nx.k[1] = nx.k[0] ^ 64u; pin_v(nx.k[1]); }
    if constexpr (o == 21) { nx.k[2] = nx.k[0] ^ 128u; pin_v(nx.k[2]); }
    if constexpr (o == 22) { nx.k[3] = nx.k[0] ^ 192u; pin_v(nx.k[3]); }
    if constexpr (o == 23) { nx.v = s.v_read + st_next; pin_v(nx.v); }
    if constexpr (o == 24) { nx.vp = c.v ^ 64u; pin_v(nx.vp); }
    if constexpr (o == 28) { s.valid = __builtin_amdgcn_readfirstlane((s.valid >> 8) | ((ent & 127u) << 24)); }
  };
  static_for<32>([&](auto oc) __attribute__((always_inline)) {
    constexpr int o = decltype(oc)::value;
    const bf16x8 a = st.ring[o & 3];
    static_for<kQT>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value, k = j >> 1;
      constexpr bool even = (j & 1) == 0, last = j == kQT - 1;
      // ---- the MFMA ----
      if constexpr (o < 8 || (o >= 16 && o < 24)) {
        constexpr int t = (o < 8 ? 0 : 2) + ((o & 7) >> 2);
        if constexpr ((o & 3) == 0) mfma_s(sa[t][j], a, st.q[j][0], st.s_init[j]);
        else mfma_s(sa[t][j], a, st.q[j][o & 3], sa[t][j]);
        pin_v(sa[t][j]);
      } else if constexpr (o < 16) {
        if constexpr (!kFirst) {
          mfma_o(st.o[o - 8][j], a, as_bf16x8(st.p1[j]));
          if constexpr (o == 15) mfma_o(st.l[j], as_bf16x8(st.ones), as_bf16x8(st.p1[j]));
        }
      } else {
        if constexpr (kFirst) mfma_o_first(st.o[o - 24][j], a, as_bf16x8(p0[j]));
        else mfma_o(st.o[o - 24][j], a, as_bf16x8(p0[j]));
        if constexpr (o == 31) {
          if constexpr (kFirst) mfma_o_first(st.l[j], as_bf16x8(st.ones), as_bf16x8(p0[j]));
          else mfma_o(st.l[j], as_bf16x8(st.ones), as_bf16x8(p0[j]));
        }
      }
      sched_fence();
      // ---- this slot's share of the rest ----
      if constexpr (kLazy && (o == 8 || o == 24)) take_max(jc, Const<o == 8 ? 0 : 2>{});
      if constexpr (kLazy && (o == 9 || o == 25)) take_top(jc);
      if constexpr (j == 1) {
        constexpr int n = o + kRingAhead;
        if constexpr (!(kFirst && n >= 8 && n < 16)) st.ring[n & 3] = oread(Const<n>{});
      }
      if constexpr (even) {
        if constexpr (o < 8) exp_x(Const<k>{}, Const<24 + o>{});
        else if constexpr (o == 10) exp_x(Const<k>{}, Const<0>{});
        else if constexpr (o == 11) exp_x(Const<k>{}, Const<2>{});
        else if constexpr (o >= 12 && o < 24) exp_x(Const<k>{}, Const<o - 8>{});
        else if constexpr (o == 26) exp_x(Const<k>{}, Const<16>{});
        else if constexpr (o == 27) exp_x(Const<k>{}, Const<18>{});
        else if constexpr (o >= 28) exp_x(Const<k>{}, Const<o - 8>{});
      }
      if constexpr (!even || last) {
        if constexpr (o < 8 && (o & 1)) pack_x(Const<k>{}, Const<24 + o - 1>{});
        else if constexpr (o == 10) exp_x(Const<k>{}, Const<1>{});
        else if constexpr (o == 11) { exp_x(Const<k>{}, Const<3>{}); pack_x(Const<k>{}, Const<0>{}); }
        else if constexpr (o == 12) pack_x(Const<k>{}, Const<2>{});
        else if constexpr (o > 12 && o < 24 && (o & 1)) pack_x(Const<k>{}, Const<o - 9>{});
        else if constexpr (o == 26) exp_x(Const<k>{}, Const<17>{});
        else if constexpr (o == 27) { exp_x(Const<k>{}, Const<19>{}); pack_x(Const<k>{}, Const<16>{}); }
        else if constexpr (o == 28) pack_x(Const<k>{}, Const<18>{});
        else if constexpr (o > 28 && (o & 1)) pack_x(Const<k>{}, Const<o - 9>{});
      }
      if constexpr (last) {
        if constexpr (o < kDmaPerPage) issue_load<o>(s, c);
        next_ctx(oc);
        if constexpr (o == 14 || o == 30) pin_v(st.ones);
      }
      sched_fence();
    });
    if constexpr (o == 9) check_chunk(Const<0>{});
    if constexpr (o == 25) check_chunk(Const<2>{});
    if constexpr (kLazy && (o == 7 || o == 23)) scale_raised(st);
  });
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    st.s3[j] = sa[3][j];
    st.p1[j] = p1n[j];
  }
  // After a range's first page everything is waited for: a load the compiler
  // knows of and believes in flight on entry to the page loop would be waited
  // for in every iteration, with all the direct loads behind it.
  if constexpr (kFirst) wait_dma_all();
  else wait_dma_all_but_last_page();
  s.c = nx;
  s.at += 1;
  s.stage = st_next;
  stream_reach(s);
}

// Finishes the last page of a range (its stage is the one before the
// stream's current): tile 3's exponentials, then the P*V of chunk 1.
template <int kQT>
__device__ __forceinline__ void video_flush(VideoState<kQT>& st, const VideoStream& s) {
  const uint32_t v1 = s.c.vp;
  mfma_drain();
#pragma unroll
  for (int j = 0; j < kQT; ++j)
#pragma unroll
    for (int r = 0; r < 4; r += 2)
      put_word(st.p1[j], 2 + (r >> 1), fast_exp2(st.s3[j][r]), fast_exp2(st.s3[j][r + 1]));
  bf16x8 v[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) v[dt] = lds_read16(v1 + 2048u * dt);
  pin_v(st.ones);
  mfma_drain();
#pragma unroll
  for (int j = 0; j < kQT; ++j) mfma_o(st.l[j], as_bf16x8(st.ones), as_bf16x8(st.p1[j]));
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int j = 0; j < kQT; ++j) mfma_o(st.o[dt][j], v[dt], as_bf16x8(st.p1[j]));
  mfma_drain();
}

// One segment of a video workgroup's stream: the query tile of rows
// [q_lo, min(q_lo + 256, q_hi)) of head `head` against n pages of the stream,
// which are key range `seg` of the ranges that split this head's pages
// (`whole`: the only one; q_hi ends the tile's query class).  With one range
// the output is written in bf16; otherwise the softmax-normalised partial and
// its log-sum-exp go to the split-KV workspace for the combine kernel.
struct VideoSeg {
  int head, n, seg, q_lo, q_hi;
  bool whole;
};

// A wave's query rows as the call gives them: raw[j][s] = Q[row j][32 s + 8 g .. + 8].
template <int kQT>
struct RawQueries {
  u32x4 raw[kQT][4];
  bool rider[kQT];  // rider rows (at and past rq_row0): prepared rows of their own
  bool ok[kQT];
  int3 pos[kQT];
};
template <int kQT, bool kPrepared>
__device__ __forceinline__ void fetch_queries(const AttnArgs& a, const VideoSeg& sg, int wrow, int lane,
                                              RawQueries<kQT>& x) {
  const int lane_o = opaque(lane), g = lane_o >> 4, i16 = lane_o & 15;
  // row j's pointer is the first row's plus 16 j token strides (uniform);
  // rows past the end read the zero block (zeros cost the matrix pipe little)
  const uint16_t* qp = a.q + sg.head * a.q_head_stride + (wrow + i16) * a.q_tok_stride + 8 * g;
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    const int row = wrow + 16 * j + i16;
    x.ok[j] = row < sg.q_hi;
    x.rider[j] = false;
    const uint16_t* p = x.ok[j] ? qp + 16 * j * a.q_tok_stride : a.zeros + 8 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s) x.raw[j][s] = *reinterpret_cast<const u32x4*>(p + 32 * s);
    x.pos[j] = make_int3(0, 0, 0);
    if (!kPrepared && a.mode == 1 && x.ok[j])
      x.pos[j] = make_int3(a.positions[3 * row], a.positions[3 * row + 1], a.positions[3 * row + 2]);
  }
  if (a.n_rq > 0 && wrow + 16 * kQT > a.rq_row0) {  // rider rows among them
#pragma unroll
    for (int j = 0; j < kQT; ++j) {
      const int q = wrow + 16 * j + i16 - a.rq_row0;
      if (q >= 0 && q < a.n_rq) {
        const uint16_t* p = a.rq + q * a.rq_tok_stride + sg.head * a.rq_head_stride + 8 * g;
#pragma unroll
        for (int s = 0; s < 4; ++s) x.raw[j][s] = *reinterpret_cast<const u32x4*>(p + 32 * s);
        x.rider[j] = true;
      }
    }
  }
}

// The prepared queries, st.q[j][s] = Q''[row j][32 s + 8 g .. + 8], by the
// call's query mode (kPrepared: 2, given as they are, else 0 or 1); rider rows
// (at and past rq_row0) come prepared.
template <int kQT, bool kPrepared>
__device__ __forceinline__ void prepare_rows(const AttnArgs& a, const RawQueries<kQT>& x, int g, VideoState<kQT>& st) {
  if (kPrepared) {
#pragma unroll
    for (int j = 0; j < kQT; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s) st.q[j][s] = as_bf16x8(x.raw[j][s]);
    return;
  }
  if (a.mode == 0) {
#pragma unroll
    for (int j = 0; j < kQT; ++j) {
      const float sc = x.rider[j] ? 1.0f : a.scale_log2;  // riders: x 1 is exact
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = pack_bf16(bf16_lo(x.raw[j][s][i]) * sc, bf16_hi(x.raw[j][s][i]) * sc);
        st.q[j][s] = as_bf16x8(w);
      }
    }
    return;
  }
  // Norm and rotation.  The lane's 16 pairs are 16 s + 4 g + i; a pair's band
  // is a select on its index (no branch), the table rows' offsets are per row.
  const int p0 = a.rope.pairs[0], p01 = p0 + a.rope.pairs[1];
  float inv[kQT];
  const float2* row[kQT][3];
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    int pt = 0, ph = 0, pw = 0;
    if (x.ok[j] && !x.rider[j]) clamp_pos(a.rope, x.pos[j].x, x.pos[j].y, x.pos[j].z, a.flags, pt, ph, pw);
    row[j][0] = a.rope.tab[0] + static_cast<int64_t>(pt) * a.rope.pairs[0];
    row[j][1] = a.rope.tab[1] + static_cast<int64_t>(ph) * a.rope.pairs[1] - p0;
    row[j][2] = a.rope.tab[2] + static_cast<int64_t>(pw) * a.rope.pairs[2] - p01;
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) ss += norm2_fma(x.raw[j][s]);
    ss = pair_sum<32>(pair_sum<16>(ss));
    inv[j] = rsqrtf(ss * (1.0f / kHeadDim) + a.eps);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float4 g0 = *reinterpret_cast<const float4*>(a.gamma + 32 * s + 8 * g);
    const float4 g1 = *reinterpret_cast<const float4*>(a.gamma + 32 * s + 8 * g + 4);
    const float gam[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    float2 cs[kQT][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = 16 * s + 4 * g + i;
#pragma unroll
      for (int j = 0; j < kQT; ++j) cs[j][i] = (p < p0 ? row[j][0] : p < p01 ? row[j][1] : row[j][2])[p];
    }
#pragma unroll
    for (int j = 0; j < kQT; ++j) {
      u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float y0 = bf16_lo(x.raw[j][s][i]) * inv[j] * gam[2 * i];
        const float y1 = bf16_hi(x.raw[j][s][i]) * inv[j] * gam[2 * i + 1];
        w[i] = pack_bf16((y0 * cs[j][i].x - y1 * cs[j][i].y) * a.scale_log2,
                         (y0 * cs[j][i].y + y1 * cs[j][i].x) * a.scale_log2);
      }
      // riders come prepared; a row past the call's end stays all zeros (with
      // eps = 0 its norm gives 0 * inf)
      st.q[j][s] = as_bf16x8(x.ok[j] ? w : x.raw[j][s]);
    }
  }
}

template <int kQT, bool kPrepared>
__device__ __forceinline__ void video_segment(const AttnArgs& a, const VideoSeg& sg, VideoStream& s, int wave) {
  const int wrow = sg.q_lo + wave * 16 * kQT;
  VideoState<kQT> st;
  {
    RawQueries<kQT> raw;
    fetch_queries<kQT, kPrepared>(a, sg, wrow, s.lane, raw);
    prepare_rows<kQT, kPrepared>(a, raw, s.lane >> 4, st);
  }

  // ---- softmax shift ----
  // Logits arrive in the log2 domain (the scale and log2(e) are folded into
  // Q'').  By Cauchy-Schwarz every logit of row q is at most
  // B_q = |Q''_q| * max |k| over the segment's pages (knorm2 holds the
  // squared norms of the stored keys).  Softmax is shift invariant, so B_q
  // serves as the exp2 shift as it stands: p = exp2(s - B_q) <= 1, with no
  // running maximum and no rescale of O.  The row's largest p is at least
  // 2^(-2 B_q), so for B_q <= kShiftBoundMax every weight above 2^-46 of the
  // row maximum stays a normal bf16/fp32 number.  Rows with a larger bound run
  // under a running maximum (video_iter).
  float kn2 = 0.f;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = 64 * k + s.lane;
    if (idx >= s.at && idx < s.at + sg.n) kn2 = fmaxf(kn2, s.kn2[k]);
  }
  for (int k = max(s.at, 128) + s.lane; k < s.at + sg.n; k += 64)
    kn2 = fmaxf(kn2, a.knorm2[stream_entry(s, k) >> 7]);
  kn2 = fminf(wave_max(kn2), 3.0e38f);  // (finite: a zero query's bound is 0)
  bool lazy = false;
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    float qn2 = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) qn2 = norm2_words(__builtin_bit_cast(u32x4, st.q[j][t]), qn2);
    const float bound = sqrtf(pair_sum<32>(pair_sum<16>(qn2)) * kn2);
    const bool is = a.fixed_shift == 0 || bound > kShiftBoundMax;
    lazy = lazy || is;
    st.m[j] = is ? -1.f : bound;  // (-1: to be set by the first keys)
    const float neg = is ? 0.f : -bound;
    st.s_init[j] = (f32x4){neg, neg, neg, neg};
  }
  st.any_lazy = __any(lazy);
  st.raised = 0;
  pin_queries(st);
  st.ones = (u32x4){0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  asm volatile("" : "+v"(st.ones));

  // ---- the segment's pages ----
  if (s.at == 0) wait_dma_all_but_last_page();
  const int end = s.at + sg.n;
  video_iter<kQT, true, false>(st, s);
  // (one-armed branches in turn: of an if-else the compiler keeps both arms'
  // accumulators.  In this order, and with the last scaling in the second arm,
  // the first loop keeps its speed: 40 heads, 920 rows, 139 and 479 pages 132.5 and
  // 443.4 us a step; the other way round 133.8 and 448.0, with the scaling in the
  // flush as well; without the second loop 131.8 and 441.1.)
  if (!st.any_lazy)
    while (s.at < end) video_iter<kQT, false, false>(st, s);
  if (st.any_lazy) {
    while (s.at < end) video_iter<kQT, false, true>(st, s);
    mfma_drain();
    scale_raised(st);
  }
  video_flush<kQT>(st, s);
  if (s.at == s.n) wait_dma_all();  // no direct load may still be writing this workgroup's LDS when it exits

  // ---- epilogue: lane holds O^T[16 dt + 4 g + r][q] ----
  const int lane_e = opaque(s.lane), ge = lane_e >> 4, ie = lane_e & 15;
  const bool riders = a.n_rq > 0 && wrow + 16 * kQT > a.rq_row0;
  // bf16: the output itself, or the partial of a key range: the
  // softmax-normalised O (a convex combination of V rows, so bf16 keeps its
  // range; the merge adds at most one more bf16 rounding of the output's size)
  // and its fp32 log-sum-exp.
  const int64_t part_row = (static_cast<int64_t>(sg.seg) * a.num_heads + sg.head) * a.n_q;
  uint16_t* const base = sg.whole ? a.out + sg.head * a.out_head_stride
                                  : reinterpret_cast<uint16_t*>(a.part_o) + part_row * kHeadDim;
  const int64_t stride = sg.whole ? a.out_tok_stride : kHeadDim;
  uint16_t* const op = base + (wrow + ie) * stride + 16 * (ge & 1) + 8 * (ge >> 1);
#pragma unroll
  for (int j = 0; j < kQT; ++j) {
    const int row = wrow + 16 * j + ie;
    const float l = st.l[j][0];
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const float lse = l > 0.f ? st.m[j] + __log2f(l) : kNegInf;
    if (riders) {  // always a partial, fp32, for the rider rows' own merge
      const int q = row - a.rq_row0;
      if (q >= 0 && q < a.n_rq) {
        const int64_t prow = (static_cast<int64_t>(sg.seg) * a.num_heads + sg.head) * a.n_rq + q;
        float* po = a.rpart_o + prow * kHeadDim + 4 * ge;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<f32x4*>(po + 16 * dt) = st.o[dt][j] * inv;
        if (ge == 0) a.rpart_lse[prow] = lse;
      }
    }
    // Lane groups trade halves of two neighbouring d tiles, so that each lane
    // writes 16 bytes: lane group g of (x[0], x[1]) -> groups (0, 2): d tile
    // dt, (1, 3): dt + 1.
    u32x4 w[4];
#pragma unroll
    for (int dt = 0; dt < 8; dt += 2) {
      uint32_t x[2][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 v = st.o[dt + h][j] * inv;
        x[h][0] = pack_bf16(v[0], v[1]);
        x[h][1] = pack_bf16(v[2], v[3]);
      }
      const auto w0 = __builtin_amdgcn_permlane16_swap(x[0][0], x[1][0], false, false);
      const auto w1 = __builtin_amdgcn_permlane16_swap(x[0][1], x[1][1], false, false);
      w[dt >> 1] = (u32x4){w0[0], w1[0], w0[1], w1[1]};
    }
    if (row < sg.q_hi) {
#pragma unroll
      for (int n = 0; n < 4; ++n) *reinterpret_cast<u32x4*>(op + 16 * j * stride + 32 * n) = w[n];
      if (!sg.whole && ge == 0) a.part_lse[part_row + row] = lse;
    }
  }
}

// The class table, read in place from the kernel arguments (the kernel's only
// argument is the AttnArgs; indexing the by-value argument at a run-time class
// would make the compiler copy it to private memory).
typedef const __attribute__((address_space(4))) AttnClass* const_class_table;
__device__ __forceinline__ const_class_table class_table() {
  const __attribute__((address_space(4))) char* seg =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  return (const_class_table)(seg + offsetof(AttnArgs, cls));
}
// ------------------------------------------------------------------------- //
// audio_attn: the few audio queries, memory-bound.  A workgroup of 4 waves
// takes one (head, 16-query tile, key range); wave w streams pages w, w + 4,
// ... of the range on its own (no LDS staging, no barriers), loading each
// page's valid K rows and V^T columns straight into registers in MFMA
// operand layout, and the four waves merge through LDS at the end.  Two
// workgroups fit a CU, so 8 independent waves per CU keep enough bytes in
// flight to stream the cache from HBM.  Each workgroup writes the partial of
// its key range; the combine kernel merges them.  Where a head is one range its
// workgroup writes the output itself, without the merge's launch (4 us): a CU
// takes 0.45 us per page, so that pays for up to 12 pages.  (On 8 waves
// instead of 4 the same 0.45 us: 8, 16 and 24 pages take 10.6, 13.4 and 17.2 us
// against 9.1, 12.7 and 16.5.)
//
// With lane l = 16 g + i (i = query column, g = lane group), per page:
//   S^T (16 keys x 16 queries) = K Q''^T  4 key tiles x 4 v_mfma_f32_16x16x32_bf16
//   O^T (16 d x 16 queries) += V^T P^T    8 d tiles x 2 key chunks, same MFMA
// Row m = 4 g' + r of key tile t holds key 32 (t/2) + 8 g' + 4 (t%2) + r, so
// that accumulator registers r of tiles 2c and 2c + 1 in lane group g are
// keys 32 c + 8 g + 0..7: exactly the B operand of the P*V MFMA of key chunk c.
// ------------------------------------------------------------------------- //
// Loads of one page's K operands, k[t][s] = K[key(t, i)][32 s + 8 g .. + 8],
// and V^T operands, v[dt][c] = V^T[16 dt + i][32 c + 8 g .. + 8].  Rows and
// columns past n_valid are read from the 1 KB zero block instead (a cache
// hit), so partly filled pages cost only their valid tokens in HBM traffic
// and no load is predicated.
__device__ __forceinline__ void audio_load_k(u32x4 (&k)[4][4], const uint16_t* kt, const uint16_t* zeros,
                                             int n_valid, int g, int i, int lane) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int key = audio_key(t, i);
    const uint16_t* src = key < n_valid ? kt + k_tile_index(key, 8 * g) : zeros + 8 * lane;
    const int step = key < n_valid ? k_tile_index(0, 32) : 0;  // next 32 d
#pragma unroll
    for (int s = 0; s < 4; ++s) k[t][s] = *reinterpret_cast<const u32x4*>(src + step * s);
  }
}
__device__ __forceinline__ void audio_load_v(u32x4 (&v)[8][2], const uint16_t* vt, const uint16_t* zeros,
                                             int n_valid, int g, int i, int lane) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const bool ok = 32 * c + 8 * g < n_valid;
    const uint16_t* src = ok ? vt + v_tile_index(32 * c + 8 * g, i) : zeros + 8 * lane;
    const int step = ok ? v_tile_index(0, 16) : 0;  // next 16 d
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) v[dt][c] = *reinterpret_cast<const u32x4*>(src + step * dt);
  }
}

// S^T of one page's four key tiles.
__device__ __forceinline__ void audio_scores(const u32x4 (&kreg)[4][4], const bf16x8 (&qreg)[4], f32x4 (&sacc)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    sacc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      sacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kreg[t][s]), qreg[s], sacc[t], 0, 0, 0);
  }
}

// Softmax weights of one page (sacc, masked past n_valid here) as bf16 words
// pw (word c of chunk c: keys 32 c + 8 g + 0..7), with the running maximum,
// the row sum (over the same bf16 values the MFMAs consume) and O kept up to
// date.
__device__ __forceinline__ void audio_softmax(f32x4 (&sacc)[4], int n_valid, bool fixed_shift, int g, u32x4 (&pw)[2],
                                              f32x4 (&o)[8], float& m_run, float& l_run) {
  const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
  if (n_valid < kPageTokens) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (audio_key(t, 4 * g + r) >= n_valid) sacc[t][r] = kNegInf;
  }
  float alpha = 1.f;
  if (!fixed_shift) {
    float mx = kNegInf;
#pragma unroll
    for (int t = 0; t < 4; ++t) mx = fmaxf(mx, fmaxf(fmaxf(sacc[t][0], sacc[t][1]), fmaxf(sacc[t][2], sacc[t][3])));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    alpha = m_new == kNegInf ? 1.f : fast_exp2(m_run - m_new);
    m_run = m_new;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt] *= alpha;
  }
  const float m_use = m_run == kNegInf ? 0.f : m_run;
  float psum = 0.f;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4& sc = sacc[2 * c + h];
      const uint32_t w0 = pack_bf16(fast_exp2(sc[0] - m_use), fast_exp2(sc[1] - m_use));
      const uint32_t w1 = pack_bf16(fast_exp2(sc[2] - m_use), fast_exp2(sc[3] - m_use));
      pw[c][2 * h] = w0;
      pw[c][2 * h + 1] = w1;
      psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w0), ones, psum, false);
      psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w1), ones, psum, false);
    }
  l_run = l_run * alpha + psum;
}

__device__ __forceinline__ void audio_pv(const u32x4 (&vreg)[8][2], const u32x4 (&pw)[2], f32x4 (&o)[8]) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(vreg[dt][c]), as_bf16x8(pw[c]), o[dt], 0, 0, 0);
}

// The page loop of the audio path, one wave: pages p_begin, p_begin + step,
// ... (< p_end) of the list, whose first page's operands kreg and vreg hold
// on entry.  Accumulates O^T (o), the running maximum and the row sum of the
// wave's 16 query columns (m_run and l_run as set up by the caller: the
// fixed shift, or -inf for a running maximum).
//
// Each page's K registers are reloaded (for the wave's next page) as soon as
// its S products are issued, and its V^T registers as soon as the P*V
// products are, so both loads of a page are in flight while the wave waits on
// the one before it.
__device__ __forceinline__ void audio_page_loop(const_page_list pages, int p_begin, int p_end, int step,
                                                const uint16_t* kpool, const uint16_t* vpool, int64_t page_stride,
                                                const uint16_t* zeros, const bf16x8 (&qreg)[4], bool fixed_shift,
                                                u32x4 (&kreg)[4][4], u32x4 (&vreg)[8][2], int g, int i16, int lane,
                                                f32x4 (&o)[8], float& m_run, float& l_run) {
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) o[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int pi = p_begin; pi < p_end; pi += step) {
    const int n_valid = pages[pi].y;
    int2 nxt = make_int2(0, 0);  // past the last page: zeros
    if (pi + step < p_end) nxt = make_int2(pages[pi + step].x, pages[pi + step].y);
    f32x4 sacc[4];
    audio_scores(kreg, qreg, sacc);
    audio_load_k(kreg, kpool + nxt.x * page_stride, zeros, nxt.y, g, i16, lane);
    u32x4 pw[2];
    audio_softmax(sacc, n_valid, fixed_shift, g, pw, o, m_run, l_run);
    audio_pv(vreg, pw, o);
    audio_load_v(vreg, vpool + nxt.x * page_stride, zeros, nxt.y, g, i16, lane);
  }
}

// The softmax shift bound of the audio path: |Q''_q| times the largest key
// norm (squared: kn2, the lane's part of the pages), the same in all lane
// groups of a row.
__device__ __forceinline__ float audio_bound(const bf16x8 (&qreg)[4], float kn2) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) kn2 = fmaxf(kn2, __shfl_xor(kn2, off));
  float qn2 = 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const u32x4 w = __builtin_bit_cast(u32x4, qreg[s]);
#pragma unroll
    for (int k = 0; k < 4; ++k) qn2 += bf16_lo(w[k]) * bf16_lo(w[k]) + bf16_hi(w[k]) * bf16_hi(w[k]);
  }
  qn2 += __shfl_xor(qn2, 16);
  qn2 += __shfl_xor(qn2, 32);
  return sqrtf(qn2 * kn2);
}

__global__ __launch_bounds__(256, 2) void audio_attn_kernel(const AttnArgs a) {
  __shared__ float sm_o[4][kHeadDim][16];  // per wave O^T, merged at the end
  __shared__ float sm_ml[4][2][16];        // per wave (m, l) per query
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, i16 = lane & 15;
  const int bid = blockIdx.x;
  const int split = bid % a.n_splits;
  const int rest = bid / a.n_splits;
  const int qtile = rest % a.n_qtiles;
  const int head = rest / a.n_qtiles;
  const int p_begin = split * a.pages_per_split + wave;
  const int p_end = min(a.n_pages, (split + 1) * a.pages_per_split);
  const_page_list pages = page_list(a);
  const int64_t page_stride = static_cast<int64_t>(a.num_heads) * kPageHeadElems;
  const uint16_t* kpool = a.kpool + head * kPageHeadElems;
  const uint16_t* vpool = a.vpool + head * kPageHeadElems;

  // the wave's first page is requested before the query prologue
  u32x4 kreg[4][4], vreg[8][2];
  {
    int2 pg = make_int2(0, 0);  // no page: zeros
    if (p_begin < p_end) pg = make_int2(pages[p_begin].x, pages[p_begin].y);
    audio_load_k(kreg, kpool + pg.x * page_stride, a.zeros, pg.y, g, i16, lane);
    audio_load_v(vreg, vpool + pg.x * page_stride, a.zeros, pg.y, g, i16, lane);
  }

  // Q prologue: lane holds Q''[q][32 s + 8 g + j], s = 0..3, with the
  // softmax scale and log2(e) folded in
  const int q = qtile * kAudioQTile + i16;
  const bool q_ok = q < a.n_q;
  u32x4 qraw[4];
  const uint16_t* qp = a.q + q * a.q_tok_stride + head * a.q_head_stride + 8 * g;
#pragma unroll
  for (int s = 0; s < 4; ++s)
    qraw[s] = q_ok ? *reinterpret_cast<const u32x4*>(qp + 32 * s) : (u32x4){0u, 0u, 0u, 0u};
  bf16x8 qreg[4];
  if (a.mode == 1) {
    int pt = 0, ph = 0, pw = 0;
    if (q_ok) load_pos(a.rope, a.positions, q, a.flags, pt, ph, pw);
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x0 = bf16_lo(qraw[s][k]), x1 = bf16_hi(qraw[s][k]);
        ss += x0 * x0 + x1 * x1;
      }
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    const float inv = rsqrtf(ss * (1.0f / kHeadDim) + a.eps);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int d0 = 32 * s + 8 * g;
      const float4 g0 = *reinterpret_cast<const float4*>(a.gamma + d0);
      const float4 g1 = *reinterpret_cast<const float4*>(a.gamma + d0 + 4);
      const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
      u32x4 w;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float y0 = bf16_lo(qraw[s][k]) * inv * gg[2 * k];
        const float y1 = bf16_hi(qraw[s][k]) * inv * gg[2 * k + 1];
        const float2 cs = rope_cs(a.rope, (d0 >> 1) + k, pt, ph, pw);
        w[k] = pack_bf16((y0 * cs.x - y1 * cs.y) * a.scale_log2, (y0 * cs.y + y1 * cs.x) * a.scale_log2);
      }
      qreg[s] = as_bf16x8(q_ok ? w : (u32x4){0u, 0u, 0u, 0u});
    }
  } else if (a.mode == 2) {  // prepared: Q'' as given
#pragma unroll
    for (int s = 0; s < 4; ++s) qreg[s] = as_bf16x8(qraw[s]);
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 w;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        w[k] = pack_bf16(bf16_lo(qraw[s][k]) * a.scale_log2, bf16_hi(qraw[s][k]) * a.scale_log2);
      qreg[s] = as_bf16x8(w);
    }
  }

  // Softmax shift, as in the video kernel: the logit bound |Q''_q| max |k|
  // (log2 units) over the wave's pages when it is at most kShiftBoundMax for
  // all 16 queries, else a running maximum.
  float kn2 = 0.f;
  for (int pi = p_begin + 4 * lane; pi < p_end; pi += 256)
    kn2 = fmaxf(kn2, a.knorm2[static_cast<int64_t>(pages[pi].x) * a.num_heads + head]);
  const float bound = audio_bound(qreg, kn2);
  const bool fixed_shift = a.fixed_shift != 0 && __all(bound <= kShiftBoundMax);
  float m_run = fixed_shift ? bound : kNegInf, l_run = 0.f;

  f32x4 o[8];
  audio_page_loop(pages, p_begin, p_end, 4, kpool, vpool, page_stride, a.zeros, qreg, fixed_shift, kreg, vreg,
                  g, i16, lane, o, m_run, l_run);

  // merge the four waves: lane holds O^T[16 dt + 4 g + r][q] of its keys
  float l_w = l_run + __shfl_xor(l_run, 16);
  l_w += __shfl_xor(l_w, 32);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int r = 0; r < 4; ++r) sm_o[wave][16 * dt + 4 * g + r][i16] = o[dt][r];
  if (g == 0) {
    sm_ml[wave][0][i16] = m_run;
    sm_ml[wave][1][i16] = l_w;
  }
  __syncthreads();
  // thread t: query t % 16, d = 8 (t / 16) .. + 8
  const int qi = tid & 15, d0 = 8 * (tid >> 4);
  float mw[4], big = kNegInf;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    mw[w] = sm_ml[w][0][qi];
    big = fmaxf(big, mw[w]);
  }
  float ew[4], l_tot = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    ew[w] = big == kNegInf ? 0.f : fast_exp2(mw[w] - big);
    l_tot += ew[w] * sm_ml[w][1][qi];
  }
  const int qq = qtile * kAudioQTile + qi;
  if (qq >= a.n_q) return;
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  f32x4 out0, out1;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += ew[w] * sm_o[w][d0 + k][qi];
    if (k < 4) out0[k] = v * inv; else out1[k - 4] = v * inv;
  }
  if (a.audio_direct) {  // the only range: what the merge of one range gives (a row without weight: zeros)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      out0[k] = l_tot > 0.f ? out0[k] + 0.f : 0.f;  // (+ 0: the merge's sum turns -0 to 0)
      out1[k] = l_tot > 0.f ? out1[k] + 0.f : 0.f;
    }
    *reinterpret_cast<u32x4*>(a.out + qq * a.out_tok_stride + head * a.out_head_stride + d0) =
        (u32x4){pack_bf16(out0[0], out0[1]), pack_bf16(out0[2], out0[3]), pack_bf16(out1[0], out1[1]),
                pack_bf16(out1[2], out1[3])};
    return;
  }
  const int64_t row = (static_cast<int64_t>(split) * a.num_heads + head) * a.n_q + qq;
  float* po = a.part_o + row * kHeadDim + d0;
  *reinterpret_cast<f32x4*>(po) = out0;
  *reinterpret_cast<f32x4*>(po + 4) = out1;
  if (tid < 16) a.part_lse[row] = l_tot > 0.f ? big + __log2f(l_tot) : kNegInf;
}

// ------------------------------------------------------------------------- //
// The rider rows' own pages (entries rx_page0 .. of the page list, visible to
// them only), inside the video kernel: the last wave of the last query tile's
// workgroups attends them with the audio path's arithmetic; each of a head's
// first rx_ranges ranges takes its part of them and writes it as a key range of
// its own (after the head's ranges of the shared pages) of the rows' fp32
// partials.  A wave without rows does so between the page loads it issues
// anyway: one page's registers are requested in one iteration of the stream
// and consumed in the next (the request in the same iteration as a computation
// would hold up the page barrier), so the other waves never wait for it.  (With
// three such waves attending three pages each ahead of their first page
// barrier, the barrier waited 7 us.)  A wave with rows does it after its
// segments: a page or two, against a launch of the audio kernel (6 us).
// ------------------------------------------------------------------------- //
struct RiderWork {
  int head, range, p0, np;  // pages [p0, p0 + np) of the list
  int item, n_items;        // item: (16-row subtile, page), the pages innermost
  bool loaded;              // the item's operands are requested
  bool fixed_shift;
  float m, l;
  u32x4 k[4][4], v[8][2];
  f32x4 o[8];
  bf16x8 q[4];
};

__device__ __forceinline__ void rider_request(const AttnArgs& a, RiderWork& w, int lane) {
  const int g = lane >> 4, i16 = lane & 15;
  const const_page_list pages = page_list(a);
  const int per = max(w.np, 1), sub = w.item / per, pg = w.item - sub * per;
  if (pg == 0) {
    const int q = 16 * sub + i16;
    const bool ok = q < a.n_rq;
    const uint16_t* qp = a.rq + q * a.rq_tok_stride + w.head * a.rq_head_stride + 8 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      w.q[s] = as_bf16x8(ok ? *reinterpret_cast<const u32x4*>(qp + 32 * s) : (u32x4){0u, 0u, 0u, 0u});
    float kn2 = 0.f;
    for (int pi = w.p0 + lane; pi < w.p0 + w.np; pi += 64)
      kn2 = fmaxf(kn2, a.knorm2[static_cast<int64_t>(pages[pi].x) * a.num_heads + w.head]);
    const float bound = audio_bound(w.q, kn2);
    w.fixed_shift = a.fixed_shift != 0 && __all(bound <= kShiftBoundMax);
    w.m = w.fixed_shift ? bound : kNegInf;
    w.l = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) w.o[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  int2 p = make_int2(0, 0);  // no page: zeros
  if (pg < w.np) p = make_int2(pages[w.p0 + pg].x, pages[w.p0 + pg].y);
  const int64_t tile = (static_cast<int64_t>(p.x) * a.num_heads + w.head) * kPageHeadElems;
  audio_load_k(w.k, a.kpool + tile, a.zeros, p.y, g, i16, lane);
  audio_load_v(w.v, a.vpool + tile, a.zeros, p.y, g, i16, lane);
  w.loaded = true;
}

__device__ __forceinline__ void rider_compute(const AttnArgs& a, RiderWork& w, int lane) {
  const int g = lane >> 4, i16 = lane & 15;
  const const_page_list pages = page_list(a);
  const int per = max(w.np, 1), sub = w.item / per, pg = w.item - sub * per;
  f32x4 sacc[4];
  u32x4 pw[2];
  audio_scores(w.k, w.q, sacc);
  audio_softmax(sacc, pg < w.np ? pages[w.p0 + pg].y : 0, w.fixed_shift, g, pw, w.o, w.m, w.l);
  audio_pv(w.v, pw, w.o);
  if (pg == per - 1) {  // lane holds O^T[16 dt + 4 g + r][q]
    float l = w.l + __shfl_xor(w.l, 16);
    l += __shfl_xor(l, 32);
    const int q = 16 * sub + i16;
    if (q < a.n_rq) {
      const int64_t row = (static_cast<int64_t>(w.range) * a.num_heads + w.head) * a.n_rq + q;
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      float* po = a.rpart_o + row * kHeadDim + 4 * g;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<f32x4*>(po + 16 * dt) = w.o[dt] * inv;
      if (g == 0) a.rpart_lse[row] = l > 0.f ? w.m + __log2f(l) : kNegInf;
    }
  }
  ++w.item;
  w.loaded = false;
}

// The rider rows' pages that range sg.seg of the n_seg of its head takes.
__device__ __forceinline__ void rider_share(const AttnArgs& a, const VideoSeg& sg, int n_seg, RiderWork& w) {
  const int parts = min(n_seg, a.rx_ranges);
  w.item = 0;
  w.n_items = 0;
  w.loaded = false;
  if (sg.seg >= parts) return;
  w.head = sg.head;
  w.range = n_seg + sg.seg;
  w.p0 = a.rx_page0 + a.rx_pages * sg.seg / parts;
  w.np = a.rx_page0 + a.rx_pages * (sg.seg + 1) / parts - w.p0;
  w.n_items = ((a.n_rq + 15) / 16) * max(w.np, 1);
}
__device__ __forceinline__ void rider_rest(const AttnArgs& a, RiderWork& w, int lane) {
  while (w.item < w.n_items) {
    if (!w.loaded) rider_request(a, w, lane);
    rider_compute(a, w, lane);
  }
}

// A segment for a wave without query rows: it issues its share of the page
// loads and attends the rider rows' pages (n_seg > 0: the head's ranges).
__device__ __forceinline__ void video_idle_segment(const AttnArgs& a, const VideoSeg& sg, VideoStream& s, int n_seg) {
  RiderWork w;
  w.item = w.n_items = 0;
  w.loaded = false;
  if (n_seg > 0) rider_share(a, sg, n_seg, w);
  if (s.at == 0) wait_dma_all_but_last_page();
  for (int k = 0; k < sg.n; ++k) {
    page_barrier();
    if (w.item < w.n_items) {
      if (w.loaded) rider_compute(a, w, s.lane);
      else rider_request(a, w, s.lane);
    }
    issue_page(s, s.c);
    const uint32_t e = stream_peek(s, min(s.at + 4, s.n - 1));
    s.at += 1;
    s.stage = ring_add(s.stage, 1);
    set_load(s, e, ring_add(s.stage, 3), s.c);
    wait_dma_all_but_last_page();
    stream_reach(s);
  }
  rider_rest(a, w, s.lane);  // a short segment's
}

// The segment at stream offset k of group `group`'s share.
__device__ __forceinline__ VideoPartition32 part_of(const __attribute__((address_space(4))) AttnClass& c) {
  const auto& p = c.part;
  return VideoPartition32{p.pages, p.cost, p.len, p.groups, p.quot, p.rem, p.fits,
                          {p.by_pages.mul, p.by_pages.shift}, {p.by_stride.mul, p.by_stride.shift},
                          {p.by_groups.mul, p.by_groups.shift}, {p.by_len.mul, p.by_len.shift}};
}
struct VideoWork {
  VideoPartition32 part;
  int group, q_lo, q_hi;
};
__device__ __forceinline__ VideoSeg video_seg(const VideoWork& w, const VideoStream& s, int k) {
  const int x = s.lo + k;
  const int head = static_cast<int>(fast_div(x, s.div_pages)), h0 = head * s.n_pages;
  const int n = min(s.n - k, h0 + s.n_pages - x);
  const int seg = x == h0 ? 0 : w.group - static_cast<int>(part_group_of(w.part, h0));
  return VideoSeg{head, n, seg, w.q_lo, w.q_hi, x == h0 && n == s.n_pages};
}

// Ranges of a head (for the rider rows' partials).
__device__ __forceinline__ int head_ranges(const VideoWork& w, const VideoStream& s, int head) {
  const int h0 = head * s.n_pages;
  return static_cast<int>(part_group_of(w.part, h0 + s.n_pages - 1) - part_group_of(w.part, h0)) + 1;
}

template <int kQT, bool kPrepared>
__device__ __forceinline__ void video_wave(const AttnArgs& a, const VideoWork& w, VideoStream& s, int wave) {
  stream_start(a, s);
  while (s.at < s.n) video_segment<kQT, kPrepared>(a, video_seg(w, s, s.at), s, wave);
}

// The rider rows' pages for a wave with rows of its own, after its segments.
__device__ __forceinline__ void rider_segments(const AttnArgs& a, const VideoWork& w, const VideoStream& s) {
  for (int k = 0; k < s.n;) {
    const VideoSeg sg = video_seg(w, s, k);
    RiderWork r;
    rider_share(a, sg, head_ranges(w, s, sg.head), r);
    rider_rest(a, r, opaque(s.lane));
    k += sg.n;
  }
}

// Rows that see nothing: output 0.
__device__ __forceinline__ void video_empty(const AttnArgs& a, int head, int q_lo, int q_hi) {
  const int n = (q_hi - q_lo) * (kHeadDim / 8);
  for (int i = threadIdx.x; i < n; i += kVideoWaves * 64) {
    const int64_t q = q_lo + i / (kHeadDim / 8);
    *reinterpret_cast<u32x4*>(a.out + q * a.out_tok_stride + head * a.out_head_stride + 8 * (i % (kHeadDim / 8))) =
        (u32x4){0u, 0u, 0u, 0u};
  }
}

// kPrepared: the video queries come prepared (query mode 2).
template <bool kPrepared>
__device__ __forceinline__ void unit_attn(const AttnArgs& a) {
  // Work decode.  Each query class (the rows of one unit's queries, with the
  // pages its mask leaves visible) owns a block of workgroups: n_groups
  // groups of n_qtiles workgroups; group g takes a contiguous share of the
  // class's (head, page) units in head-major order (VideoPartition: even
  // shares of pages plus a cost per head started), one workgroup per query
  // tile, so the work fits a single round, and a share that crosses a head
  // boundary is processed as several segments.  Workgroups are dispatched
  // round-robin over the 8 XCDs; renumber so that consecutive work items
  // (the query tiles of a group, which read the same pages at the same time,
  // and neighbouring groups) run on one XCD and share its L2.  The divisions
  // are multiplications by host-made reciprocals: with the partition's own
  // integer divisions a workgroup spent 5 us before its first load.
  const int nblk = gridDim.x, bid = blockIdx.x;
  const int xcd = bid & 7, per = nblk >> 3, rem = nblk & 7;
  const int item = xcd * per + min(xcd, rem) + (bid >> 3);
  const const_class_table tab = class_table();
  int ci = 0;
  for (int k = 1; k < a.n_classes; ++k)
    if (item >= tab[k].wg0) ci = k;
  const int local = item - tab[ci].wg0;
  const int n_qtiles = tab[ci].n_qtiles;
  const int group = static_cast<int>(fast_div(local, FastDiv{tab[ci].by_qtiles.mul, tab[ci].by_qtiles.shift}));
  const int qt = local - group * n_qtiles;
  const int q0 = tab[ci].q0, q_hi = q0 + tab[ci].n_q;
  const int tile_rows = tab[ci].tile_rows, q_lo = q0 + qt * tile_rows;
  // rider rows follow the video rows (a single class then)
  const int row_end = min(q_lo + tile_rows, a.n_rq > 0 ? a.rq_row0 + a.n_rq : q_hi);
  const int wave_rows = video_wave_rows(tile_rows, row_end - q_lo);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));

  VideoWork w;
  w.group = group;
  w.q_lo = q_lo;
  w.q_hi = q_hi;
  VideoStream s;
  s.pages = page_list(a);
  s.num_heads = a.num_heads;
  s.n_pages = tab[ci].n_pages;
  s.page0 = tab[ci].page0;
  s.lane = lane;
  s.kpool = a.kpool;
  s.vpool = a.vpool;
  s.at = 0;
  s.stage = 0;
  s.valid = 0;
  if (s.n_pages == 0) {  // nothing visible: one group per head
    if (group < a.num_heads) video_empty(a, group, q_lo, min(q_lo + tile_rows, q_hi));
    return;
  }
  w.part = part_of(tab[ci]);
  s.div_pages = w.part.by_pages;
  s.lo = static_cast<int>(part_group_lo(w.part, group));
  s.n = static_cast<int>(part_group_lo(w.part, group + 1)) - s.lo;
  if (s.n == 0) return;
  // the list entries of the window are under way while the lane's offsets are
  // computed; stream_start waits for them, and the first segment's queries are
  // loaded behind the direct loads it issues
  stream_request(s);
  {
    // K block wave: row 4 wave + lane / 16 of key tile 0, position lane % 16
    const int m = 4 * wave + (lane >> 4);
    s.dma_k = 2 * k_tile_index(audio_key(0, m), 8 * ((lane & 15) ^ m));
    // V^T block wave: row d = 8 wave + lane / 8, position lane % 8
    const int d = 8 * wave + (lane >> 3);
    s.dma_v = 2 * v_tile_index(8 * ((lane & 7) ^ ((d >> 1) & 7)), d);
    const uint32_t lds = lds_offset(g_stages);
    s.lds0 = __builtin_amdgcn_readfirstlane(lds + 1024u * wave);
    const int g = lane >> 4, i16 = lane & 15;
    s.k_read = lds + 256u * i16 + 16u * (g ^ i16);
    s.v_read = lds + kStageV + 128u * i16 + 16u * (g ^ ((i16 >> 1) & 7));
  }
  const bool rx = a.rx_pages > 0 && qt == n_qtiles - 1 && wave == kVideoWaves - 1;
  if (q_lo + wave * wave_rows >= row_end) {
    stream_start(a, s);
    while (s.at < s.n) {
      const VideoSeg sg = video_seg(w, s, s.at);
      video_idle_segment(a, sg, s, rx ? head_ranges(w, s, sg.head) : 0);
    }
    wait_dma_all();
    return;
  }
  if (wave_rows == 64) video_wave<4, kPrepared>(a, w, s, wave);
  else if (wave_rows == 48) video_wave<3, kPrepared>(a, w, s, wave);
  else video_wave<2, kPrepared>(a, w, s, wave);
  if (rx) rider_segments(a, w, s);
}

#define WS_ONE_WAVE_PER_SIMD __launch_bounds__(kVideoWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1)))
__global__ WS_ONE_WAVE_PER_SIMD void unit_attn_kernel(const AttnArgs a) { unit_attn<true>(a); }
__global__ WS_ONE_WAVE_PER_SIMD void unit_attn_rows_kernel(const AttnArgs a) { unit_attn<false>(a); }

// ------------------------------------------------------------------------- //
// combine (audio key ranges): 16 threads per (head, query) row, 8 d each, 16
// rows per block.  A thread reads the row's log-sum-exps, then requests the
// 8 values of kMergeBatch ranges before using any (one memory round trip per
// batch) and folds them against the largest.  The batch sets the registers a
// thread holds: the audio call's own merge takes 16 ranges at once; inside
// the merge launch of a step, whose video rows need few registers, 3 (more
// would cap the occupancy of the video rows' blocks).
// ------------------------------------------------------------------------- //
template <int kMergeBatch>
__device__ __forceinline__ void combine_block(const CombineArgs& a, int bid) {
  const int lane = threadIdx.x & 15;
  const int row = bid * 16 + (threadIdx.x >> 4);
  if (row >= a.num_heads * a.n_q) return;
  const int head = row / a.n_q, q = row % a.n_q;
  int n_splits = a.n_splits;
  if (a.r_groups > 0) {  // the ranges the video kernel wrote for rider rows
    const VideoPartition part{a.num_heads, a.r_pages, a.seg_cost, a.r_groups};
    const int64_t h0 = static_cast<int64_t>(head) * a.r_pages;
    const int ranges = static_cast<int>(video_group_of(part, h0 + a.r_pages - 1) - video_group_of(part, h0) + 1);
    n_splits += ranges + min(ranges, a.r_extra);  // and those of the rows' own pages
  }
  const int d0 = 8 * lane;
  const int64_t split_stride = static_cast<int64_t>(a.num_heads) * a.n_q;
  // The largest log-sum-exp first: every range is then weighted the same way
  // whatever the batch, so the step's merge launch and the audio call's own
  // give the same bits.  (With all ranges in one batch it comes from that
  // batch's loads.)
  float mx = kNegInf;
  for (int sp0 = 0; n_splits > kMergeBatch && sp0 < n_splits; sp0 += 16) {
    float lb[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) lb[i] = sp0 + i < n_splits ? a.part_lse[(sp0 + i) * split_stride + row] : kNegInf;
#pragma unroll
    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, lb[i]);
  }
  float wsum = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int sp0 = 0; sp0 < n_splits; sp0 += kMergeBatch) {
    float lb[kMergeBatch];
    f32x4 o0[kMergeBatch], o1[kMergeBatch];
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const int sp = sp0 + i;
      const bool ok = sp < n_splits;
      const float* po = a.part_o + (sp * split_stride + row) * kHeadDim + d0;
      lb[i] = ok ? a.part_lse[sp * split_stride + row] : kNegInf;
      o0[i] = ok ? *reinterpret_cast<const f32x4*>(po) : (f32x4){0.f, 0.f, 0.f, 0.f};
      o1[i] = ok ? *reinterpret_cast<const f32x4*>(po + 4) : (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    if (n_splits <= kMergeBatch) {
#pragma unroll
      for (int i = 0; i < kMergeBatch; ++i) mx = fmaxf(mx, lb[i]);
    }
    if (mx == kNegInf) break;
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const float w = lb[i] == kNegInf ? 0.f : fast_exp2(lb[i] - mx);
      wsum += w;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc[k] += w * o0[i][k];
        acc[4 + k] += w * o1[i][k];
      }
    }
  }
  const float inv = mx != kNegInf ? 1.0f / wsum : 0.f;
  u32x4 w;
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = pack_bf16(acc[2 * k] * inv, acc[2 * k + 1] * inv);
  *reinterpret_cast<u32x4*>(a.out + q * a.out_tok_stride + head * a.out_head_stride + d0) = w;
}

__global__ __launch_bounds__(256) void combine_kernel(const CombineArgs a) { combine_block<16>(a, blockIdx.x); }

// ------------------------------------------------------------------------- //
// video_combine: merges the key ranges of the video schedule.  A head's
// range count follows from the groups' shares (VideoPartition; a head
// in one range was written in bf16 by the attention kernel: nothing to
// merge).  16 threads per (head, query) row, 8 d each (16-byte loads), 16
// rows per block; all of a row's (at most kMaxVideoSplits) partials are
// requested before any is used.
// ------------------------------------------------------------------------- //
__device__ __forceinline__ void video_combine_block(const CombineArgs& a, const_class_table tab, int bid) {
  const int lane = threadIdx.x & 15;
  const int row = bid * 16 + (threadIdx.x >> 4);
  if (row >= a.num_heads * a.n_q) return;
  const int head = row / a.n_q, q = row % a.n_q;
  // the row's query class: every table entry is read with uniform (scalar)
  // loads and the row's fields are selected per lane
  int32_t cls_pages = tab[0].n_pages, cls_groups = tab[0].n_groups;
  for (int k = 1; k < a.n_classes; ++k) {
    const bool in = q >= tab[k].q0;
    cls_pages = in ? tab[k].n_pages : cls_pages;
    cls_groups = in ? tab[k].n_groups : cls_groups;
  }
  const int64_t n_pages = cls_pages;
  if (n_pages == 0) return;
  const VideoPartition part{a.num_heads, n_pages, a.seg_cost, cls_groups};
  const int64_t h0 = static_cast<int64_t>(head) * n_pages;
  const int n_ranges = static_cast<int>(video_group_of(part, h0 + n_pages - 1) - video_group_of(part, h0) + 1);
  if (n_ranges < 2) return;
  const int d0 = 8 * lane;
  const int64_t split_stride = static_cast<int64_t>(a.num_heads) * a.n_q;
  const uint16_t* po = reinterpret_cast<const uint16_t*>(a.part_o);
  float l[kMaxVideoSplits];
  u32x4 w[kMaxVideoSplits];
#pragma unroll
  for (int sp = 0; sp < kMaxVideoSplits; ++sp) {
    if (sp < n_ranges) {
      l[sp] = a.part_lse[sp * split_stride + row];
      w[sp] = *reinterpret_cast<const u32x4*>(po + (sp * split_stride + row) * kHeadDim + d0);
    } else {
      l[sp] = kNegInf;
      w[sp] = (u32x4){0u, 0u, 0u, 0u};
    }
  }
  float mx = kNegInf;
#pragma unroll
  for (int sp = 0; sp < kMaxVideoSplits; ++sp) mx = fmaxf(mx, l[sp]);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (mx != kNegInf) {
    float wsum = 0.f;
#pragma unroll
    for (int sp = 0; sp < kMaxVideoSplits; ++sp) {
      if (l[sp] == kNegInf) continue;
      const float e = fast_exp2(l[sp] - mx);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += e * bf16_lo(w[sp][i]);
        acc[2 * i + 1] += e * bf16_hi(w[sp][i]);
      }
      wsum += e;
    }
    const float inv = 1.0f / wsum;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= inv;
  }
  u32x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = pack_bf16(acc[2 * i], acc[2 * i + 1]);
  *reinterpret_cast<u32x4*>(a.out + q * a.out_tok_stride + head * a.out_head_stride + d0) = o;
}

// The class table of the video CombineArgs, which is the first kernel
// argument of both merge kernels below, read in place.
__device__ __forceinline__ const_class_table combine_class_table() {
  const __attribute__((address_space(4))) char* seg =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  return (const_class_table)(seg + offsetof(CombineArgs, cls));
}

__global__ __launch_bounds__(256) void video_combine_kernel(const CombineArgs a) {
  video_combine_block(a, combine_class_table(), blockIdx.x);
}

// The merges of one step's video and audio calls in one launch: blocks below
// n_audio merge audio rows (they start first: their rows fold more ranges),
// the rest video rows.
__global__ __launch_bounds__(256) void step_combine_kernel(const CombineArgs v, const CombineArgs au,
                                                           int n_audio) {
  if (static_cast<int>(blockIdx.x) < n_audio)
    combine_block<3>(au, blockIdx.x);
  else
    video_combine_block(v, combine_class_table(), blockIdx.x - n_audio);
}

}  // namespace

// The no-allocation entry point's split-KV workspace.  Host code never
// passes this name to a kernel or a copy (in host code it is only a stand-in
// for the symbol): it uses the device address static_scratch() looks up.
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

hipError_t static_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// With start or stop events, a launch goes through hipExtLaunchKernelGGL,
// whose events take the dispatch's own start and end timestamps (the
// kernel's execution, without the queue's event processing around it).
hipError_t launch_kv_append(const AppendArgs& a, hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
  const int tiles = a.n_blocks * a.num_heads;
  const int grid = std::min(tiles, std::max(1, a.grid_blocks));
  if (start || stop)
    hipExtLaunchKernelGGL(kv_append_kernel, dim3(grid), dim3(256), 0, stream, start, stop, 0, a);
  else
    hipLaunchKernelGGL(kv_append_kernel, dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_unit_attention(const AttnArgs& a, hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(a.n_wg), block(kVideoWaves * 64);
  const auto kernel = a.mode == 2 ? unit_attn_kernel : unit_attn_rows_kernel;
  if (start || stop)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, start, stop, 0, a);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_audio_attention(const AttnArgs& a, hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(a.num_heads * a.n_qtiles * a.n_splits);
  if (start || stop)
    hipExtLaunchKernelGGL(audio_attn_kernel, grid, dim3(256), 0, stream, start, stop, 0, a);
  else
    hipLaunchKernelGGL(audio_attn_kernel, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_step_combine(const CombineArgs& v, const CombineArgs& au, hipStream_t stream) {
  const int n_video = v.n_groups > 0 ? (v.num_heads * v.n_q + 15) / 16 : 0;
  const int n_audio = au.num_heads > 0 ? (au.num_heads * au.n_q + 15) / 16 : 0;
  if (n_video + n_audio == 0) return hipSuccess;
  hipLaunchKernelGGL(step_combine_kernel, dim3(n_video + n_audio), dim3(256), 0, stream, v, au, n_audio);
  return hipGetLastError();
}

hipError_t launch_combine(const CombineArgs& a, hipStream_t stream) {
  const int rows = a.num_heads * a.n_q;
  if (a.n_groups > 0)
    hipLaunchKernelGGL(video_combine_kernel, dim3((rows + 15) / 16), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(combine_kernel, dim3((rows + 15) / 16), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ws
