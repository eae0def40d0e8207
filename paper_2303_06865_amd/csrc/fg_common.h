// Internal helpers shared by the HIP sources of libfg (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fg.h"

namespace fg {

typedef _Float16 half_t;
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u2_t __attribute__((ext_vector_type(2)));

constexpr int kGroup = 64;           // elements per quantization group (Section 5)
constexpr int kWave = 64;            // CDNA wavefront width

// ---- error plumbing ---------------------------------------------------------------------
void set_device_error(hipError_t e, const char* what);

#define FG_HIP(expr)                                   \
  do {                                                 \
    hipError_t _e = (expr);                            \
    if (_e != hipSuccess) {                            \
      ::fg::set_device_error(_e, #expr);               \
      return FG_ERR_DEVICE;                            \
    }                                                  \
  } while (0)

// Call after a kernel launch: picks up launch-configuration errors.
#define FG_LAUNCH_CHECK() FG_HIP(hipGetLastError())

// ---- per-kernel-class event timing --------------------------------------------------------
bool profile_enabled();
void profile_mark(int kclass, hipStream_t stream, bool begin);

struct ProfScope {
  int k;
  hipStream_t s;
  bool on;
  ProfScope(int kclass, hipStream_t stream) : k(kclass), s(stream), on(profile_enabled()) {
    if (on) profile_mark(k, s, true);
  }
  ~ProfScope() {
    if (on) profile_mark(k, s, false);
  }
};

static inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

// ---- entry points of the individual kernel files (host side, already validated) ----------
struct LinearArgs {
  const void* w_data;      // codes or FP16
  const void* w_meta;      // {min,scale} pairs or NULL
  int dtype;
  int64_t n, k;            // W is [n, k]
  const half_t* x;         // [m, k], row stride ldx
  int64_t ldx;
  int64_t m;
  const half_t* bias;      // [n] or NULL
  const half_t* residual;  // [m, n] row stride ldr, or NULL
  int64_t ldr;
  int relu;
  half_t* out_f16;         // [m, n] row stride ldo (NULL when out_f32 is used)
  float* out_f32;          // [m, n] row stride ldo, no FP16 rounding (LM head logits)
  int64_t ldo;
};
size_t linear_workspace_bytes(int dtype, int64_t n, int64_t k, int64_t m);
int linear_launch(const LinearArgs& a, void* ws, size_t ws_bytes, hipStream_t stream);

// a few rows, any weight format (csrc/fg_gemm_fewrows.hip); needs no workspace
bool gemm_fewrows_takes(int dtype, int64_t n, int64_t k, int64_t m);
int gemm_fewrows_launch(const LinearArgs& a, hipStream_t stream);
// ... of LayerNorm(a.x), with FP16 results and no residual (csrc/fg_gemm_fewrows_ln.hip; ct: column tiles per workgroup)
bool gemm_ln_fewrows_takes(int dtype, int64_t n, int64_t k, int64_t m);
int gemm_ln_fewrows_launch(const LinearArgs& a, const half_t* gamma, const half_t* beta, float eps, hipStream_t stream);
bool gemm_fewrows_ln_takes(int dtype, int64_t n, int64_t k, int64_t m, int ct);
int gemm_fewrows_ln_launch(const LinearArgs& a, const half_t* gamma, const half_t* beta, float eps, int ct, hipStream_t stream);
// small-M (decode) and large-M (prefill) kernels behind linear_launch
size_t gemm_small_m_workspace(int dtype, int64_t n, int64_t k, int64_t m);
int gemm_small_m_launch(const LinearArgs& a, void* ws, size_t ws_bytes, hipStream_t stream);
int gemm_large_m_launch(const LinearArgs& a, hipStream_t stream);
// tiled 4-bit weights: weight-streaming kernel for few rows, and the repacking kernel
// row-major FP16 weights, up to 128 rows (csrc/fg_gemm_f16w.hip); pick_cols returns 0 for shapes it does not take
int gemm_f16w_pick_cols(int64_t n, int64_t k, int64_t m);
int gemm_f16w_forced(int64_t n);   // column tiles fixed by the environment, or 0
size_t gemm_f16w_workspace(int64_t n, int64_t k, int64_t m);
int gemm_f16w_launch(const LinearArgs& a, void* ws, size_t ws_bytes, hipStream_t stream);
// row-major FP16 weights, some hundred rows (csrc/fg_gemm_f16_tiles.hip); any workspace will do
struct F16TilePick {
  int mt, nt, splits;   // tiles of 32 mt x 32 nt, ranges of the contraction
  int64_t items;        // workgroups
  float us;             // expected time
};
F16TilePick gemm_f16_tiles_pick(int64_t n, int64_t k, int64_t m, size_t ws_bytes);
bool gemm_f16_tiles_takes(int dtype, int64_t n, int64_t k, int64_t m, bool residual);
int gemm_f16_tiles_launch(const LinearArgs& a, void* ws, size_t ws_bytes, hipStream_t stream);
size_t gemm_stream_workspace(int64_t n, int64_t k, int64_t m);
// FP16 weights: are the tiles the largest of their kind (160, 192 or 256 rows) and their number one that keeps all workgroups
// busy to the end; the expected time, from 321 rows up
bool gemm_stream_f16_whole_rounds(int64_t n, int64_t k, int64_t m);
float gemm_stream_f16_us(int64_t n, int64_t k, int64_t m);
int gemm_stream_launch(const LinearArgs& a, void* ws, size_t ws_bytes, hipStream_t stream);
int pack_weights_launch(const void* codes, const void* meta, bool meta_f16, int64_t n, int64_t k, void* codes_out, void* meta_out,
                        hipStream_t stream);

int layernorm_launch(const half_t* x, int64_t ldx, const half_t* g, const half_t* b, int64_t rows,
                     int64_t cols, float eps, half_t* out, int64_t ldo, hipStream_t stream);
int embed_launch(const half_t* emb, const half_t* pos, const int32_t* ids, int64_t ids_stride, int64_t rows,
                 int32_t s_len, int32_t pos0, int32_t h1, int32_t vocab, half_t* out, hipStream_t stream);
int embed_ragged_launch(const half_t* emb, const half_t* pos, const int32_t* ids, const int32_t* id_index,
                        const int32_t* positions, int64_t rows, int32_t h1, int32_t vocab, int32_t max_pos,
                        half_t* out, hipStream_t stream);
int argmax_launch(const float* logits, int64_t rows, int64_t cols, int32_t* out, int64_t out_stride,
                  hipStream_t stream, const int32_t* out_index = nullptr);

int kv_append_launch(const fg_model_cfg& cfg, const half_t* k, const half_t* v, int64_t row_stride,
                     int32_t b, int32_t s, const fg_kv_cache& kv, int32_t batch_offset, int32_t pos0,
                     hipStream_t stream);
bool decode_attention_appends(const fg_model_cfg& cfg, const fg_kv_cache& kv, int32_t b);
int decode_attention_launch(const fg_model_cfg& cfg, const half_t* q, int64_t q_stride, int32_t b,
                            int32_t rows, const fg_kv_cache& kv, int32_t batch_offset, half_t* out,
                            hipStream_t stream, const half_t* k_new = nullptr, const half_t* v_new = nullptr);
int prefill_attention_launch(const fg_model_cfg& cfg, const half_t* qkv, int32_t b, int32_t s,
                             half_t* out, hipStream_t stream);
// paged cache (sequences at different steps): s rows per sequence from position pos[i] (nullptr: 0);
// attention over pos[i] + rows_bias rows
int kv_append_paged_launch(const fg_model_cfg& cfg, const half_t* k, const half_t* v, int64_t row_stride,
                           int32_t b, int32_t s, const fg_kv_pages& pages, const fg_ragged& seqs, bool use_pos,
                           hipStream_t stream);
int decode_attention_paged_launch(const fg_model_cfg& cfg, const half_t* q, int64_t q_stride, int32_t b,
                                  const fg_kv_pages& pages, const fg_ragged& seqs, int32_t rows_bias, half_t* out,
                                  hipStream_t stream);
int check_pages(const fg_model_cfg* cfg, const fg_kv_pages* pages, const fg_ragged* seqs);
// Top-K sparse decode attention (4-bit caches): contiguous cache, and paged cache with a length per row
int decode_attention_topk_launch(const fg_model_cfg& cfg, const half_t* q, int64_t q_stride, int32_t b, int32_t rows,
                                 int32_t topk, const fg_kv_cache& kv, int32_t batch_offset, half_t* out,
                                 int32_t* sel_out, hipStream_t stream);
int decode_attention_topk_paged_launch(const fg_model_cfg& cfg, const half_t* q, int64_t q_stride, int32_t b,
                                       int32_t topk, const fg_kv_pages& pages, const fg_ragged& seqs,
                                       int32_t rows_bias, half_t* out, int32_t* sel_out, hipStream_t stream);

// validation helpers (host only)
int check_cfg(const fg_model_cfg* cfg);
int check_mat(const fg_mat* w, bool for_pack = false);
int check_kv(const fg_model_cfg* cfg, const fg_kv_cache* kv);

// ---- device helpers -------------------------------------------------------------------------
#if defined(__HIPCC__)

// Reductions over lanes, without LDS: inside 16 lanes the partner's value is a DPP operand, across the four rows
// of 16 it comes from v_permlane16_swap / v_permlane32_swap.  (ds_bpermute, which __shfl_xor becomes, is an LDS
// round trip per step, and six of them in a chain are most of what a short attention stream or a normalised row
// waits for.)
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// quad_perm 1032 and 2301; lanes reversed inside 8 and inside 16: once the quads (the eights) are uniform, the
// mirror brings the other quad's (the other eight's) value
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
// lanes of 16 rotated: once the eights (the quads of the eights) repeat, the other eight's (quad's) value at one's own place
constexpr int kDppRor8 = 0x128, kDppRor4 = 0x124;

template <class Op>
__device__ __forceinline__ float row16_reduce(float v, Op op) {   // over each 16 lanes, result in all of them
  v = op(v, dpp_f32<kDppXor1>(v));
  v = op(v, dpp_f32<kDppXor2>(v));
  v = op(v, dpp_f32<kDppHalfMirror>(v));
  return op(v, dpp_f32<kDppMirror>(v));
}
template <class Op>
__device__ __forceinline__ float xor16_reduce(float v, Op op) {
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (uint32_t)s[0]), __builtin_bit_cast(float, (uint32_t)s[1]));
}
template <class Op>
__device__ __forceinline__ float xor32_reduce(float v, Op op) {
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto s = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (uint32_t)s[0]), __builtin_bit_cast(float, (uint32_t)s[1]));
}
struct OpMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
struct OpAdd {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
__device__ __forceinline__ float wave_max(float v) {
  return xor32_reduce(xor16_reduce(row16_reduce(v, OpMax()), OpMax()), OpMax());
}
// The halves first, neighbouring lanes last.  The order is part of what LayerNorm returns: another one moves its mean
// by a last bit, some of its FP16 results by an ulp and, behind the QKV projection, a few 4-bit codes of the cache by a
// step, which in 12288-wide layers showed as single outputs off by 0.05 of their root mean square.
__device__ __forceinline__ float wave_sum(float v) {
  v = xor16_reduce(xor32_reduce(v, OpAdd()), OpAdd());
  v += dpp_f32<kDppRor8>(v);
  v += dpp_f32<kDppRor4>(v);
  v += dpp_f32<kDppXor2>(v);
  return v + dpp_f32<kDppXor1>(v);
}

// The places of LayerNorm where a product could be rounded before it is added, or a result once or twice on its way to FP16:
// written out, because what one kernel leaves to the compiler another one, that normalizes the same rows, may get otherwise.
// q plus the squared distances of a piece of eight; of the first piece's first two squares the second one is rounded.
__device__ __forceinline__ float ln_add_squares(const h8_t v, float mean, float q, bool first) {
  float d[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) d[i] = (float)v[i] - mean;
  q = first ? __builtin_fmaf(d[0], d[0], d[1] * d[1]) : __builtin_fmaf(d[1], d[1], __builtin_fmaf(d[0], d[0], q));
#pragma unroll
  for (int i = 2; i < 8; ++i) q = __builtin_fmaf(d[i], d[i], q);
  return q;
}
__device__ __forceinline__ h8_t ln_normalize(const h8_t v, float mean, float rstd, const h8_t gamma, const h8_t beta) {
  h8_t o;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float y = __builtin_fmaf(((float)v[i] - mean) * rstd, (float)gamma[i], (float)beta[i]);
    __asm__("" : "+v"(y));   // a binary32 number: v_fma_mixlo_f16 would round only once
    o[i] = (half_t)y;
  }
  return o;
}

// Between LDS writes of a wave's lanes and LDS reads of the same wave's other lanes.  No instruction comes of it (a wave's
// LDS accesses complete in order), but the compiler, which thinks lane by lane, may not exchange them.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Unpack one 32-bit word of eight 4-bit codes c0..c7 (c0 in the lowest nibble) into four FP16
// pairs WITHOUT leaving the register file.  The pairs come out in the order
//   p[0] = (c0, c4) + 1024,  p[1] = (c1, c5) + 64,  p[2] = (c2, c6) + 1024,  p[3] = (c3, c7) + 64
// because OR-ing a nibble into the mantissa of 1024.0 (0x6400, ulp 1) or, four bits higher, of
// 64.0 (0x5400, ulp 1/16) yields those integers exactly.
__device__ __forceinline__ void unpack8_biased(uint32_t x, uint32_t p[4]) {
  const uint32_t y = x >> 8;
  p[0] = (x & 0x000F000Fu) | 0x64006400u;
  p[1] = (x & 0x00F000F0u) | 0x54005400u;
  p[2] = (y & 0x000F000Fu) | 0x64006400u;
  p[3] = (y & 0x00F000F0u) | 0x54005400u;
}

// Same word -> eight FP16 codes (exact small integers), pair order (c0,c4),(c1,c5),(c2,c6),(c3,c7).
__device__ __forceinline__ void unpack8_codes(uint32_t x, h2_t p[4]) {
  uint32_t r[4];
  unpack8_biased(x, r);
  const h2_t k1024 = {(half_t)1024.0f, (half_t)1024.0f};
  const h2_t k64 = {(half_t)64.0f, (half_t)64.0f};
  p[0] = __builtin_bit_cast(h2_t, r[0]) - k1024;
  p[1] = __builtin_bit_cast(h2_t, r[1]) - k64;
  p[2] = __builtin_bit_cast(h2_t, r[2]) - k1024;
  p[3] = __builtin_bit_cast(h2_t, r[3]) - k64;
}

// Exact dequantization of one word of eight codes to FP16: w_i = RN16(mn + c_i * scale), one rounding
// from the real number (Section 5: "converted back to FP16 before computation").
// A nibble masked in place is the FP16 subnormal c * 2^-24 (low nibble of a half) or c * 2^-20 (next
// nibble); gfx950 mixed-precision FMAs take FP16 subnormals at full rate, multiply by the pre-scaled
// s24 = scale * 2^24 / s20 = scale * 2^20 (exact scalings), add mn and round once into an FP16 half
// of the destination (v_fma_mixlo_f16 / v_fma_mixhi_f16).  Thirteen VALU instructions per eight
// weights.  Output in natural order: p[0] = (w0,w1), p[1] = (w2,w3), p[2] = (w4,w5), p[3] = (w6,w7).
__device__ __forceinline__ void dequant8_exact(uint32_t x, float s24, float s20, float mn, uint32_t p[4]) {
  const uint32_t y = x >> 8;
  const uint32_t a = x & 0x000F000Fu;   // halves: c0 * 2^-24 , c4 * 2^-24
  const uint32_t b = x & 0x00F000F0u;   //         c1 * 2^-20 , c5 * 2^-20
  const uint32_t c = y & 0x000F000Fu;   //         c2 * 2^-24 , c6 * 2^-24
  const uint32_t d = y & 0x00F000F0u;   //         c3 * 2^-20 , c7 * 2^-20
  const h2_t ha = __builtin_bit_cast(h2_t, a), hb = __builtin_bit_cast(h2_t, b);
  const h2_t hc = __builtin_bit_cast(h2_t, c), hd = __builtin_bit_cast(h2_t, d);
  const h2_t q0 = {(half_t)__builtin_fmaf((float)ha.x, s24, mn), (half_t)__builtin_fmaf((float)hb.x, s20, mn)};
  const h2_t q1 = {(half_t)__builtin_fmaf((float)hc.x, s24, mn), (half_t)__builtin_fmaf((float)hd.x, s20, mn)};
  const h2_t q2 = {(half_t)__builtin_fmaf((float)ha.y, s24, mn), (half_t)__builtin_fmaf((float)hb.y, s20, mn)};
  const h2_t q3 = {(half_t)__builtin_fmaf((float)hc.y, s24, mn), (half_t)__builtin_fmaf((float)hd.y, s20, mn)};
  const uint32_t r0 = __builtin_bit_cast(uint32_t, q0), r1 = __builtin_bit_cast(uint32_t, q1);
  const uint32_t r2 = __builtin_bit_cast(uint32_t, q2), r3 = __builtin_bit_cast(uint32_t, q3);
  p[0] = r0;
  p[1] = r1;
  p[2] = r2;
  p[3] = r3;
}

// The same numbers from a {min, scale} pair of FP16 numbers: codes placed at bits 6..9 of each half are the FP16 subnormals
// c * 2^-18, scale * 2^18 is exact, and v_pk_fma_f16 rounds c * scale + min once, two weights at a time.  Sixteen VALU
// instructions per eight weights, of 56 cycles together where the thirteen of dequant8_exact take 85 (v_fma_mixlo_f16 and
// v_fma_mixhi_f16: 9 each).  For scales below 0.25, else scale * 2^18 is no finite FP16 number: dequant8_pk_takes().
// (gemm_decode16h_kernel uses it; on the other kernels that read such pairs it has not been tried.)
struct PkPair {
  h2_t s18, mn;
};
__device__ __forceinline__ bool dequant8_pk_takes(uint32_t pair) { return (pair & 0x7fff0000u) < 0x34000000u; }
__device__ __forceinline__ PkPair dequant8_pk_pair(uint32_t pair) {
  const h2_t s = __builtin_bit_cast(h2_t, __builtin_amdgcn_perm(pair, pair, 0x03020302u));
  const h2_t k = {(half_t)512.0f, (half_t)512.0f};
  return {s * k * k, __builtin_bit_cast(h2_t, __builtin_amdgcn_perm(pair, pair, 0x01000100u))};
}
__device__ __forceinline__ void dequant8_pk(uint32_t x, const PkPair& q, uint32_t p[4]) {
  uint32_t d[4] = {(x << 6) & 0x03C003C0u, (x << 2) & 0x03C003C0u, (x >> 2) & 0x03C003C0u, (x >> 6) & 0x03C003C0u};
#pragma unroll
  for (int i = 0; i < 4; ++i)   // halves: weights i and i + 4
    d[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(h2_t, d[i]), q.s18, q.mn));
  p[0] = __builtin_amdgcn_perm(d[1], d[0], 0x05040100u);
  p[1] = __builtin_amdgcn_perm(d[3], d[2], 0x05040100u);
  p[2] = __builtin_amdgcn_perm(d[1], d[0], 0x07060302u);
  p[3] = __builtin_amdgcn_perm(d[3], d[2], 0x07060302u);
}

// Reorder eight consecutive FP16 values h0..h7 (four words) into the pair order produced by
// unpack8_*: (h0,h4),(h1,h5),(h2,h6),(h3,h7), so that a contraction against unpacked codes lines up.
__device__ __forceinline__ u4_t permute8_like_codes(u4_t d) {
  u4_t o;
  o.x = __builtin_amdgcn_perm(d.z, d.x, 0x05040100u);  // (h0, h4)
  o.y = __builtin_amdgcn_perm(d.z, d.x, 0x07060302u);  // (h1, h5)
  o.z = __builtin_amdgcn_perm(d.w, d.y, 0x05040100u);  // (h2, h6)
  o.w = __builtin_amdgcn_perm(d.w, d.y, 0x07060302u);  // (h3, h7)
  return o;
}

#endif  // __HIPCC__

}  // namespace fg
