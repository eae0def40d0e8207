// Row-wise kernels around the projections: LayerNorm (OPT pre-LN placement), token + position
// embedding, and the greedy argmax over logits.  All are HBM/L2-bound streaming kernels.
#include <type_traits>

#include "fg_common.h"

namespace fg {

__device__ __forceinline__ float block_sum_256(float v, float* red) {   // red: four floats, used once per launch
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// One 256-thread block per row.  Mean first, then the centred second moment (both in binary32
// over FP16 inputs), then the normalised row; the re-reads hit L2.
__global__ __launch_bounds__(256) void layernorm_kernel(const half_t* __restrict__ x, int64_t ldx,
                                                        const half_t* __restrict__ gamma,
                                                        const half_t* __restrict__ beta, int cols,
                                                        float eps, half_t* __restrict__ out, int64_t ldo) {
  __shared__ float red[2][4];
  const half_t* xr = x + (int64_t)blockIdx.x * ldx;
  half_t* orow = out + (int64_t)blockIdx.x * ldo;
  const int nchunk = cols >> 3;
  float s = 0.f;
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    const h8_t v = *reinterpret_cast<const h8_t*>(xr + c * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) s += (float)v[i];
  }
  const float mean = block_sum_256(s, red[0]) / (float)cols;
  float q = 0.f;
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    const h8_t v = *reinterpret_cast<const h8_t*>(xr + c * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float d = (float)v[i] - mean;
      q = __builtin_fmaf(d, d, q);
    }
  }
  const float var = block_sum_256(q, red[1]) / (float)cols;
  const float rstd = 1.0f / sqrtf(var + eps);
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    const h8_t v = *reinterpret_cast<const h8_t*>(xr + c * 8);
    const h8_t g = *reinterpret_cast<const h8_t*>(gamma + c * 8);
    const h8_t b = *reinterpret_cast<const h8_t*>(beta + c * 8);
    *reinterpret_cast<h8_t*>(orow + c * 8) = ln_normalize(v, mean, rstd, g, b);
  }
}

// The same arithmetic in the same order for rows of up to 256 * 8 * NC elements, with the row held in
// registers between the three phases (one read of x instead of three).
// AHEAD, for few rows: one workgroup per row leaves CUs idle and the time is a chain of latencies (row in, two sums over
// the workgroup, gamma and beta in, row out), so gamma and beta are on their way before the sums and a sum is one barrier.
// (More waves per row were faster still, but cannot add in this order: see wave_sum.)
template <int NC, bool AHEAD>
__global__ __launch_bounds__(256) void layernorm_reg_kernel(const half_t* __restrict__ x, int64_t ldx,
                                                            const half_t* __restrict__ gamma,
                                                            const half_t* __restrict__ beta, int cols,
                                                            float eps, half_t* __restrict__ out, int64_t ldo) {
  __shared__ float red[2][4];
  const half_t* xr = x + (int64_t)blockIdx.x * ldx;
  half_t* orow = out + (int64_t)blockIdx.x * ldo;
  const int nchunk = cols >> 3;
  h8_t v[NC], g[NC], b[NC];
  auto load_gb = [&](int j) {
    const int c = threadIdx.x + 256 * j;
    g[j] = *reinterpret_cast<const h8_t*>(gamma + c * 8);
    b[j] = *reinterpret_cast<const h8_t*>(beta + c * 8);
  };
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int c = threadIdx.x + 256 * j;
    if (c < nchunk) v[j] = *reinterpret_cast<const h8_t*>(xr + c * 8);
  }
  if (AHEAD) {
#pragma unroll
    for (int j = 0; j < NC; ++j)
      if (threadIdx.x + 256 * j < nchunk) load_gb(j);
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < NC; ++j)
    if (threadIdx.x + 256 * j < nchunk) {
#pragma unroll
      for (int i = 0; i < 8; ++i) s += (float)v[j][i];
    }
  const float mean = block_sum_256(s, red[0]) / (float)cols;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NC; ++j)
    if (threadIdx.x + 256 * j < nchunk) q = ln_add_squares(v[j], mean, q, j == 0);
  const float var = block_sum_256(q, red[1]) / (float)cols;
  const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int c = threadIdx.x + 256 * j;
    if (c < nchunk) {
      if (!AHEAD) load_gb(j);
      *reinterpret_cast<h8_t*>(orow + c * 8) = ln_normalize(v[j], mean, rstd, g[j], b[j]);
    }
  }
}

// Where the line lies: back to back, later / ahead, us: 4 x 4096 2.62 / 2.54, 37 x 7168 3.50 / 3.22, 144 x 12288 4.51 / 4.23,
// 256 x 12288 4.88 / 4.57, 333 x 7168 4.10 / 3.98, 512 x 12288 6.22 / 5.95; 1000 x 4096 4.36 / 4.42, 1000 x 12288 9.77 / 10.19.
constexpr int64_t kFewLnRows = 512;
int layernorm_launch(const half_t* x, int64_t ldx, const half_t* g, const half_t* b, int64_t rows,
                     int64_t cols, float eps, half_t* out, int64_t ldo, hipStream_t stream) {
  if (rows == 0) return FG_OK;
  ProfScope prof(FG_K_LAYERNORM, stream);
  const dim3 grid((unsigned)rows), block(256);
  const bool few = rows <= kFewLnRows;
#define FG_LN(NC_)                                                                                                      \
  do {                                                                                                                  \
    if (few)                                                                                                            \
      hipLaunchKernelGGL((layernorm_reg_kernel<NC_, true>), grid, block, 0, stream, x, ldx, g, b, (int)cols, eps, out, ldo);  \
    else                                                                                                                \
      hipLaunchKernelGGL((layernorm_reg_kernel<NC_, false>), grid, block, 0, stream, x, ldx, g, b, (int)cols, eps, out, ldo); \
  } while (0)
  if (cols <= 256 * 8 * 2)
    FG_LN(2);
  else if (cols <= 256 * 8 * 4)
    FG_LN(4);
  else if (cols <= 256 * 8 * 8)
    FG_LN(8);
  else
    hipLaunchKernelGGL(layernorm_kernel, grid, block, 0, stream, x, ldx, g, b, (int)cols, eps, out, ldo);
#undef FG_LN
  FG_LAUNCH_CHECK();
  return FG_OK;
}

// x0[row] = E[ids[row]] + P[pos0 + row % s_len]; one 16-byte chunk per thread.
__global__ __launch_bounds__(256) void embed_kernel(const half_t* __restrict__ emb,
                                                    const half_t* __restrict__ pos,
                                                    const int32_t* __restrict__ ids, int64_t ids_stride,
                                                    int64_t rows, int s_len, int pos0, int h1, int vocab,
                                                    half_t* __restrict__ out) {
  const int cpr = h1 >> 3;
  const int64_t n = rows * cpr;
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; c < n; c += stride) {
    const int64_t row = c / cpr;
    const int ci = (int)(c - row * cpr);
    int id = ids[row * ids_stride];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);  // never read outside the table
    const int p = pos0 + (int)(row % s_len);
    const h8_t e = *reinterpret_cast<const h8_t*>(emb + (int64_t)id * h1 + ci * 8);
    const h8_t q = *reinterpret_cast<const h8_t*>(pos + (int64_t)p * h1 + ci * 8);
    h8_t o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (half_t)((float)e[i] + (float)q[i]);
    *reinterpret_cast<h8_t*>(out + row * h1 + ci * 8) = o;
  }
}

// The same with a position per row (rows of sequences that are at different steps); row r takes
// its token from ids[id_index[r]] (id_index == nullptr: ids[r]).
__global__ __launch_bounds__(256) void embed_ragged_kernel(const half_t* __restrict__ emb,
                                                           const half_t* __restrict__ pos,
                                                           const int32_t* __restrict__ ids,
                                                           const int32_t* __restrict__ id_index,
                                                           const int32_t* __restrict__ positions, int64_t rows,
                                                           int h1, int vocab, int max_pos,
                                                           half_t* __restrict__ out) {
  const int cpr = h1 >> 3;
  const int64_t n = rows * cpr;
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; c < n; c += stride) {
    const int64_t row = c / cpr;
    const int ci = (int)(c - row * cpr);
    int id = ids[id_index ? (int64_t)id_index[row] : row];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);   // never read outside the tables
    int p = positions[row];
    p = p < 0 ? 0 : (p >= max_pos ? max_pos - 1 : p);
    const h8_t e = *reinterpret_cast<const h8_t*>(emb + (int64_t)id * h1 + ci * 8);
    const h8_t q = *reinterpret_cast<const h8_t*>(pos + (int64_t)p * h1 + ci * 8);
    h8_t o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (half_t)((float)e[i] + (float)q[i]);
    *reinterpret_cast<h8_t*>(out + row * h1 + ci * 8) = o;
  }
}

// Greedy token: argmax over a row of binary32 logits, lowest index on ties.
// Row r's result goes to out[r * out_stride], or to out[out_index[r]] when out_index is given.
// One workgroup of T threads per row, kLoads pieces of it in flight per thread (a piece is 16 bytes; VEC == false, for
// rows that do not start on 16-byte boundaries: one element).  With few rows the time is that of one CU taking in a row,
// so it has sixteen waves, and as many loads as the row is long; what is loaded beyond the row's end is lost, and many
// rows pay for it.  LM head (64 wide) and argmax together, us, threads x loads 256 x 1 / 1024 x 1 / 1024 x 4 / 1024 x 16:
// 4 rows of 1000 logits 8.7 / 8.9 / 9.2 / 10.9, 2000 rows 39 / 43 / 45 / 67; 4 rows of 8192 12.0 / 10.0 / 10.4 / 13.7,
// 2000 rows 39 / 41 / 43 / 78; 4 rows of 50272 34 / 18.9 / 16.8 / 18.1, 128 rows 69 / 54 / 52 / 53, 2000 rows 211 / 221 /
// 220 / 221; 300 rows of 256000 305 / 209 / 212 / 203, 512 rows 325 / 274 / 279 / 267.  (256 threads with one 4-byte load
// each: 59 us for the argmax alone of 4 rows of 50272.)
template <bool VEC, int T, int kLoads>
__global__ __launch_bounds__(T) void argmax_kernel(const float* __restrict__ logits, int64_t cols,
                                                   int32_t* __restrict__ out, int64_t out_stride,
                                                   const int32_t* __restrict__ out_index) {
  constexpr int NW = T / 64, kW = VEC ? 4 : 1;
  __shared__ float bv[NW];
  __shared__ int bi[NW];
  const float* r = logits + (int64_t)blockIdx.x * cols;
  float best = -INFINITY;
  int idx = 0x7fffffff;
  const uint32_t n = (uint32_t)(cols / kW);   // (VEC is only taken where cols is a multiple of 4)
  for (uint32_t c = threadIdx.x; c < n; c += kLoads * T) {
    float v[kLoads][kW];
    uint32_t at[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      at[j] = c + j * T;
      at[j] = (at[j] < n ? at[j] : n - 1) * kW;   // past the end: the last piece again, which changes nothing
      if constexpr (VEC)
        *reinterpret_cast<float4*>(v[j]) = *reinterpret_cast<const float4*>(r + at[j]);
      else
        v[j][0] = r[at[j]];
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j)
#pragma unroll
      for (int e = 0; e < kW; ++e)
        if (v[j][e] > best || (v[j][e] == best && (int)at[j] + e < idx)) {
          best = v[j][e];
          idx = (int)at[j] + e;
        }
  }
  auto merge = [&](float ov, int oi) {
    if (ov > best || (ov == best && oi < idx)) {
      best = ov;
      idx = oi;
    }
  };
  auto merge_dpp = [&](auto CTRL_) {
    constexpr int ctrl = decltype(CTRL_)::value;
    merge(dpp_f32<ctrl>(best), __builtin_amdgcn_update_dpp(0, idx, ctrl, 0xF, 0xF, true));
  };
  auto merge_row16 = [&]() {
    merge_dpp(std::integral_constant<int, kDppXor1>{});
    merge_dpp(std::integral_constant<int, kDppXor2>{});
    merge_dpp(std::integral_constant<int, kDppHalfMirror>{});
    merge_dpp(std::integral_constant<int, kDppMirror>{});
  };
  merge_row16();
  merge(__shfl_xor(best, 16, 64), __shfl_xor(idx, 16, 64));
  merge(__shfl_xor(best, 32, 64), __shfl_xor(idx, 32, 64));
  if ((threadIdx.x & 63) == 0) {
    bv[threadIdx.x >> 6] = best;
    bi[threadIdx.x >> 6] = idx;
  }
  __syncthreads();
  static_assert(NW <= 16 && 16 % NW == 0, "one DPP row merges the waves");
  if (threadIdx.x < 64) {
    best = bv[threadIdx.x & (NW - 1)];
    idx = bi[threadIdx.x & (NW - 1)];
    merge_row16();
    if (threadIdx.x == 0) {
      const int64_t dst = out_index ? (int64_t)out_index[blockIdx.x] : (int64_t)blockIdx.x * out_stride;
      out[dst] = idx == 0x7fffffff ? 0 : idx;
    }
  }
}

int argmax_launch(const float* logits, int64_t rows, int64_t cols, int32_t* out, int64_t out_stride,
                  hipStream_t stream, const int32_t* out_index) {
  if (rows == 0) return FG_OK;
  ProfScope prof(FG_K_ARGMAX, stream);
  const bool vec = cols % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15u) == 0;
#define FG_ARGMAX(T_, LOADS_)                                                                                            \
  do {                                                                                                                   \
    if (vec)                                                                                                             \
      hipLaunchKernelGGL((argmax_kernel<true, T_, LOADS_>), dim3((unsigned)rows), dim3(T_), 0, stream, logits, cols, out,  \
                         out_stride, out_index);                                                                         \
    else                                                                                                                 \
      hipLaunchKernelGGL((argmax_kernel<false, T_, LOADS_>), dim3((unsigned)rows), dim3(T_), 0, stream, logits, cols, out, \
                         out_stride, out_index);                                                                         \
  } while (0)
  // pieces of a row: 16 bytes, or one element
  const int64_t pieces = vec ? cols / 4 : cols;
  if (pieces <= 256)
    FG_ARGMAX(256, 1);
  else if (pieces <= 2048)
    FG_ARGMAX(1024, 1);
  else if (pieces <= 16384)
    FG_ARGMAX(1024, 4);
  else
    FG_ARGMAX(1024, 16);
#undef FG_ARGMAX
  FG_LAUNCH_CHECK();
  return FG_OK;
}

int embed_launch(const half_t* emb, const half_t* pos, const int32_t* ids, int64_t ids_stride, int64_t rows,
                 int32_t s_len, int32_t pos0, int32_t h1, int32_t vocab, half_t* out, hipStream_t stream) {
  if (rows == 0) return FG_OK;
  const int64_t chunks = rows * (h1 / 8);
  int64_t blocks = ceil_div(chunks, 256);
  if (blocks > 256 * 32) blocks = 256 * 32;
  ProfScope prof(FG_K_EMBED, stream);
  hipLaunchKernelGGL(embed_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, emb, pos, ids, ids_stride, rows,
                     (int)s_len, (int)pos0, (int)h1, (int)vocab, out);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

int embed_ragged_launch(const half_t* emb, const half_t* pos, const int32_t* ids, const int32_t* id_index,
                        const int32_t* positions, int64_t rows, int32_t h1, int32_t vocab, int32_t max_pos,
                        half_t* out, hipStream_t stream) {
  if (rows == 0) return FG_OK;
  const int64_t chunks = rows * (h1 / 8);
  int64_t blocks = ceil_div(chunks, 256);
  if (blocks > 256 * 32) blocks = 256 * 32;
  ProfScope prof(FG_K_EMBED, stream);
  hipLaunchKernelGGL(embed_ragged_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, emb, pos, ids, id_index,
                     positions, rows, (int)h1, (int)vocab, (int)max_pos, out);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

}  // namespace fg

using namespace fg;

extern "C" int fg_embed_ragged(const fg_model_cfg* cfg, const void* embed_f16, const void* pos_f16,
                               const int32_t* ids, const int32_t* positions, int64_t rows, void* out_f16,
                               void* stream) {
  if (!cfg) return FG_ERR_NULL;
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (rows < 0) return FG_ERR_SHAPE;
  if (rows == 0) return FG_OK;
  if (!embed_f16 || !pos_f16 || !ids || !positions || !out_f16) return FG_ERR_NULL;
  return embed_ragged_launch(reinterpret_cast<const half_t*>(embed_f16), reinterpret_cast<const half_t*>(pos_f16), ids,
                             nullptr, positions, rows, cfg->h1, cfg->vocab, cfg->max_pos,
                             reinterpret_cast<half_t*>(out_f16), as_stream(stream));
}

extern "C" int fg_layernorm(const void* x_f16, const void* gamma_f16, const void* beta_f16, int64_t rows,
                            int64_t cols, float eps, void* out_f16, void* stream) {
  if (rows < 0 || cols <= 0 || cols % 8 != 0 || rows > 0x7fffffff) return FG_ERR_SHAPE;
  if (rows == 0) return FG_OK;
  if (!x_f16 || !gamma_f16 || !beta_f16 || !out_f16) return FG_ERR_NULL;
  return layernorm_launch(reinterpret_cast<const half_t*>(x_f16), cols, reinterpret_cast<const half_t*>(gamma_f16),
                          reinterpret_cast<const half_t*>(beta_f16), rows, cols, eps,
                          reinterpret_cast<half_t*>(out_f16), cols, as_stream(stream));
}

extern "C" int fg_embed(const fg_model_cfg* cfg, const void* embed_f16, const void* pos_f16, const int32_t* ids,
                        int64_t rows, int32_t s_len, int32_t pos0, void* out_f16, void* stream) {
  if (!cfg) return FG_ERR_NULL;
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (rows < 0 || s_len <= 0 || pos0 < 0 || (int64_t)pos0 + s_len > cfg->max_pos) return FG_ERR_SHAPE;
  if (rows == 0) return FG_OK;
  if (!embed_f16 || !pos_f16 || !ids || !out_f16) return FG_ERR_NULL;
  return embed_launch(reinterpret_cast<const half_t*>(embed_f16), reinterpret_cast<const half_t*>(pos_f16), ids, 1,
                        rows, s_len, pos0, cfg->h1, cfg->vocab, reinterpret_cast<half_t*>(out_f16),
                        as_stream(stream));
}
