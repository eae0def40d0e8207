// Projections of a LayerNorm for up to eight rows of activations, on weights in any of the stored formats: LayerNorm and
// t.wQ, t.wK, t.wV, or LayerNorm and .w1, of a decode step (Section 3) of a small block in one launch.
//
// out[M, N] = act(LayerNorm(x)[M, K] . W[N, K]^T + bias)
//
// What bounds it: a launch takes 2.3 us however little it does, and the LayerNorm of a few rows is little more than that.
// So a workgroup normalizes the rows for itself, into LDS, while its first weights are on their way.  A 4096-wide 4-bit
// layer of one row 54.2 -> 48.2 us, of five rows on canonical weights 66.9 -> 59.7, of eight 68.5 -> 64.0; FP16 weights, four
// rows, 105 -> 99.7; a 768-wide layer of four rows 26.4 -> 24.2.
//   * Same results as layernorm_reg_kernel (fg_norm.hip) and gemm_fewrows_kernel (fg_gemm_fewrows.hip), bit for bit: 256
//     lanes take pieces of eight elements, four groups of 64 lanes fold, the four sums are added in order; eight ranges of
//     the contraction, four 16x16x32 MFMAs per step of 128 and column tile, the ranges' sums added in order.
//   * One step of weights is requested before the LayerNorm and the second behind it.  A wave that asks for more is held at
//     its loads until the memory system has room for them, that is for as long as the transfer of most of the matrix
//     takes, and its LayerNorm waits with it (4096 wide, one row, us a layer: one step 47.6, one and one 48.2, three 52.0,
//     four 53.4; with eight rows 59.2 / 57.9 / 62.7 / 64.7).
//   * No asynchronous copy in the loop: a kernel that mixes copies into LDS with loads into registers makes the compiler
//     wait for ALL loads in flight at every use, because it no longer counts them.  Here every use waits for its own step.
//   * Every address is a scalar base and one offset per lane.
#include "fg_common.h"

namespace fg {

namespace {

constexpr int NW = 8;           // waves of a workgroup = ranges of the contraction
constexpr int kStep = 128;      // contraction elements per step: 32 per lane
constexpr int kLnRows = 8;      // rows of activations: four for each of two groups of four waves
constexpr int kLnMaxK = 4096;   // 64 KiB of LDS for eight such rows

enum LnFormat { kLnF16 = 0, kLnQ4 = 1, kLnQ4Tiled = 2, kLnQ4TiledH16 = 3 };

struct LnArgs {
  const uint8_t* w;
  const uint8_t* meta;
  const half_t* x;
  int64_t ldx;
  int M, N, K;
  int steps;              // ceil(K / 128)
  const half_t* bias;
  half_t* out16;
  int64_t ldo;
  const half_t* gamma;
  const half_t* beta;
  float eps;
  int relu;
};

// Waits for the LDS accesses of this wave, then for the other waves; loads of weights in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

// NW waves = ranges of the contraction; CT column tiles per workgroup; D steps of weights in flight per wave; NC pieces of
// eight elements per lane and row, K <= 2048 NC.
template <int FMT, int CT, int D, int NC>
__global__ __launch_bounds__(NW * 64) void gemm_fewrows_ln_kernel(LnArgs a) {
  constexpr bool Q4 = FMT != kLnF16;
  constexpr int NB = Q4 ? 1 : 4;                           // 16-byte weight loads per column tile and step
  constexpr int kPairBytes = FMT == kLnQ4TiledH16 ? 4 : 8;
  constexpr int kWStep = FMT == kLnF16 ? 256 : FMT == kLnQ4 ? 64 : 2048;    // bytes from a step's weights to the next's
  constexpr int kMStep = FMT == kLnQ4 ? 16 : 64 * kPairBytes;               // ... of {min, scale} pairs
  constexpr int kWTail = FMT == kLnF16 ? 128 : FMT == kLnQ4 ? 32 : 1024;
  constexpr int kMTail = FMT == kLnQ4 ? 8 : 32 * kPairBytes;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // activations; then the ranges' sums
  __shared__ float ln_red[2][kLnRows][4];

  // all arguments at once: each one loaded where it is first needed would be another wait of its own
  __asm__ volatile("" ::"s"(a.w), "s"(a.meta), "s"(a.x), "s"(a.ldx), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.steps));
  __asm__ volatile("" ::"s"(a.bias), "s"(a.relu), "s"(a.out16), "s"(a.ldo), "s"(a.gamma), "s"(a.beta), "s"(a.eps));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kb = lane >> 4;
  const int n0 = blockIdx.x * (16 * CT);
  const uint32_t row_bytes = (uint32_t)a.steps * 256;
  const int s0 = a.steps * wave / NW, s1 = a.steps * (wave + 1) / NW;
  const int pieces = a.K >> 3;
  const int vw = wave & 3, grp = wave >> 2;   // quarter of every 256 pieces, first row

  // ---- rows, gamma and beta
  u4_t xv[kLnRows / 2][NC], gv[NC], bv[NC];
  int at[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int c = 64 * vw + lane + 256 * j;
    at[j] = (c < pieces ? c : pieces - 1) * 8;
  }
#pragma unroll
  for (int i = 0; i < kLnRows / 2; ++i) {
    const int row = grp + 2 * i;
    if (row < a.M) {   // wave-uniform
#pragma unroll
      for (int j = 0; j < NC; ++j) xv[i][j] = *reinterpret_cast<const u4_t*>(a.x + (int64_t)row * a.ldx + at[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    gv[j] = *reinterpret_cast<const u4_t*>(a.gamma + at[j]);
    bv[j] = *reinterpret_cast<const u4_t*>(a.beta + at[j]);
  }
  // ---- the bias of the outputs this thread finishes: wave w finishes column tile w
  const int ecol = n0 + 16 * wave + l16, erow0 = 4 * kb;
  uint32_t bias_v = 0;   // FP16 bits
  if (a.bias && wave < CT) bias_v = reinterpret_cast<const uint16_t*>(a.bias)[ecol < a.N ? ecol : a.N - 1];

  // ---- weights: a scalar base per column tile, one offset per lane
  // K = 64 mod 128: in the last step lanes kb = 2, 3 have no elements; they read those of kb - 2 (valid memory), and zeros
  // replace them on both sides of the product (an infinite weight times a zero would be a NaN)
  const int tail_step = (a.K & 64) ? a.steps - 1 : a.steps;
  const bool tail_lane = kb >= 2;
  const uint8_t* wbase[CT];
  const uint8_t* mbase[CT];
  uint32_t woff[CT], moff[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    int c0 = n0 + 16 * ct;   // ragged last column block: load valid data, never store it
    if constexpr (FMT == kLnQ4Tiled || FMT == kLnQ4TiledH16) {
      c0 = c0 < a.N ? c0 : a.N - 16;
      const int64_t t = (int64_t)(c0 >> 5) * (a.K >> 6);
      const int c = (c0 & 16) + l16;
      wbase[ct] = a.w + t * 1024;
      woff[ct] = (kb >> 1) * 1024 + 16 * (32 * (kb & 1) + c);
      mbase[ct] = a.meta + t * 32 * kPairBytes;
      moff[ct] = ((kb >> 1) * 32 + c) * kPairBytes;
    } else {
      c0 = c0 < a.N ? c0 : a.N - 1;
      const int c = c0 + l16 < a.N ? l16 : a.N - 1 - c0;
      if constexpr (FMT == kLnF16) {
        wbase[ct] = a.w + (int64_t)c0 * a.K * 2;
        woff[ct] = (uint32_t)c * (uint32_t)(a.K * 2) + 64 * kb;
        mbase[ct] = nullptr;
        moff[ct] = 0;
      } else {
        wbase[ct] = a.w + (int64_t)c0 * (a.K >> 1);
        woff[ct] = (uint32_t)c * (uint32_t)(a.K >> 1) + 16 * kb;
        mbase[ct] = a.meta + (int64_t)c0 * (a.K >> 6) * 8;
        moff[ct] = ((uint32_t)c * (uint32_t)(a.K >> 6) + (kb >> 1)) * 8;
      }
    }
  }

  struct Buf {
    u4_t w[CT][NB];
    float2 pair[CT];
    uint32_t pair16[CT];
  };
  auto load = [&](Buf& b, int step) {
    const bool back = step == tail_step && tail_lane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint8_t* wb = wbase[ct] + (int64_t)step * kWStep;
      const uint32_t wo = woff[ct] - (back ? kWTail : 0);
#pragma unroll
      for (int i = 0; i < NB; ++i) b.w[ct][i] = *reinterpret_cast<const u4_t*>(wb + wo + 16 * i);
      if constexpr (Q4) {
        const uint8_t* mb = mbase[ct] + (int64_t)step * kMStep;
        const uint32_t mo = moff[ct] - (back ? kMTail : 0);
        if constexpr (FMT == kLnQ4TiledH16)
          b.pair16[ct] = *reinterpret_cast<const uint32_t*>(mb + mo);
        else
          b.pair[ct] = *reinterpret_cast<const float2*>(mb + mo);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f4_t acc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) acc[ct] = (f4_t){0.f, 0.f, 0.f, 0.f};
  const int xr = l16 < a.M ? l16 : a.M - 1;   // (rows beyond M: results that are never stored)
  const unsigned char* x_row = smem + xr * row_bytes;
  const int x_swz = xr & 15;
  const u4_t zero4 = {0u, 0u, 0u, 0u};

  auto compute = [&](Buf& b, int step) {
    u4_t x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const u4_t*>(x_row + step * 256 + (((4 * kb + i) ^ x_swz) << 4));
    if (step == tail_step) {   // wave-uniform; the activations' tail in LDS is zeros
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int i = 0; i < NB; ++i) b.w[ct][i] = tail_lane ? zero4 : b.w[ct][i];
        if constexpr (FMT == kLnQ4TiledH16)
          b.pair16[ct] = tail_lane ? 0u : b.pair16[ct];
        else if constexpr (Q4)
          b.pair[ct] = tail_lane ? make_float2(0.f, 0.f) : b.pair[ct];
      }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      float s24 = 0.f, s20 = 0.f, mn = 0.f;
      if constexpr (Q4) {
        float2 p;
        if constexpr (FMT == kLnQ4TiledH16) {
          const h2_t pr = __builtin_bit_cast(h2_t, b.pair16[ct]);
          p = make_float2((float)pr.x, (float)pr.y);
        } else {
          p = b.pair[ct];
        }
        s24 = p.y * 16777216.0f;
        s20 = p.y * 1048576.0f;
        mn = p.x;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u4_t bw;
        if constexpr (Q4) {
          uint32_t c[4];
          dequant8_exact(b.w[ct][0][i], s24, s20, mn, c);
          bw = (u4_t){c[0], c[1], c[2], c[3]};
        } else {
          bw = b.w[ct][i];
        }
        acc[ct] =
            __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, x[i]), __builtin_bit_cast(h8_t, bw), acc[ct], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // No load stands under a condition: behind one the compiler would have to wait as if it had not been issued, that is
  // for everything.  A wave with fewer steps than D, or than it has room for at the end, loads its last step again.
  Buf b[D];
  const int last = s1 > s0 ? s1 - 1 : s0;
  auto clamped = [&](int step) { return step < last ? step : last; };
  load(b[0], clamped(s0));

  // ---- LayerNorm, while the weights are on their way
  const float cols = (float)a.K;
#pragma unroll
  for (int i = 0; i < kLnRows / 2; ++i) {
    const int row = grp + 2 * i;
    if (row < a.M) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NC; ++j) __asm__ volatile("" : "+v"(xv[i][j]));   // not to be converted where it is loaded
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (64 * vw + lane + 256 * j < pieces) {
          const h8_t v = __builtin_bit_cast(h8_t, xv[i][j]);
#pragma unroll
          for (int e = 0; e < 8; ++e) s += (float)v[e];
        }
      s = wave_sum(s);
      if (lane == 0) ln_red[0][row][vw] = s;
    }
  }
  lds_barrier();
  float mean[kLnRows / 2];
#pragma unroll
  for (int i = 0; i < kLnRows / 2; ++i) {
    const int row = grp + 2 * i;
    if (row < a.M) {
      const float* red = ln_red[0][row];
      mean[i] = (red[0] + red[1] + red[2] + red[3]) / cols;
      float q = 0.f;
#pragma unroll
      for (int j = 0; j < NC; ++j)
        if (64 * vw + lane + 256 * j < pieces) q = ln_add_squares(__builtin_bit_cast(h8_t, xv[i][j]), mean[i], q, j == 0);
      q = wave_sum(q);
      if (lane == 0) ln_red[1][row][vw] = q;
    }
  }
  lds_barrier();
#pragma unroll
  for (int i = 0; i < kLnRows / 2; ++i) {
    const int row = grp + 2 * i;
    if (row < a.M) {
      const float* red = ln_red[1][row];
      const float rstd = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / cols + a.eps);
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int c = 64 * vw + lane + 256 * j;
        if (c < a.steps * 16) {   // 16-byte chunk c of row r lies at chunk c ^ (r & 15) of its row; past K: zeros
          const h8_t o = ln_normalize(__builtin_bit_cast(h8_t, xv[i][j]), mean[i], rstd, __builtin_bit_cast(h8_t, gv[j]), __builtin_bit_cast(h8_t, bv[j]));
          *reinterpret_cast<u4_t*>(smem + row * row_bytes + ((c ^ (row & 15)) << 4)) = c < pieces ? __builtin_bit_cast(u4_t, o) : zero4;
        }
      }
    }
  }
#pragma unroll
  for (int j = 1; j < D; ++j) load(b[j], clamped(s0 + j));
  lds_barrier();

  int s = s0;
  for (; s + D < s1; s += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      compute(b[j], s + j);
      load(b[j], clamped(s + j + D));
    }
  }
#pragma unroll
  for (int j = 0; j < D; ++j)
    if (s + j < s1) compute(b[j], s + j);

  // ---- the ranges' sums meet in LDS, over the activations
  lds_barrier();
  float4(*red)[CT][64] = reinterpret_cast<float4(*)[CT][64]>(smem);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) red[wave][ct][lane] = make_float4(acc[ct][0], acc[ct][1], acc[ct][2], acc[ct][3]);
  lds_barrier();
  if (wave >= CT || ecol >= a.N || erow0 >= a.M) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float4 p = red[w][wave < CT ? wave : 0][lane];
    v[0] += p.x;
    v[1] += p.y;
    v[2] += p.z;
    v[3] += p.w;
  }
  __asm__ volatile("" : "+v"(bias_v));
  const float bias_f = (float)__builtin_bit_cast(half_t, (uint16_t)bias_v);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = erow0 + r;
    if (row >= a.M) break;
    float y = v[r] + bias_f;
    if (a.relu) y = fmaxf(y, 0.f);
    a.out16[(int64_t)row * a.ldo + ecol] = (half_t)y;
  }
}

template <int FMT, int CT, int D, int NC>
int launch_ln(const LnArgs& a, hipStream_t stream) {
  auto* kern = &gemm_fewrows_ln_kernel<FMT, CT, D, NC>;
  static bool attr_done = false;
  if (!attr_done) {
    FG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLnRows * kLnMaxK * 2));
    attr_done = true;
  }
  const size_t rows = (size_t)a.M * a.steps * 256, red = (size_t)NW * CT * 1024;
  hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(a.N, 16 * CT)), dim3(NW * 64), rows > red ? rows : red, stream, a);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

template <int FMT>
int launch_ln_fmt(const LnArgs& a, int ct, hipStream_t stream) {
  if (a.steps <= NW) return launch_ln<FMT, 1, 1, 1>(a, stream);   // at most one step per wave
  switch (ct) {
    case 1: return launch_ln<FMT, 1, 2, 2>(a, stream);
    case 2: return launch_ln<FMT, 2, 2, 2>(a, stream);
    case 3: return launch_ln<FMT, 3, 2, 2>(a, stream);
    default: return launch_ln<FMT, 4, 2, 2>(a, stream);
  }
}

}  // namespace

// As long as the workgroups are one round (each round would normalize again: 7168 wide, 336 and 448 workgroups, one row, 107
// -> 116 us a layer) and the rows few enough not to hold up the weights: tiled 4-bit 4096 wide, six rows 57.8 -> 55.2 us,
// eight 58.6 -> 57.9, but 2048 wide, eight rows, 37.7 -> 38.0.
bool gemm_fewrows_ln_takes(int dtype, int64_t n, int64_t k, int64_t m, int ct) {
  const int64_t rows = dtype == FG_F16 || dtype == FG_Q4G64 ? kLnRows : kLnRows - 2;
  return m >= 1 && m <= rows && k <= kLnMaxK && ceil_div(n, 16 * (k <= NW * kStep ? 1 : ct)) <= 256;
}

int gemm_fewrows_ln_launch(const LinearArgs& la, const half_t* gamma, const half_t* beta, float eps, int ct, hipStream_t stream) {
  if (la.residual || la.out_f32) return FG_ERR_UNSUPPORTED;
  LnArgs a;
  a.w = reinterpret_cast<const uint8_t*>(la.w_data);
  a.meta = reinterpret_cast<const uint8_t*>(la.w_meta);
  a.x = la.x;
  a.ldx = la.ldx;
  a.M = (int)la.m;
  a.N = (int)la.n;
  a.K = (int)la.k;
  a.steps = (int)ceil_div(la.k, kStep);
  a.bias = la.bias;
  a.relu = la.relu;
  a.out16 = la.out_f16;
  a.ldo = la.ldo;
  a.gamma = gamma;
  a.beta = beta;
  a.eps = eps;
  switch (la.dtype) {
    case FG_F16: return launch_ln_fmt<kLnF16>(a, ct, stream);
    case FG_Q4G64: return launch_ln_fmt<kLnQ4>(a, ct, stream);
    case FG_Q4G64_TILED: return launch_ln_fmt<kLnQ4Tiled>(a, ct, stream);
    case FG_Q4G64_H16_TILED: return launch_ln_fmt<kLnQ4TiledH16>(a, ct, stream);
  }
  return FG_ERR_UNSUPPORTED;
}

}  // namespace fg
