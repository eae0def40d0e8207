// Projections for a few rows of activations (Section 3: t.wQ, t.wK, t.wV, .wO, .w1, .w2 in a decode step of a
// small block, or the LM head on it), on weights in any of the stored formats: row-major FP16, canonical 4-bit,
// tiled 4-bit with binary32 or FP16 pairs.
//
// out[M, N] = act(x[M, K] . W[N, K]^T + bias) + residual
//
// With so few rows the product is the reading of the weights, and at the sizes of a decode layer that is a few
// microseconds: what decides the time is how many workgroups read at once, and that nothing follows the reading.
//   * A workgroup owns 16 CT output columns over the WHOLE contraction; its NW waves take NW ranges of it and meet
//     once in LDS: no partial sums in memory and no reduction pass (which took as long as the contraction: 8-23 us
//     behind 10-15 us on the OPT-6.7B shapes, 39 us on a 768-wide layer).
//   * Weights go straight to registers, 16 bytes per lane and load, two steps of 128 on their way at a time, without a
//     barrier in the loop.  (The compiler's one wait per pair of steps is for everything in flight, the step requested
//     last among it, so every pair exposes a memory latency.)  A lane holds 32 consecutive codes of one column (the 16 bytes that every 4-bit layout stores
//     together), so a step is four MFMAs per column tile, the i-th taking elements 8 i .. 8 i + 7 of every lane's
//     32: lane (row, kb) of the activation operand holds k = 128 step + 32 kb + 8 i.  (One 4-byte load per MFMA,
//     with k in its natural order, was up to twice as slow: the loads are bound by their number.)
//   * Activations: every wave copies its own ranges' rows global -> LDS, 1 KiB per transfer and only the four-row
//     pieces that exist, into a ring of two steps that no other wave touches.  Read as MFMA operands straight
//     from global memory (64 rows or columns of 16 bytes per load) they cost more than the weights from 16 rows up
//     (12288 x 49152, 16 rows: 108 -> 82 us; 4096 x 16384, 32 rows: 33 -> 23).
//   * 4-bit weights are dequantized in registers exactly as everywhere else (one rounding of min + code * scale).
// Measured against the kernels it took these row counts from, GEMM and reduction pass together, one run, us, 1 / 16
// / 32 rows.  Tiled 4-bit: 12288 x 4096 25.5 / 25.9 / 28.1 -> 9.6 / 10.9 / 13.1; 4096 x 16384 36.8 / 38.6 / 41.4 ->
// 11.9 / 16.5 / 23.1; 36864 x 12288 69 / 70 / - -> 51 / 66 / - (HBM time 45).  Canonical 4-bit: 4096 x 4096
// 26.9 / 220 / 431 -> 5.2 / 6.3 / 8.0.  FP16: 4096 x 4096 16 / 16.7 / 16.8 -> 8.1 / 10 / 12; 12288 x 4096 25.4 / 26 /
// 26.3 -> 18.5 / 21.5 / 24.3 (HBM time 16); 50272 x 4096 87 / 90 / - -> 68 / 88 / - (HBM time 66).
#include "fg_common.h"
#include "fg_async_lds.h"

namespace fg {

namespace {

constexpr int kFewStep = 128;   // contraction elements per step: 32 per lane

enum FewFormat { kFewF16 = 0, kFewQ4 = 1, kFewQ4Tiled = 2, kFewQ4TiledH16 = 3 };

struct FewArgs {
  const uint8_t* w;
  const uint8_t* meta;
  const half_t* x;
  int64_t ldx;
  int M, N, K;
  int steps;              // ceil(K / 128)
  const half_t* bias;
  const half_t* residual;
  int64_t ldr;
  int relu;
  half_t* out16;
  float* out32;
  int64_t ldo;
};

// NP = four-row pieces of activations a step needs (rows beyond 4 NP of the row tiles are never stored); NW = waves of
// the workgroup = ranges of the contraction
template <int FMT, int NP, int CT, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_fewrows_kernel(FewArgs a) {
  constexpr bool Q4 = FMT != kFewF16;
  constexpr int MT = (NP + 3) / 4;                         // row tiles of 16
  constexpr int NB = Q4 ? 1 : 4;                           // 16-byte weight loads per column tile and step
  constexpr int kPairBytes = FMT == kFewQ4TiledH16 ? 4 : 8;
  constexpr int kWStep = FMT == kFewF16 ? 256 : FMT == kFewQ4 ? 64 : 2048;    // bytes from a step's weights to the next's
  constexpr int kMStep = FMT == kFewQ4 ? 16 : 64 * kPairBytes;                // ... of {min, scale} pairs
  constexpr int kRing = 2 * NP * 1024;                     // bytes of a wave's activation ring
  constexpr int kRedBytes = NW * MT * CT * 1024;
  constexpr int kSmem = NW * kRing > kRedBytes ? NW * kRing : kRedBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kSmem];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kb = lane >> 4;
  const int n0 = blockIdx.x * (16 * CT);
  const int m0 = blockIdx.y * (4 * NP);
  // K = 64 mod 128: in the last step lanes kb = 2, 3 have no elements; they read those of kb - 2 (valid
  // memory), and zeros replace them on both sides of the product (an infinite weight times a zero would be a NaN)
  const int tail_step = (a.K & 64) ? a.steps - 1 : a.steps;
  const bool tail_lane = kb >= 2;

  const uint8_t* wp[CT];
  const uint8_t* mp[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    int col = n0 + 16 * ct + l16;
    col = col < a.N ? col : a.N - 1;   // ragged last column block: load valid data, never store it
    if constexpr (FMT == kFewF16) {
      wp[ct] = a.w + ((int64_t)col * a.K + 32 * kb) * 2;
      mp[ct] = nullptr;
    } else if constexpr (FMT == kFewQ4) {
      wp[ct] = a.w + (int64_t)col * (a.K >> 1) + 16 * kb;
      mp[ct] = a.meta + ((int64_t)col * (a.K >> 6) + (kb >> 1)) * 8;
    } else {
      const int64_t t = (int64_t)(col >> 5) * (a.K >> 6) + (kb >> 1);   // tile of the lane's first group
      wp[ct] = a.w + t * 1024 + 16 * (32 * (kb & 1) + (col & 31));
      mp[ct] = a.meta + (t * 32 + (col & 31)) * kPairBytes;
    }
  }
  constexpr int kWTail = FMT == kFewF16 ? 128 : FMT == kFewQ4 ? 32 : 1024;
  constexpr int kMTail = FMT == kFewQ4 ? 8 : 32 * kPairBytes;
  // Activations: piece p of a step is rows 4 p .. 4 p + 3 x 256 bytes, copied by one wave-wide asynchronous
  // transfer; 16-byte chunk c of row r lies at chunk c ^ (r & 15) of its row
  const half_t* xp[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 4 * p + (lane >> 4);
    int row = m0 + r;
    row = row < a.M ? row : a.M - 1;
    xp[p] = a.x + (int64_t)row * a.ldx;
  }
  unsigned char* ring = smem + wave * kRing;
  const uint32_t ring0 = (uint32_t)(uintptr_t)(lptr_t)ring;

  struct Buf {
    u4_t w[CT][NB];
    float2 pair[CT];
    uint32_t pair16[CT];
  };
  auto load = [&](Buf& b, int d, int step) {
    const bool tail = step == tail_step;
    const int xo = step * kFewStep;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      int c = l16 ^ ((4 * p + (lane >> 4)) & 15);
      c = tail ? c & 7 : c;
      __builtin_amdgcn_global_load_lds((gptr_t)(xp[p] + xo + 8 * c), (lptr_t)(ring + (d * NP + p) * 1024), 16, 0, 0);
    }
    // compute() takes the arrival of a weight register for the arrival of these copies: no weight load before them
    __builtin_amdgcn_sched_barrier(0);
    __asm__ volatile("; activation copies issued" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const bool back = tail && tail_lane;
    const int64_t wo = (int64_t)step * kWStep - (back ? kWTail : 0);
    const int64_t mo = (int64_t)step * kMStep - (back ? kMTail : 0);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
      for (int i = 0; i < NB; ++i) b.w[ct][i] = *reinterpret_cast<const u4_t*>(wp[ct] + wo + 16 * i);
      if constexpr (FMT == kFewQ4TiledH16)
        b.pair16[ct] = *reinterpret_cast<const uint32_t*>(mp[ct] + mo);
      else if constexpr (Q4)
        b.pair[ct] = *reinterpret_cast<const float2*>(mp[ct] + mo);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f4_t acc[MT][CT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[m][ct] = (f4_t){0.f, 0.f, 0.f, 0.f};

  // LDS offset of the lane's row in row tile m, and its chunk 4 kb + i
  uint32_t x_row[MT];
  int x_swz[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    int r = 16 * m + l16;
    r = r < 4 * NP ? r : 4 * NP - 1;
    x_row[m] = ring0 + r * 256;
    x_swz[m] = r & 15;
  }

  auto compute = [&](Buf& b, int d, int step) {
    // The step's activation copies were issued before its weight loads and loads complete in order: once the
    // first weight register is there, so are the activations.  The empty statement makes the reads' address
    // depend on that register.
    uint32_t off = d * NP * 1024;
    __asm__ volatile("" : "+v"(off) : "v"(b.w[0][0]));
    u4_t x[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[m][i] = lds_read128<0>(off + x_row[m] + (((4 * kb + i) ^ x_swz[m]) << 4));
    if (step == tail_step) {   // wave-uniform
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int i = 0; i < NB; ++i) b.w[ct][i] = tail_lane ? (u4_t){0u, 0u, 0u, 0u} : b.w[ct][i];
        if constexpr (FMT == kFewQ4TiledH16)
          b.pair16[ct] = tail_lane ? 0u : b.pair16[ct];
        else if constexpr (Q4)
          b.pair[ct] = tail_lane ? make_float2(0.f, 0.f) : b.pair[ct];
      }
    }
    bool waited = false;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      float s24 = 0.f, s20 = 0.f, mn = 0.f;
      if constexpr (Q4) {
        float2 p;
        if constexpr (FMT == kFewQ4TiledH16) {
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
        if (!waited) {
          waited = true;
          lds_wait();
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_landed(x[m][j]);
          if (step == tail_step) {   // wave-uniform
            const u4_t z = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
              for (int j = 0; j < 4; ++j) x[m][j] = tail_lane ? z : x[m][j];
          }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
          acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, x[m][i]),
                                                              __builtin_bit_cast(h8_t, bw), acc[m][ct], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // Two steps in flight, none loaded twice (a 768-wide contraction is one step per wave).  The steady loop has
  // no condition around its loads.
  int s = a.steps * wave / NW;
  const int s1 = a.steps * (wave + 1) / NW;
  Buf b0, b1;
  if (s1 - s >= 4) {
    load(b0, 0, s);
    load(b1, 1, s + 1);
    for (; s + 4 <= s1; s += 2) {
      compute(b0, 0, s);
      load(b0, 0, s + 2);
      compute(b1, 1, s + 1);
      load(b1, 1, s + 3);
    }
  } else {
    if (s < s1) load(b0, 0, s);
    if (s + 1 < s1) load(b1, 1, s + 1);
  }
  const int left = s1 - s;   // 0 .. 3, the first two of them loaded
  if (left >= 1) compute(b0, 0, s);
  if (left == 3) load(b0, 0, s + 2);
  if (left >= 2) compute(b1, 1, s + 1);
  if (left == 3) compute(b0, 0, s + 2);

  // ---- the waves' sums meet in LDS (over the rings: every copy has landed and been read); thread t finishes
  // items t, t + 64 NW, ... of (row tile, column tile, lane)
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  float4(*red)[MT * CT][64] = reinterpret_cast<float4(*)[MT * CT][64]>(smem);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      red[wave][m * CT + ct][lane] = make_float4(acc[m][ct][0], acc[m][ct][1], acc[m][ct][2], acc[m][ct][3]);
  __syncthreads();
  for (int e = tid; e < MT * CT * 64; e += NW * 64) {
    const int mc = e >> 6, el = e & 63, m = mc / CT, ct = mc - m * CT;
    const int col = n0 + 16 * ct + (el & 15), r0 = 16 * m + 4 * (el >> 4), row0 = m0 + r0;
    if (col >= a.N || row0 >= a.M || r0 >= 4 * NP) continue;
    const float bv = a.bias ? (float)a.bias[col] : 0.f;
    float res[4] = {0.f, 0.f, 0.f, 0.f};
    if (a.residual) {
#pragma unroll
      for (int r = 0; r < 4; ++r) res[r] = (float)a.residual[(int64_t)(row0 + r < a.M ? row0 + r : row0) * a.ldr + col];
    }
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 p = red[w][mc][el];
      v[0] += p.x;
      v[1] += p.y;
      v[2] += p.z;
      v[3] += p.w;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + r;
      if (row >= a.M) break;
      float y = v[r] + bv;
      if (a.relu) y = fmaxf(y, 0.f);
      y += res[r];
      if (a.out32)
        a.out32[(int64_t)row * a.ldo + col] = y;
      else
        a.out16[(int64_t)row * a.ldo + col] = (half_t)y;
    }
  }
}

template <int FMT, int NP, int CT, int NW>
int launch_few(const FewArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)ceil_div(a.N, 16 * CT), (unsigned)ceil_div(a.M, 4 * NP));
  hipLaunchKernelGGL((gemm_fewrows_kernel<FMT, NP, CT, NW>), grid, dim3(NW * 64), 0, stream, a);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

FewArgs make_few(const LinearArgs& la) {
  FewArgs a;
  a.w = reinterpret_cast<const uint8_t*>(la.w_data);
  a.meta = reinterpret_cast<const uint8_t*>(la.w_meta);
  a.x = la.x;
  a.ldx = la.ldx;
  a.M = (int)la.m;
  a.N = (int)la.n;
  a.K = (int)la.k;
  a.steps = (int)ceil_div(la.k, kFewStep);
  a.bias = la.bias;
  a.residual = la.residual;
  a.ldr = la.ldr;
  a.relu = la.relu;
  a.out16 = la.out_f16;
  a.out32 = la.out_f32;
  a.ldo = la.ldo;
  return a;
}

// Column tiles per workgroup.  A CU's share is ceil(workgroups / 256) of them (a row block of 32 has its own), and a workgroup costs its CT column
// tiles plus the activations it pulls in, which in units of a column tile's weights are 0.04 per row (FP16 weights:
// 0.015, their tiles are three times the bytes).  Fitted to sweeps of CT = 1..6 over 25 matrices; it picks the fastest
// or one within 4 % of it in all but two of them.
int pick_ct(int fmt, int64_t n, int64_t m) {
  const int64_t blocks = ceil_div(m, 32);
  const double rows = (fmt == kFewF16 ? 0.015 : 0.04) * (double)(m < 32 ? m : 32);
  int best = 1;
  double best_cost = 0;
  for (int ct = 1; ct <= 4; ++ct) {
    const double cost = (double)ceil_div(ceil_div(n, 16 * ct) * blocks, 256) * (ct + rows);
    if (ct == 1 || cost < best_cost) {
      best = ct;
      best_cost = cost;
    }
  }
  return best;
}

template <int FMT, int NP>
int launch_few_np(const FewArgs& a, hipStream_t stream) {
  const int ct = pick_ct(FMT, a.N, a.M);
  // Where every CU has one workgroup and a long contraction, sixteen waves keep twice the bytes in flight: 4096 x
  // 16384, one row, FP16 38 -> 31 us, tiled 13.8 -> 11.9; 7168 x 28672 tiled 31.8 -> 28.3.  Shorter contractions gain
  // nothing, canonical 4-bit weights lose 4 %, FP16 weights lose 15 % with two column tiles.
  if constexpr (FMT != kFewQ4 && NP <= 4) {
    if (ceil_div(a.N, 16 * ct) <= 256 && a.steps >= (FMT == kFewF16 ? 128 : 64)) {
      if (ct == 1) return launch_few<FMT, NP, 1, 16>(a, stream);
      if constexpr (FMT != kFewF16)
        if (ct == 2) return launch_few<FMT, NP, 2, 16>(a, stream);
    }
  }
  switch (ct) {
    case 1: return launch_few<FMT, NP, 1, 8>(a, stream);
    case 2: return launch_few<FMT, NP, 2, 8>(a, stream);
    case 3: return launch_few<FMT, NP, 3, 8>(a, stream);
    default: return launch_few<FMT, NP, 4, 8>(a, stream);
  }
}

template <int FMT>
int launch_few_fmt(const FewArgs& a, hipStream_t stream) {
  if (a.M <= 4) return launch_few_np<FMT, 1>(a, stream);
  if (a.M <= 8) return launch_few_np<FMT, 2>(a, stream);
  if (a.M <= 16) return launch_few_np<FMT, 4>(a, stream);
  return launch_few_np<FMT, 8>(a, stream);
}

}  // namespace

// Which calls this kernel takes.  Up to 16 rows all of them but FP16 weights of few columns and a long contraction; up
// to 32 rows those whose matrix is small enough for the activations of its many workgroups not to cost more than the
// wider tiles' partial sums.  Measured at 32 rows against the kernel that otherwise runs (us): tiled 28672 x 7168 43 vs 48,
// 7168 x 28672 49 vs 56, 36864 x 12288 84 vs 76, 12288 x 49152 101 vs 98; FP16 21504 x 7168 68 vs 69, 12288 x 12288
// 58 vs 70, 7168 x 28672 100 vs 97, 50272 x 4096 102 vs 96; canonical always (46 vs 135 and more).
// FP16 weights, few columns, long contraction: a workgroup's time grows with the contraction and too few of them read.
//   columns x contraction, this kernel vs the one that splits it, us: 1 row 1280 x 16384 18.6 vs 19.2, x 20480 23.8 vs
//   21.1; 8 rows 2560 x 20480 31 vs 34, 2048 x 20480 30 vs 25; 16 rows 3072 x 16384 31 vs 34, 2048 x 16384 29 vs 23;
//   24 rows 3072 x 12288 27 vs 30, 2560 x 12288 26 vs 23.  (Up to 8192 deep it is level or better: 640 x 8192, 16 rows,
//   12 vs 12.)
// More rows, in blocks of 32 that each read the matrix: as long as matrix x blocks is small, the other kernels leave most
// of the chip without work, or split the contraction into partial sums.  The line is where both take the same time, us:
//   tiled, 110 M    768 x 768 x 128 rows 4.6 vs 12.4; 2304 x 768 x 1000 22 vs 32; 2048 x 2048 x 640 21 vs 43;
//                   4096 x 4096 x 64 9.1 vs 20, x 192 23 vs 24; 7168 x 7168 x 64 21 vs 25, x 96 33 vs 32;
//                   12288 x 4096 x 64 22.8 vs 23.3; 4096 x 16384 x 64 29 vs 26
//   FP16, 34 M      2048 x 2048 x 128 8.1 vs 13; 4096 x 4096 x 64 15.9 vs 15.7, x 96 27 vs 19
//   FP16 beyond 128 rows, 70 M   2304 x 768 x 320 10 vs 18; 2048 x 2048 x 450 22 vs 39; 6144 x 2048 x 144 24 vs 30,
//                   x 192 29 vs 26
//   canonical, 600 M   7168 x 7168 x 320 118 vs 184, x 384 level; 4096 x 16384 x 320 0.62 of the other's time; 7168 x
//                   28672 x 33 85 vs 325; 36864 x 12288 x 33 201 vs 183.  From 161 rows the wider matrices lose earlier:
//                   12288 x 4096 x 320 (503 M) 119 vs 161, x 333 (553 M) 128 vs 113; 33000 x 1024 x 320 (337 M) 0.86 of
//                   the other's time, x 384 (405 M) 124 vs 105; 16384 x 4096 x 161 (402 M) 92 vs 73
//   canonical beyond 512 rows, 300 M   2048 x 2048 x 1000 36 vs 87; 6144 x 2048 x 640 66 vs 87, x 1000 98 vs 89
// and, where the contraction is short, as long as columns x blocks is: then a workgroup is little more than its start and
// its epilogue, and the wider tiles have fewer of them.
//   tiled           16384 x 64 x 128 rows (65536) 13.9 vs 14.8, x 200 (114688) 23 vs 14.7; 4096 x 256 x 1000 (131072)
//                   31 vs 39; 8192 x 768 x 512 (131072) 32 vs 38; 16384 x 768 x 192 (98304) 25 vs 27, x 256 (131072) 32 vs
//                   31; 50272 x 64 x 32 14.4 vs 8.6, x 256 x 32 16.1 vs 17.6
//   FP16            up to 128 rows the narrow tiles come without remainder where 4096 divides the columns: 4096 x 768 x
//                   64 (8192) 5.0 vs 5.6, x 100 (16384) 6.5 vs 6.3, 4096 x 64 x 64 3.5 vs 3.0; elsewhere 6144 x 1024 x
//                   128 (24576) 12 vs 15, 28672 x 1024 x 40 (57344) 33 vs 26.  Beyond 128 rows 8192 x 768 x 256
//                   (65536) 22 vs 25; 4096 x 512 x 1000 (131072) 33 vs 38; 16384 x 512 x 200 (114688) 32 vs 28
//   canonical       16384 x 64 x 128 (65536) 13.7 vs 17.7, x 200 (114688) 23 vs 18; 50272 x 192 x 128 (201088) 50 vs 63,
//                   x 200 (351904) 82 vs 76; 50272 x 384 x 320 (502720) 104 vs 130, x 512 164 vs 124; 16384 x 512 x 512
//                   (262144) 61 vs 28; beyond 512 rows 4096 x 64 x 1000 (131072) 26 vs 29, 16384 x 256 x 1000 116 vs 43
// The FP16 lines beyond 32 rows are older than gemm_f16_tiles_kernel, which takes what lies past them now: measured against the
// kernels before it, they keep sizes at which it would be the faster one (2304 x 768 at 1000 rows 29.7 us here, 12.3 there).
// (FP16 columns that 32 does not divide are outside the FP16 exceptions: the kernel they would fall to is the slow one.)
bool gemm_fewrows_takes(int dtype, int64_t n, int64_t k, int64_t m) {
  if (m < 1 || m > 1024 || k % kGroup != 0) return false;
  const bool f16 = dtype == FG_F16, streams = n % 32 == 0;
  if (f16 && streams && k > 8192 && k > n * (m <= 4 ? 10 : (m <= 8 ? 8 : (m <= 16 ? 6 : 4)))) return false;
  if (m <= 16) return true;
  const int64_t size = n * k, blocks = ceil_div(m, 32), wide = n * blocks;
  if (m <= 32) {
    if (dtype == FG_Q4G64) return true;
    if (f16) return size <= 160000000 && n <= 32768;
    return size <= 220000000 && (k >= 256 || n <= 32768);
  }
  if (dtype == FG_Q4G64) {
    const int64_t line = m <= 160                ? 600000000
                         : m > 512               ? 300000000
                         : n <= 10240            ? 600000000
                         : n < 16384             ? 510000000
                                                 : 340000000;
    if (size > line / blocks) return false;
    if (m <= 512 && k < 192) return wide <= 81920;
    return (m <= 320 && k >= 256) || wide <= 204800;
  }
  if (f16) {
    if (size > (m <= 128 ? 34000000 : 70000000) / blocks) return false;
    if (!streams) return true;
    if (m > 128) return wide <= (k < 256 || n > 8192 ? 65536 : 131072);
    return n % 4096 == 0 ? wide <= 8192 && k >= 192 : wide <= 24576;
  }
  return size <= 110000000 / blocks && wide <= (k < 256 ? 65536 : (n <= 8192 ? 131072 : 98304));
}

bool gemm_ln_fewrows_takes(int dtype, int64_t n, int64_t k, int64_t m) {
  return gemm_fewrows_takes(dtype, n, k, m) &&
         gemm_fewrows_ln_takes(dtype, n, k, m, pick_ct(dtype == FG_F16 ? kFewF16 : kFewQ4, n, m));
}

int gemm_ln_fewrows_launch(const LinearArgs& la, const half_t* gamma, const half_t* beta, float eps, hipStream_t stream) {
  ProfScope prof(FG_K_GEMM_SMALL_M, stream);
  return gemm_fewrows_ln_launch(la, gamma, beta, eps, pick_ct(la.dtype == FG_F16 ? kFewF16 : kFewQ4, la.n, la.m), stream);
}

int gemm_fewrows_launch(const LinearArgs& la, hipStream_t stream) {
  if (la.m == 0 || la.n == 0) return FG_OK;
  const FewArgs a = make_few(la);
  ProfScope prof(FG_K_GEMM_SMALL_M, stream);
  switch (la.dtype) {
    case FG_F16: return launch_few_fmt<kFewF16>(a, stream);
    case FG_Q4G64: return launch_few_fmt<kFewQ4>(a, stream);
    case FG_Q4G64_TILED: return launch_few_fmt<kFewQ4Tiled>(a, stream);
    case FG_Q4G64_H16_TILED: return launch_few_fmt<kFewQ4TiledH16>(a, stream);
  }
  return FG_ERR_UNSUPPORTED;
}

}  // namespace fg
