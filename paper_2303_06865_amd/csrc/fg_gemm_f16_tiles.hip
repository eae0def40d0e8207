// Projections of some hundred rows on row-major FP16 weights (the prefill of one or a few prompts, the LM head of a block).
//
// out[M, N] = act(x[M, K] . W[N, K]^T + bias) + residual
//
// What bounds them: how fast a CU takes operands in.  256 CUs together read 30 TB/s from L2, but 60 to 75 GB/s each while
// part of it comes from HBM, and a tile of BM x BN takes in BM + BN rows of 128 bytes per step of 64, so the tiles have
// to be as large as leaves none of the CUs idle.  The kernels that this one took these sizes from have one tile of 192 or
// 256 x 256; at these sizes they cut it along the contraction to fill the chip, and pay with partial sums and a second pass.
//   * Tiles from 32 x 64 to 256 x 128, each with the whole contraction to itself where there are enough of them; which one, and
//     into how many ranges a long contraction is cut, is decided by what each measured (gemm_f16_tiles_pick).
//   * Four waves compute, as 2 x 2, one per SIMD: of 16 MT x 16 NT each, so an operand that is in LDS is read twice and not
//     eight times.  Four other waves do nothing but copy, global -> LDS, three to five steps ahead.  A copy holds the
//     wave that issues it for as long as the path into the CU is busy; in the computing waves that was time without an MFMA
//     (333 rows, 12288 x 4096: 66 us with the copies between the MFMAs, 57 with waves of their own).
//   * One barrier per step: the copies of the next step have landed, and nobody reads the stage of this step any more.
//   * The finished sums go through LDS, so that residual and results move 16 bytes per lane, all residual loads at once (57 ->
//     46 us; row by row, each load waited for the one before).
//   * The accumulators are updated in place by hand-placed instructions: left to the compiler, the loop moves them between
//     register files (92 -> 82 us at 16384 x 4096 when that was changed).
// Measured against those kernels, GEMM and second pass, us: 333 rows 12288 x 4096 72.5 -> 46.2, 4096 x 4096 32.9 -> 21.2, 16384 x
// 4096 74.3 -> 55.8, 4096 x 16384 69.6 -> 60.3; 512 rows 12288 x 4096 100.6 -> 61.4, 7168 x 7168 105 -> 62; 2048 rows 12288 x
// 4096 247 -> 195.
#include "fg_common.h"
#include "fg_async_lds.h"

namespace fg {

namespace {

constexpr int kTS = 64;   // contraction elements per step

struct TileArgs {
  const half_t* w;
  const half_t* x;
  int64_t ldx;
  int M, N, K;
  int m_blocks, n_tiles, splits, ksteps;
  const half_t* bias;
  const half_t* residual;
  int64_t ldr;
  int relu;
  half_t* out16;
  float* out32;
  int64_t ldo;
  float* partial;       // [tile][split][(m, ct)][256 threads] float4
};

// Bias, residual and FP32 results may lie at any address that their type allows, and which kernel takes a call must not depend
// on it (kernels add in different orders): pieces of 16 bytes without an alignment.  512 rows, 7168 x 7168, bias and residual on
// a 16-byte boundary 55.1 us, one element off it 56.9 (99.6 on the kernel that took such calls otherwise).
typedef half_t h8_any_t __attribute__((ext_vector_type(8), aligned(2)));
typedef float f4_any_t __attribute__((ext_vector_type(4), aligned(4)));

// Opaque to the compiler: others may read the result only behind mfma_drain().
__device__ __forceinline__ void mfma_inplace(f4_t& acc, const h8_t& a, const h8_t& b) {
  __asm__ volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_drain() { __asm__ volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory"); }

template <int MT, int NT>
struct TileCfg {
  static constexpr int kBM = 2 * MT * 16, kBN = 2 * NT * 16;
  static constexpr int kAStage = kBM * kTS * 2, kStage = (kBM + kBN) * kTS * 2;
  static constexpr int kST = 160 * 1024 / kStage > 5 ? 5 : 160 * 1024 / kStage;
  static constexpr int kLds = kST * kStage;
  static constexpr int kAC = kBM / 32, kWC = kBN / 32, kCopies = kAC + kWC;   // 8-row pieces per copying wave and step
  static_assert(kST >= 3, "the step at hand, the next one and one on its way");
  static_assert(4 * MT * 16 * (NT * 16 + 4) * 4 <= kLds, "the sums go through LDS");
};

template <int MT, int NT>
__global__ __launch_bounds__(512) void gemm_f16_tiles_kernel(TileArgs a) {
  using C = TileCfg<MT, NT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = (wave >> 1) & 1;   // of the waves that compute
  const int l16 = lane & 15, g4 = lane >> 4;
  const int total = a.m_blocks * a.n_tiles * a.splits, per_xcd = (total + 7) >> 3;
  const int p = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || p >= total) return;
  // item p: row block (fastest, so that neighbours on an XCD share the weights), range of the contraction, column tile
  const int q = p / a.m_blocks, mblk = p - q * a.m_blocks, n_tile = q / a.splits, split = q - n_tile * a.splits;
  const int m0 = mblk * C::kBM, n0 = n_tile * C::kBN;
  const int ks0 = a.ksteps * split / a.splits, ks1 = a.ksteps * (split + 1) / a.splits;

  // ---- waves 4..7 bring the operands in
  if (wave >= 4) {
    const int pw = wave - 4;
    // a scalar base that moves on with the step, and one 32-bit offset per lane and piece: no vector instructions in the loop
    uint32_t a_src[C::kAC], w_src[C::kWC];
#pragma unroll
    for (int i = 0; i < C::kAC; ++i) {
      const int prow = 8 * (pw + 4 * i) + (lane >> 3);
      const int row = m0 + prow < a.M ? prow : a.M - 1 - m0;
      a_src[i] = ((uint32_t)row * (uint32_t)a.ldx + swz(prow, lane & 7) * 8) * 2;
    }
#pragma unroll
    for (int i = 0; i < C::kWC; ++i) {
      const int prow = 8 * (pw + 4 * i) + (lane >> 3);
      const int col = n0 + prow < a.N ? prow : a.N - 1 - n0;   // ragged last column block: load valid data, never store it
      w_src[i] = ((uint32_t)col * (uint32_t)a.K + swz(prow, lane & 7) * 8) * 2;
    }
    const char* a_base = reinterpret_cast<const char*>(a.x + (int64_t)m0 * a.ldx);
    const char* w_base = reinterpret_cast<const char*>(a.w + (int64_t)n0 * a.K);
    auto copy_one = [&](int c, int ks, int stage) {
      const int64_t kc = (int64_t)(ks < ks1 ? ks : ks1 - 1) * (kTS * 2);   // past the end: the last step again, which nobody reads
      unsigned char* st = smem + stage * C::kStage;
      if (c < C::kAC)
        __builtin_amdgcn_global_load_lds((gptr_t)(a_base + kc + a_src[c]), (lptr_t)(st + (pw + 4 * c) * 1024), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((gptr_t)(w_base + kc + w_src[c - C::kAC]), (lptr_t)(st + C::kAStage + (pw + 4 * (c - C::kAC)) * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < C::kST; ++t)
#pragma unroll
      for (int c = 0; c < C::kCopies; ++c) copy_one(c, ks0 + t, t);
    __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"((C::kST - 1) * C::kCopies) : "memory");
    __builtin_amdgcn_s_barrier();
    int stage = 0;
    for (int ks = ks0; ks < ks1; ++ks) {
      __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"((C::kST - 2) * C::kCopies) : "memory");
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int c = 0; c < C::kCopies; ++c) copy_one(c, ks + C::kST, stage);
      stage = stage + 1 == C::kST ? 0 : stage + 1;
    }
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may still target LDS behind the last barrier
    __builtin_amdgcn_s_barrier();
    return;
  }
  f4_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) acc[m][ct] = (f4_t){0.f, 0.f, 0.f, 0.f};

  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
  uint32_t a_off[2], w_off[2];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    const uint32_t o = (l16 * kTS + swz(l16, 4 * sl + g4) * 8) * 2;
    a_off[sl] = lds0 + wm * (MT * 16 * kTS * 2) + o;
    w_off[sl] = lds0 + C::kAStage + wn * (NT * 16 * kTS * 2) + o;
  }
  h8_t aop[2][MT], wop[2][NT];
  auto read = [&](uint32_t st, int sl, int buf) __attribute__((always_inline)) {
    static_for<0, NT>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      wop[buf][i] = __builtin_bit_cast(h8_t, lds_read128<i * 16 * kTS * 2>(st + w_off[sl]));
    });
    static_for<0, MT>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value;
      aop[buf][i] = __builtin_bit_cast(h8_t, lds_read128<i * 16 * kTS * 2>(st + a_off[sl]));
    });
  };
  auto landed = [&](int buf) __attribute__((always_inline)) {
    lds_wait();
#pragma unroll
    for (int i = 0; i < NT; ++i) lds_landed(wop[buf][i]);
#pragma unroll
    for (int i = 0; i < MT; ++i) lds_landed(aop[buf][i]);
  };

  __builtin_amdgcn_s_barrier();
  read(0, 0, 0);
  landed(0);

  constexpr int kNM = MT * NT;
  int stage = 0;
  for (int ks = ks0; ks < ks1; ++ks) {
    const int stage1 = stage + 1 == C::kST ? 0 : stage + 1;
    // ---- slice 0, the operands of slice 1 on their way
    read(stage * C::kStage, 1, 1);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, kNM>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value, ct = i / MT, m = i - ct * MT;
      mfma_inplace(acc[m][ct], aop[0][m], wop[0][ct]);
    });
    __builtin_amdgcn_sched_barrier(0);
    landed(1);
    // step ks + 1 has landed for every wave, and nobody reads the stage of step ks any more
    __builtin_amdgcn_s_barrier();   // bare barrier: no fence, the copies in flight stay in flight
    __builtin_amdgcn_sched_barrier(0);
    // ---- slice 1, the operands of the next step's slice 0 on their way
    read(stage1 * C::kStage, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, kNM>([&](auto I) __attribute__((always_inline)) {
      constexpr int i = decltype(I)::value, ct = i / MT, m = i - ct * MT;
      mfma_inplace(acc[m][ct], aop[1][m], wop[1][ct]);
    });
    landed(0);
    stage = stage1;
  }
  __builtin_amdgcn_s_barrier();   // every copy has landed and every operand been read

  mfma_drain();
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) __asm__ volatile("" : "+v"(acc[m][ct]));
  // lane: column l16 of each 16 x 16 tile, rows 4 g4 + 0..3
  if (a.splits > 1) {
    float4* dst = reinterpret_cast<float4*>(a.partial) + (int64_t)p * (kNM * 256) + tid;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct)
        if (m0 + wm * (MT * 16) + 16 * m < a.M)   // (a row tile of padding is never read back)
          dst[(m * NT + ct) * 256] = make_float4(acc[m][ct][0], acc[m][ct][1], acc[m][ct][2], acc[m][ct][3]);
    return;
  }
  // The sums go through LDS, each wave's through a part of its own: a lane finishes eight adjacent columns of a row
  constexpr int kCols = NT * 16, kLdsRow = kCols + 4, kPiece = kCols / 8;   // (row stride: the four rows of a store on banks of their own)
  constexpr int kItems = MT * 16 * kPiece / 64;
  float* sums = reinterpret_cast<float*>(smem) + wave * (MT * 16 * kLdsRow);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) sums[(16 * m + 4 * g4 + r) * kLdsRow + 16 * ct + l16] = acc[m][ct][r];
  wave_lds_fence();
  const int r0 = m0 + wm * (MT * 16), c0 = n0 + wn * kCols;
  h8_t res[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int e = i * 64 + lane, rr = e / kPiece, cc = (e - rr * kPiece) * 8;
    const int row = r0 + rr < a.M ? r0 + rr : a.M - 1, col = c0 + cc < a.N ? c0 + cc : a.N - 8;
    if (a.residual) res[i] = *reinterpret_cast<const h8_any_t*>(a.residual + (int64_t)row * a.ldr + col);
  }
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int e = i * 64 + lane, rr = e / kPiece, cc = (e - rr * kPiece) * 8;
    const int row = r0 + rr, col = c0 + cc;
    if (row >= a.M || col >= a.N) continue;
    float v[8];
    *reinterpret_cast<float4*>(v) = *reinterpret_cast<const float4*>(sums + rr * kLdsRow + cc);
    *reinterpret_cast<float4*>(v + 4) = *reinterpret_cast<const float4*>(sums + rr * kLdsRow + cc + 4);
    if (a.bias) {
      const h8_t b = *reinterpret_cast<const h8_any_t*>(a.bias + col);
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] += (float)b[q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (a.relu) v[q] = fmaxf(v[q], 0.f);
      if (a.residual) v[q] += (float)res[i][q];
    }
    if (a.out32) {
      float* o = a.out32 + (int64_t)row * a.ldo + col;
      *reinterpret_cast<f4_any_t*>(o) = (f4_any_t){v[0], v[1], v[2], v[3]};
      *reinterpret_cast<f4_any_t*>(o + 4) = (f4_any_t){v[4], v[5], v[6], v[7]};
    } else {
      h8_t o;
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = (half_t)v[q];
      *reinterpret_cast<h8_any_t*>(a.out16 + (int64_t)row * a.ldo + col) = o;
    }
  }
}

// The ranges' sums, added in ascending order.  blockIdx.x: tile (row block fastest), blockIdx.y: (row tile, column tile) of
// every wave.  Bias and residual are on their way with the sums.
__global__ __launch_bounds__(256) void gemm_f16_tiles_finish_kernel(TileArgs a, int mt, int nt) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave & 1, wn = wave >> 1;
  const int n_tile = blockIdx.x / a.m_blocks, mblk = blockIdx.x - n_tile * a.m_blocks;
  const int m = blockIdx.y / nt, ct = blockIdx.y - m * nt;
  const int row0 = 16 * ((2 * mblk + wm) * mt + m) + 4 * (lane >> 4);
  const int col = 16 * ((2 * n_tile + wn) * nt + ct) + (lane & 15);
  if (row0 >= a.M || col >= a.N) return;
  FinishRows fin;
  fin.request(a.bias, a.residual, a.ldr, row0, a.M, col);
  const float4* src = reinterpret_cast<const float4*>(a.partial) +
                      ((int64_t)n_tile * a.splits * a.m_blocks + mblk) * (mt * nt * 256) + blockIdx.y * 256 + tid;
  const int64_t step = (int64_t)a.m_blocks * (mt * nt * 256);
  float o[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < a.splits; s += 4) {
    float4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = s + i < a.splits ? src[(s + i) * step] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (s + i < a.splits) {
        o[0] += v[i].x;
        o[1] += v[i].y;
        o[2] += v[i].z;
        o[3] += v[i].w;
      }
  }
  fin.store(make_float4(o[0], o[1], o[2], o[3]), a.relu, a.residual, a.out16, a.out32, a.ldo, row0, a.M, col);
}

template <int MT, int NT>
int launch_tiles(const TileArgs& a, hipStream_t stream) {
  using C = TileCfg<MT, NT>;
  static bool attr_done = false;
  if (!attr_done) {
    FG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f16_tiles_kernel<MT, NT>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds));
    attr_done = true;
  }
  const int64_t items = (int64_t)a.m_blocks * a.n_tiles * a.splits;
  hipLaunchKernelGGL((gemm_f16_tiles_kernel<MT, NT>), dim3((unsigned)(ceil_div(items, 8) * 8)), dim3(512), C::kLds, stream, a);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

// What a tile shape takes, us: first + rounds of 256 workgroups x (round + steps x step), and with the contraction in ranges 4 +
// 0.17 per MB of partial sums written and read.  Fitted to 64 to 160 measured (rows, columns, contraction) each, from 33 to 4096
// rows and 768 to 50272 columns; a prediction is off by 13 % (one standard deviation), the choice between shapes by 6 %.
struct TileShape {
  int mt, nt;
  float first, round, step;
};
constexpr TileShape kShapes[] = {
    {1, 2, 0.6f, 1.31f, 0.196f},  {2, 2, -0.3f, 1.99f, 0.258f}, {2, 3, -1.4f, 3.19f, 0.390f},  {2, 4, -1.2f, 4.34f, 0.469f},
    {3, 2, -1.0f, 3.84f, 0.282f}, {4, 2, -0.6f, 3.68f, 0.397f}, {4, 3, 2.1f, 5.90f, 0.478f},   {4, 4, -5.5f, 10.14f, 0.511f},
    {6, 3, -4.7f, 10.59f, 0.528f}, {6, 4, -3.6f, 10.84f, 0.650f}, {8, 4, -5.0f, 14.04f, 0.794f},
};

}  // namespace

F16TilePick gemm_f16_tiles_pick(int64_t n, int64_t k, int64_t m, size_t ws_bytes) {
  F16TilePick best = {0, 0, 1, 0, 0.f};
  const int n32 = (int)n, m32 = (int)m, steps = (int)(k / kTS);
  for (int i = 0; i < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++i) {
    const TileShape& s = kShapes[i];
    const int bm = 32 * s.mt, bn = 32 * s.nt;
    const int64_t tiles = (int64_t)((m32 + bm - 1) / bm) * ((n32 + bn - 1) / bn);
    for (int sp = 1; sp <= 8 && (sp == 1 || steps >= 8 * sp); sp *= 2) {
      const int64_t bytes = sp == 1 ? 0 : tiles * sp * bm * bn * 4;
      if (bytes > (int64_t)ws_bytes) break;
      const float t = s.first + (float)((tiles * sp + 255) >> 8) * (s.round + (float)((steps + sp - 1) / sp) * s.step) +
                      (sp == 1 ? 0.f : 4.f + (float)bytes * 0.33e-6f);
      if (!best.mt || t < best.us) best = {s.mt, s.nt, sp, tiles * sp, t};
      if (tiles * sp >= 512) break;   // the chip is full: more ranges only add partial sums
    }
  }
  return best;
}

// Which calls this kernel takes, by measurement against the kernels that otherwise run (their time over this one's):
//   33 to 128 rows: matrices of 4 to 230 M elements (71 x 8064 x 2048 1.92, 35 x 7168 x 7168 1.31, 128 x 4096 x 4096 1.36,
//   100 x 21504 x 7168 1.25, 46 x 12288 x 44160 1.07, but 56 x 768 x 768 0.95, 48 x 2048 x 2048 0.82, 49 x 36864 x 12288 0.96).
//   LM heads from 97 rows, up to 380 M (126 x 50272 x 7168 1.05, 123 x 50272 x 4096 1.09, but 40 rows 0.96, 107 x 50272 x
//   22592 0.89).
//   129 to 2048 rows: up to 210 M (1.2 to 3.4 over 130 shapes; 7168 x 28672 1.07 to 1.54, 300 x 36864 x 12288 0.98, 512 rows
//   0.92); LM heads up to 512 rows (1330 x 50272 x 2048 0.93).
//   More rows: where tiles of 256 x 256 are less than one round of the chip and the contraction is not long (9000 x 768 x 3072
//   1.52, 6000 x 2048 x 2048 1.36, 18432 x 768 x 768 1.53, 3000 x 4096 x 4096 1.36, but 4096 x 4096 x 4096 0.94, 9000 x 2048 x 2048
//   0.90, 6000 x 2048 x 8192 0.98).
// Not within these lines (measured over 2500 shapes, this kernel's time over the other's):
//   65 to 96 rows, contractions beyond 8192 of matrices of more than 58 M, where tiles of up to 96 x 64 leave a quarter of the
//   chip and more without work, larger ones a third (the copies of those that there are don't take what HBM gives): 92 x 8352
//   x 13312 1.30, 70 x 8576 x 23744 1.23, 82 x 4256 x 17536 1.21, 80 x 12288 x 12288 1.05, but 89 x 6016 x 9408 (57 M) 0.90,
//   80 x 4096 x 10560 0.85, 85 x 7168 x 16768 0.94, 89 x 5760 x 20928 (128 x 128) 0.80; or where ranges of the small ones make
//   several rounds: 80 x 12288 x 16384 1.06, and beyond 20000 wherever the narrow tiles don't take the call: 72 x 5504 x 28928
//   1.13, 94 x 8128 x 22336 1.03, but 69 x 4864 x 28480 0.85.  97 to 128 rows, matrices of more than 80 M, where nearly half
//   of the chip has no work: 97 x 4256 x 24320 1.22, 108 x 8576 x 10176 1.07.
//   Contractions of up to 256 in more than one round, without a residual: a workgroup is its start and its epilogue, and the other
//   kernel's stay on: 1089 x 27488 x 64 2.05, 343 x 36896 x 192 1.32, 800 x 15328 x 128 1.08, 1247 x 8640 x 64 0.97.
//   Sizes that fill whole rounds of the other kernel, 256 tiles each, without a residual: of 256 x 256 1000 x 16384 x 320 1.29, x 1024
//   1.15, x 4096 1.05, x 7168 1.02, 2000 x 8192 x 768 1.22, 500 x 32768 x 2048 1.08; of 160 x 256 320 x 32768 x 1024 1.10, 160 x 65536 x
//   2048 1.06; but 2048 x 7936 x 4096 0.75, 256 x 32768 x 1024 (tiles of 128 rows) 0.87.
//   Matrices of more than 70 M in three rounds and more: 383 x 33408 x 2496 1.21, 1491 x 12416 x 13248 1.09, 231 x 41120 x 2816 1.05,
//   1260 x 27200 x 4864 1.04.  From 321 rows by what both are expected to take: kept 0.90 (29 shapes), left to the other 1.00 (81);
//   below, with a residual 0.68 to 0.84.  (In one or two rounds 0.70 to 0.82.)
bool gemm_f16_tiles_takes(int dtype, int64_t n, int64_t k, int64_t m, bool residual) {
  if (dtype != FG_F16 || n % 32 != 0 || m <= 32) return false;
  const int64_t size = n * k;
  const bool head = n > 32768;
  if (m <= 128) {
    if (head ? m <= 96 || size > 380000000 : size < 4000000 || size > 230000000) return false;
  } else if (m <= 2048) {
    if (size > 210000000 || (head && m > 512)) return false;
  } else if (k > 4096 || ceil_div(m, 256) * ceil_div(n, 256) > 224) {
    return false;
  }
  if (m > 128 && !residual && gemm_stream_f16_whole_rounds(n, k, m)) return false;
  const bool short_k = m > 320 && k <= 256 && !residual, long_k = m > 64 && m <= 128 && k > 8192;
  if (!short_k && !long_k && size <= 70000000) return true;
  const F16TilePick pick = gemm_f16_tiles_pick(n, k, m, linear_workspace_bytes(dtype, n, k, m));
  const int64_t rounds = ceil_div(pick.items, 256);
  const float fill = (float)pick.items / (float)(rounds * 256);
  if (short_k && rounds >= 2) return false;
  if (m > 64 && m <= 96 && k > 8192 && size > 58000000) {
    const bool small = pick.mt * pick.nt <= 6;   // up to 96 x 64
    if (fill <= (small ? 0.75f : 0.65f)) return false;
    if (small && (k > 20000 ? !gemm_f16w_pick_cols(n, k, m) : pick.splits > 1 && rounds > 1)) return false;
  }
  if (m > 96 && m <= 128 && k > 8192 && size > 80000000 && fill < 0.55f) return false;
  if (m > 128 && rounds >= 3 && size > 70000000) return m <= 320 ? residual : pick.us < 0.94f * gemm_stream_f16_us(n, k, m);
  return true;
}

int gemm_f16_tiles_launch(const LinearArgs& la, void* ws, size_t ws_bytes, hipStream_t stream) {
  const F16TilePick s = gemm_f16_tiles_pick(la.n, la.k, la.m, ws_bytes);
  TileArgs a;
  a.w = reinterpret_cast<const half_t*>(la.w_data);
  a.x = la.x;
  a.ldx = la.ldx;
  a.M = (int)la.m;
  a.N = (int)la.n;
  a.K = (int)la.k;
  a.m_blocks = (int)ceil_div(la.m, 32 * s.mt);
  a.n_tiles = (int)ceil_div(la.n, 32 * s.nt);
  a.splits = s.splits;
  a.ksteps = (int)(la.k / kTS);
  a.bias = la.bias;
  a.residual = la.residual;
  a.ldr = la.ldr;
  a.relu = la.relu;
  a.out16 = la.out_f16;
  a.out32 = la.out_f32;
  a.ldo = la.ldo;
  a.partial = reinterpret_cast<float*>(ws);
  ProfScope prof(la.m > 320 ? FG_K_GEMM_LARGE_M : FG_K_GEMM_SMALL_M, stream);
  int rc = FG_ERR_UNSUPPORTED;
  switch (s.mt * 10 + s.nt) {
    case 12: rc = launch_tiles<1, 2>(a, stream); break;
    case 22: rc = launch_tiles<2, 2>(a, stream); break;
    case 23: rc = launch_tiles<2, 3>(a, stream); break;
    case 24: rc = launch_tiles<2, 4>(a, stream); break;
    case 32: rc = launch_tiles<3, 2>(a, stream); break;
    case 42: rc = launch_tiles<4, 2>(a, stream); break;
    case 43: rc = launch_tiles<4, 3>(a, stream); break;
    case 44: rc = launch_tiles<4, 4>(a, stream); break;
    case 63: rc = launch_tiles<6, 3>(a, stream); break;
    case 64: rc = launch_tiles<6, 4>(a, stream); break;
    case 84: rc = launch_tiles<8, 4>(a, stream); break;
  }
  if (rc || a.splits == 1) return rc;
  hipLaunchKernelGGL(gemm_f16_tiles_finish_kernel, dim3((unsigned)(a.m_blocks * a.n_tiles), (unsigned)(s.mt * s.nt)), dim3(256), 0, stream,
                     a, s.mt, s.nt);
  FG_LAUNCH_CHECK();
  return FG_OK;
}

}  // namespace fg
