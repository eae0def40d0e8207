// Helpers shared by the GEMM kernels that stage their operands in LDS with asynchronous global -> LDS
// copies (csrc/fg_gemm_stream.hip, csrc/fg_gemm_f16w.hip).
#pragma once
#include "fg_common.h"

namespace fg {
namespace {

// ---- work shared along K: `total` (tile, K step) units cut into `parts` equal contiguous ranges, parts <= total.
// first unit of range p (p >= parts: the end)
__device__ __forceinline__ int64_t work_begin(int64_t total, int parts, int p) { return p < parts ? (total * p) / parts : total; }
// the range of workgroup `block`: consecutive ranges on one XCD, all XCDs equally loaded; >= parts: none
__device__ __forceinline__ int part_of_block(int parts, int block) {
  const int per_xcd = (parts + 7) >> 3, i = block >> 3;
  return i < per_xcd ? (block & 7) * per_xcd + i : parts;
}
__device__ __forceinline__ int part_of_block(int parts) { return part_of_block(parts, (int)blockIdx.x); }
// ranges lo .. hi share tile t of `ksteps` units; the tile is the first segment of every one of them but perhaps of lo
struct TileParts {
  int lo, hi;
  bool lo_second;   // tile t is the second segment of range lo
};
__device__ __forceinline__ TileParts tile_parts(int64_t total, int parts, int ksteps, int64_t t) {
  // work_begin(p) <= w  <=>  p <= ((w + 1) * parts - 1) / total
  const int64_t w0 = t * ksteps, w1 = w0 + ksteps;
  TileParts r;
  if (total * parts < 0xffffffffll) {   // (a 64-bit division is some hundred instructions)
    r.lo = (int)((uint32_t)((w0 + 1) * parts - 1) / (uint32_t)total);
    r.hi = (int)((uint32_t)(w1 * parts - 1) / (uint32_t)total);
    r.lo_second = (uint32_t)total * (uint32_t)r.lo / (uint32_t)parts != (uint32_t)w0;
  } else {
    r.lo = (int)(((w0 + 1) * parts - 1) / total);
    r.hi = (int)((w1 * parts - 1) / total);
    r.lo_second = work_begin(total, parts, r.lo) != w0;
  }
  return r;
}
// host: ranges that `total` units are cut into on `grid` workgroups.  Fewer than three K steps are not worth a
// workgroup: its pipeline does not fill and its partial sums cost more than the steps.  Measured with the reduction pass,
// 768 x 3072 4-bit weights at 33 / 144 / 600 rows, at least 1 / 3 / 6 / 12 steps (us): 14.5 / 10.7 / 11.3 / 14.3,
// 23.5 / 16.8 / 17.2 / 21.2, 41.3 / 29.7 / 28.8 / 31.9 (and 49.6 / 56.5 / - with ranges of less than one step).
// A tile of up to five steps is one range, with no partial sums at all, if there are 32 of them or no more than three
// steps (fewer of four are halved): us with ranges of at least 1 / 2 / 3 steps, tiled, 8192 columns x 333 rows, K = 64
// 12.9 / 20.5 / 34.7, K = 128 24.4 / 14.1 / 28.4; with 2 / 3 / 4, K = 256, 16384 x 512 38 / 44 / 23, 768 x 144 (three
// tiles) 11.7 / 17.9 / 18.4; with 3 / 5, K = 320, 16384 x 512 47 / 24, 2048 x 300 (16 tiles) 18.1 / 21.5.
constexpr int kMinPartSteps = 3;
static inline int work_parts(int64_t total, int ksteps, int grid) {
  const bool whole = ksteps <= kMinPartSteps || (ksteps <= 5 && total / ksteps >= 32);
  const int64_t p = total / (whole ? ksteps : (ksteps == 4 ? 2 : kMinPartSteps));
  return p < 1 ? 1 : p < grid ? (int)p : grid;
}

// Sum, in ascending K order, of what ranges lo .. hi left of a tile: v[i] = float4 number `at + i * step` of each
// range's slot (2 slots of slot4 float4s per range).  The loads of eight ranges are in flight together, of four with two
// items.
template <int ITEMS>
__device__ __forceinline__ void sum_parts(const float4* partial, int64_t slot4, const TileParts& tp, int64_t at, int64_t step,
                                          float4 (&v)[ITEMS]) {
  constexpr int kFly = ITEMS > 1 ? 4 : 8;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p = tp.lo; p <= tp.hi; p += kFly) {
    float4 x[kFly][ITEMS];
#pragma unroll
    for (int c = 0; c < kFly; ++c) {
      const float4* src = partial + ((int64_t)(p + c) * 2 + (p + c == tp.lo && tp.lo_second ? 1 : 0)) * slot4 + at;
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) x[c][i] = p + c <= tp.hi ? src[i * step] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int c = 0; c < kFly; ++c)
      if (p + c <= tp.hi) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
          v[i].x += x[c][i].x;
          v[i].y += x[c][i].y;
          v[i].z += x[c][i].z;
          v[i].w += x[c][i].w;
        }
      }
  }
}
// The end of a reduction pass: rows row0 .. row0 + 3 of column `col`.  Bias and residual are requested before the partial
// sums, so that they arrive with them; read where they are added, row by row behind the store of the row before (which the
// compiler has to take for an alias), they are four more round trips to memory, one after the other.  A projection of tiled
// weights with a residual, both passes, us, so -> requested ahead: 12288 x 12288 at 80 rows 47.2 -> 46.4, 144 rows 66.3 ->
// 66.0, 512 rows 170.3 -> 164.7; 7168 x 7168 at 1000 rows 133.7 -> 128.8.
struct FinishRows {
  uint32_t bias, res[4];   // FP16 bits
  __device__ __forceinline__ void request(const half_t* b, const half_t* residual, int64_t ldr, int row0, int M, int col) {
    bias = b ? reinterpret_cast<const uint16_t*>(b)[col] : 0u;
    if (residual) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + r < M ? row0 + r : M - 1;
        res[r] = reinterpret_cast<const uint16_t*>(residual)[(int64_t)row * ldr + col];
      }
    }
  }
  __device__ __forceinline__ void store(const float4& sum, int relu, bool residual, half_t* out16, float* out32, int64_t ldo, int row0,
                                        int M, int col) {
    __asm__ volatile("" : "+v"(bias));   // (else converted, that is waited for, where it was requested)
#pragma unroll
    for (int r = 0; r < 4; ++r) __asm__ volatile("" : "+v"(res[r]));
    const float o[4] = {sum.x, sum.y, sum.z, sum.w};
    const float b = (float)__builtin_bit_cast(half_t, (uint16_t)bias);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + r;
      if (row >= M) break;
      float x = o[r] + b;
      if (relu) x = fmaxf(x, 0.f);
      if (residual) x += (float)__builtin_bit_cast(half_t, (uint16_t)res[r]);
      if (out32)
        out32[(int64_t)row * ldo + col] = x;
      else
        out16[(int64_t)row * ldo + col] = (half_t)x;
    }
  }
};
__device__ __forceinline__ int swz(int row, int kc) { return kc ^ ((row >> 1) & 7); }

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// The compiler orders every LDS read it can see behind ALL outstanding asynchronous global -> LDS
// copies (it cannot tell which copy an address belongs to), which would drain the prefetch queue on
// every step.  The stages are therefore read with hand-placed ds_read instructions; the explicit
// vmcnt wait plus the barrier at the top of each step are what make the data visible.
template <int OFF>
__device__ __forceinline__ u4_t lds_read128(uint32_t addr) {
  u4_t r;
  __asm__ volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
template <int OFF>
__device__ __forceinline__ float2 lds_read64(uint32_t addr) {
  float2 r;
  __asm__ volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
template <int OFF>
__device__ __forceinline__ uint32_t lds_read32(uint32_t addr) {
  uint32_t r;
  __asm__ volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// all ds_reads issued so far have landed
__device__ __forceinline__ void lds_wait() { __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// makes later uses of v depend on a point after the preceding lds_wait()
template <class T>
__device__ __forceinline__ void lds_landed(T& v) {
  __asm__ volatile("" : "+v"(v));
}
template <int I>
struct IdxC {
  static constexpr int value = I;
};
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(IdxC<B>{});
    static_for<B + 1, E>(f);
  }
}

}  // namespace
}  // namespace fg
