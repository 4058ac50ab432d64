// Shared device helpers for the gfx950 kernels (wave64, CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace covspec {

typedef unsigned short bf16_t;  // raw bf16 bits
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;

// Fragment order of a 16 x 16 fp64 tile: lane l of a wave (i = l % 16, q = l / 16) owns the elements (row i, column 4v + q),
// v = 0..3, which is what an operand of v_mfma_f64_16x16x4_f64 wants of it in four steps, and (with rows and columns
// swapped) what a product leaves in it.  The four go out as two 16-byte pieces, each a contiguous kilobyte of the wave.
// Row-major tiles cost a wave 64 cache lines per 16-byte load, one per lane (consecutive lanes are consecutive rows).
typedef double f64x2_t __attribute__((ext_vector_type(2)));
constexpr int kFragTile = 256;
__device__ __forceinline__ int frag_at(int i, int k) { return ((k >> 3) * 64 + (k & 3) * 16 + i) * 2 + ((k >> 2) & 1); }
__device__ __forceinline__ f64x4_t frag_load(const double* tile, int lane) {
  const f64x2_t a = *(const f64x2_t*)(tile + 2 * lane), b = *(const f64x2_t*)(tile + 128 + 2 * lane);
  return (f64x4_t){a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void frag_store(double* tile, int lane, const f64x4_t& v) {
  *(f64x2_t*)(tile + 2 * lane) = (f64x2_t){v[0], v[1]};
  *(f64x2_t*)(tile + 128 + 2 * lane) = (f64x2_t){v[2], v[3]};
}

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ float bf16lo_to_f32(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t packed) { return __uint_as_float(packed & 0xFFFF0000u); }

// float -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ bf16_t f32_to_bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { T w = __shfl_xor(v, o, 64); v = w > v ? w : v; }
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { T w = __shfl_xor(v, o, 64); v = w < v ? w : v; }
  return v;
}

// fp32 -> uint32 key whose unsigned order equals the float order (-0 is folded onto +0).
__device__ __forceinline__ uint32_t float_order_key(float f) {
  uint32_t u = __float_as_uint(f + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix sum of one int per thread over a 1024-thread block (blocked order = thread order).
// `wsum` is 17 ints of LDS; the block total is returned in *total.  Contains barriers: call uniformly.
__device__ __forceinline__ int block_exscan_1024(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int k = 0; k < 16; ++k) { int t = wsum[k]; wsum[k] = run; run += t; }
    wsum[16] = run;
  }
  __syncthreads();
  *total = wsum[16];
  return wsum[w] + inc - v;
}

// value of `v` in lane k of every row of 16 lanes, in one move
template <int k>
__device__ __forceinline__ double row_lane(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + k, 0xf, 0xf, true);   // row_newbcast:k
}

// Scalar from lane l of v.
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
// 1 / p: an estimate good to 2^-24, r (1 + e + e^2).
__device__ __forceinline__ double reciprocal(double p) {
  const double r = __builtin_amdgcn_rcp(p), e = fma(-p, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Barrier in global memory over the workgroups that work on one image.  `arrived` only grows; `target` is the
// value it reaches when all of them have arrived at this barrier.  Every thread's earlier global writes are
// visible to every thread of the group behind the barrier (device-scope release before, acquire after: the
// XCDs' L2s are not coherent with one another).  The wait is bounded: when it exceeds `limit_ticks` of the
// 100 MHz wall clock, or another workgroup of the image has reported that, `failed` is set and false is
// returned; the caller then gives up on the image.  Call uniformly from all threads; `s_flag` is one int of LDS.
struct ImageBarrier {
  unsigned int arrived;
  int failed;
};
// Device-scope store: written through the XCD's L2.
__device__ __forceinline__ void store_through(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

constexpr long long kBarrierLimitTicks = 200000000LL;   // 2 s, the default of `limit_ticks`

// ---- Handing on without a meeting: a word is at kAbsent before its element is stored, and readers load past the L2s, which are not coherent,
// until it is another one.  kAbsent is the upper word of a signalling NaN, which arithmetic does not return.  Saves the acknowledgement of
// the stores and a flag's way in front of the load.
constexpr int kLoadAgent = 16;                          // buffer loads: sc1, past the L2
constexpr int kAbsent = 0x7FF4ADED;
__device__ __forceinline__ double absent() { return __hiloint2double(kAbsent, 0); }
__device__ __forceinline__ bool is_absent(double v) { return __double2hiint(v) == kAbsent; }
// What to store of an element.
__device__ __forceinline__ double present(double v) { return is_absent(v) ? __hiloint2double(0x7FF80000, 0) : v; }
// N tiles in fragment order, tile n at off[n] bytes of `src` (a lane's offset included), as soon as all their elements are there.
// False: over the limit, or *failed is set; the elements are then whatever there was.  One wave.
template <int N>
__device__ __forceinline__ bool fetch_present(__amdgpu_buffer_rsrc_t src, const int (&off)[N], f64x2_t (&out)[N][2], const int* failed, long long limit_ticks) {
  unsigned todo = (1u << N) - 1;
  long long t0 = 0;
  for (int tries = 0; todo != 0; ++tries) {
    asm volatile("" ::: "memory");                      // loads anew
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (todo >> n & 1) {
#pragma unroll
        for (int h = 0; h < 2; ++h) out[n][h] = __builtin_bit_cast(f64x2_t, __builtin_amdgcn_raw_buffer_load_b128(src, off[n] + 1024 * h, 0, kLoadAgent));
      }
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (todo >> n & 1) {
        const f64x2_t u = out[n][0], v = out[n][1];
        if (!__any(is_absent(u[0]) || is_absent(u[1]) || is_absent(v[0]) || is_absent(v[1]))) todo &= ~(1u << n);
      }
    if (todo != 0 && (tries & 63) == 63) {              // 64 tries: some 60 us
      if (tries == 63) t0 = wall_clock64();
      if (__hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > limit_ticks) return false;
    }
  }
  return true;
}

// WRITE_BACK = false: everything the workgroup hands on went out in store_through() and is at the coherence point once
// the stores are acknowledged, so the caches need no write-back.
template <bool WRITE_BACK = true>
__device__ __forceinline__ bool image_barrier_wait(ImageBarrier* bar, unsigned int target, int* s_flag, long long limit_ticks) {
  // Every wave first waits until its own stores have been acknowledged by the L2 (vmcnt counts loads and
  // stores on this architecture); the cache maintenance itself acts on the CU's L1 and the XCD's L2, not on a
  // wave, so one thread issues it for the workgroup: write-back before the arrival, invalidate after the wait.
  __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
  __syncthreads();
  if (threadIdx.x == 0) {
    int ok = 1;
    // one write-back, then relaxed polling, then one invalidate: an acquire per poll would invalidate the caches
    // under the workgroups that are still at work, a release on the counter would write them back a second time
    if (WRITE_BACK) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(&bar->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t0 = wall_clock64();
    while (__hip_atomic_load(&bar->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(&bar->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
          wall_clock64() - t0 > limit_ticks) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    if (!ok) __hip_atomic_store(&bar->failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *s_flag = ok;
  }
  __syncthreads();
  return *s_flag != 0;
}

}  // namespace covspec
