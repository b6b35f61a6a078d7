// Device helpers shared by the HIP kernels of libsem.so.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sem {

// bfloat16 stored as uint16_t: the upper half of an IEEE float
__device__ __host__ inline float bf16_to_f32(uint16_t h) {
  union {
    uint32_t u;
    float f;
  } c;
  c.u = (uint32_t)h << 16;
  return c.f;
}
// round to nearest even (finite inputs)
__device__ __host__ inline uint16_t f32_to_bf16(float f) {
  union {
    uint32_t u;
    float f;
  } c;
  c.f = f;
  uint32_t u = c.u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <class TS, class TC> struct Cvt;
template <> struct Cvt<double, double> {
  __device__ static double ld(double v) { return v; }
};
template <> struct Cvt<float, float> {
  __device__ static float ld(float v) { return v; }
};
template <> struct Cvt<uint16_t, float> {
  __device__ static float ld(uint16_t v) { return bf16_to_f32(v); }
};
template <> struct Cvt<float, double> {
  __device__ static double ld(float v) { return (double)v; }
};
template <> struct Cvt<double, float> {
  __device__ static float ld(double v) { return (float)v; }
};

// Global-memory pointer.  A pointer read from device memory (a work item's
// or a solve's descriptor) has no known address space, and loads and stores
// through it compile to FLAT instructions, which wait on both memory
// counters and keep fewer loads in flight; kernels whose buffers are global
// memory (all device buffers here) access them through gp pointers.
template <class T> using gp = T __attribute__((address_space(1))) *;

// Memory that no kernel writes while this one runs.  Uniform loads through it
// go through the scalar cache also where the pointer itself was loaded from a
// descriptor: through gp the compiler cannot know that the kernel's own stores
// leave them alone and makes them vector loads.
template <class T> using cp = const T __attribute__((address_space(4))) *;

// orders a wave's LDS writes before its later LDS reads of other lanes'
// entries: the lanes of a wave execute together and a wave's LDS
// operations complete in issue order, so only the compiler has to be kept
// from moving accesses across this point (for LDS regions that one wave
// owns; a workgroup barrier would also wait for the other waves)
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a double moved across the lanes of a wave by a DPP pattern (both halves)
template <int CTRL> __device__ inline double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// v plus its value in the other half of the wave (S = 32) or in the
// neighbouring row of 16 lanes (S = 16): a swap of v's halves (rows) with
// those of a copy of v leaves one operand of the sum in each copy
template <int S> __device__ inline double swap_add_f64(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  auto l = S == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                   : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto h = S == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                   : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return __longlong_as_double(((long long)h[0] << 32) | l[0]) +
         __longlong_as_double(((long long)h[1] << 32) | l[1]);
}

// wave64 sum in a fixed order, the same in every lane: the butterfly over
// lane distances 32, 16, 8, 4, 2, 1, in registers.  The rotations by 8 and 4
// within a row reach the lanes at these distances because the partial sums
// before them repeat with period 16 and 8.  (The same butterfly through
// ds_bpermute takes an LDS round trip per step.)
__device__ inline double wave_sum(double v) {
  v = swap_add_f64<32>(v);
  v = swap_add_f64<16>(v);
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  return v;
}

// block sum, deterministic for a fixed block size; result valid in thread 0
template <int THREADS>
__device__ inline double block_sum(double v, double *smem /* THREADS/64 */) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) smem[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < THREADS / 64; ++q) s += smem[q];
  }
  __syncthreads();
  return s;
}

}  // namespace sem
