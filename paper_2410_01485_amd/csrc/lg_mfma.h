// lg_mfma.h — small device helpers shared by the bf16 MFMA kernels (gfx950).
//
// Matrix-core layout used throughout (v_mfma_f32_32x32x16_bf16, one wavefront):
//   lane = 32*g + n,  g in {0,1},  n in 0..31
//   A operand (32 x 16): lane holds row n,    contraction slots 8g .. 8g+7  (8 bf16)
//   B operand (16 x 32): lane holds column n, contraction slots 8g .. 8g+7  (8 bf16)
//   C/D (32 x 32, 16 floats): register r of a lane is row 8*(r/4) + 4g + (r%4), column n
// Both operands always take their 8 slots from the same 8 positions of the
// contracted index, so the product does not depend on how the hardware orders
// the slots internally.
#ifndef LG_MFMA_H_
#define LG_MFMA_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16_t lg_mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Row of register r (0..15) of a 32x32 accumulator for lane-half g.
__device__ __forceinline__ constexpr int lg_crow(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// Value held by lane ^ 32.
__device__ __forceinline__ float lg_other_half(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // one of the two results is this lane's own value, the other the partner's
  const unsigned own_xor = r[0] ^ r[1];
  return __builtin_bit_cast(float, own_xor ^ u);
}

// Round two floats to bf16 (nearest even) and pack them, low element first.
__device__ __forceinline__ uint32_t lg_pack_bf16(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}

// x where bit k of `bits` is set, otherwise `other`: the bit spread over a register and a bitwise operation (a compare and a
// select through a scalar mask are three instructions and a wait).
__device__ __forceinline__ float lg_keep_or(float x, uint32_t bits, int k, float other) {
  const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)bits, k, 1);
  return __uint_as_float((__float_as_uint(x) & keep) | (__float_as_uint(other) & ~keep));
}

// Values that one workgroup leaves for another of the same launch (partial results summed by whichever finishes
// last): device-scope accesses, which go through to memory the workgroups of all XCDs see, instead of device-wide
// fences, which write back and invalidate a whole L2 (in the float32 dk/dv kernel such a fence per wave cost 87 of
// 138 us).  Stores, lg_shared_stores_done(), a barrier, then a device-scope atomic announces them.
__device__ __forceinline__ void lg_store_shared2(float* p, float x, float y) {
  const unsigned long long w =
      __builtin_bit_cast(unsigned, x) | ((unsigned long long)__builtin_bit_cast(unsigned, y) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void lg_store_shared4(float* p, f32x4_t x) {
  lg_store_shared2(p, x[0], x[1]);
  lg_store_shared2(p + 2, x[2], x[3]);
}
__device__ __forceinline__ f32x2_t lg_load_shared2(const float* p) {
  const unsigned long long w = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
  return f32x2_t{__builtin_bit_cast(float, (unsigned)w), __builtin_bit_cast(float, (unsigned)(w >> 32))};
}
__device__ __forceinline__ void lg_store_shared1(float* p, float x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float lg_load_shared1(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4_t lg_load_shared4(const float* p) {
  const f32x2_t a = lg_load_shared2(p), b = lg_load_shared2(p + 2);
  return f32x4_t{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void lg_shared_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ bf16x8_t lg_as_bf16x8(uint4 x) { return __builtin_bit_cast(bf16x8_t, x); }

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <int... I, typename F>
__device__ __forceinline__ void lg_static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void lg_static_for(F&& f) {
  lg_static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// NU matrix instructions whose LDS operands are requested DIST of them ahead: begin(read) asks for the first ones, run
// calls use(u, operand) in order.  (The compiler on its own asks for an operand just before its use and waits.)
template <int NU, int DIST>
struct LgRing {
  bf16x8_t op[DIST + 1];
  template <typename R>
  __device__ __forceinline__ void begin(R&& read) {
    lg_static_for<DIST>([&](auto U) { op[decltype(U)::value] = read(decltype(U)::value); });
  }
  template <typename R, typename F>
  __device__ __forceinline__ void run(R&& read, F&& use) {
    lg_static_for<NU>([&](auto U) {
      constexpr int u = decltype(U)::value, w = u + DIST;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (w < NU) op[w % (DIST + 1)] = read(w);
      use(u, op[u % (DIST + 1)]);
    });
  }
};

#endif  // LG_MFMA_H_
