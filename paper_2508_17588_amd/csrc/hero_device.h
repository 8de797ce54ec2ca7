// Device-side helpers shared by the HERO kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;   // raw bf16 bits

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (bf16_t)((u >> 16) | 0x40);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// round-to-nearest-even through the hardware conversion (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ bf16_t f32_to_bf16_hw(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(bf16_t, b);
}

__device__ __forceinline__ uint32_t pack_bf16x2_hw(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float floatx2_t __attribute__((ext_vector_type(2)));
  floatx2_t v = {lo, hi};
  bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
  return __builtin_bit_cast(uint32_t, b);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

__device__ __forceinline__ float unpack_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float unpack_hi(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }

template <typename T> struct ResidIO;
template <> struct ResidIO<float> {
  static __device__ __forceinline__ void load8(const float* p, float* v) {
    floatx4_t a = *reinterpret_cast<const floatx4_t*>(p);
    floatx4_t b = *reinterpret_cast<const floatx4_t*>(p + 4);
    v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
    v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  }
  static __device__ __forceinline__ void store8(float* p, const float* v) {
    floatx4_t a = {v[0], v[1], v[2], v[3]};
    floatx4_t b = {v[4], v[5], v[6], v[7]};
    *reinterpret_cast<floatx4_t*>(p) = a;
    *reinterpret_cast<floatx4_t*>(p + 4) = b;
  }
};
template <> struct ResidIO<bf16_t> {
  static __device__ __forceinline__ void load8(const bf16_t* p, float* v) {
    u32x4_t a = *reinterpret_cast<const u32x4_t*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = unpack_lo(a[i]); v[2 * i + 1] = unpack_hi(a[i]); }
  }
  static __device__ __forceinline__ void store8(bf16_t* p, const float* v) {
    u32x4_t a;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<u32x4_t*>(p) = a;
  }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// buffer resource words: base address, no stride, byte count, raw 32-bit data format
__device__ __forceinline__ u32x4_t rsrc_words(const void* p, uint32_t bytes) {
  const uint64_t addr = (uint64_t)p;
  u32x4_t r = {(uint32_t)addr, (uint32_t)(addr >> 32) & 0xffffu, bytes, 0x00020000u};
  r[0] = __builtin_amdgcn_readfirstlane(r[0]); r[1] = __builtin_amdgcn_readfirstlane(r[1]);
  r[2] = __builtin_amdgcn_readfirstlane(r[2]); r[3] = __builtin_amdgcn_readfirstlane(r[3]);
  return r;
}

// 16 bytes per lane from a buffer straight into LDS at lds_addr + 16*lane; bytes past the end of the buffer arrive
// as zero.  The bounds check covers voffset only; soffset carries an advance that stays inside a row.  Issued by hand,
// because the compiler's own builtin makes every later LDS read wait for it: completion is awaited explicitly with
// vmcnt.  Nothing else in the kernels that use it uses m0.
__device__ __forceinline__ void lds_fill(u32x4_t rsrc, uint32_t lds_addr, uint32_t voffset, uint32_t soffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset) : "memory");
}
__device__ __forceinline__ void lds_fill(u32x4_t rsrc, uint32_t lds_addr, uint32_t voffset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds_addr), "v"(voffset), "s"(rsrc) : "memory");
}

__device__ __forceinline__ float gelu_tanh(float x) {
  // x/2 (1 + tanh u) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3);
  // -2u log2(e) = x (C1 + C2 x^2) with the constants folded: five plain operations and two
  // transcendentals per element (the epilogue runs while the matrix pipe idles)
  constexpr float C1 = -2.302208198144325f;     // -2 log2(e) sqrt(2/pi)
  constexpr float C2 = -0.1029432395800235f;    // C1 * 0.044715
  float e = __builtin_amdgcn_exp2f(x * __builtin_fmaf(x * x, C2, C1));
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

// Workgroups that share the sum of one output block: each stores its part, and the one that arrives last adds them up.
// Parts go past the XCDs' L2s both ways (sc1), and a workgroup's stores are complete before its arrival is counted, so
// the last one sees all of them; none waits for another.  The count is zero again for the next launch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t parts_rsrc(float* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00020000);
}
__device__ __forceinline__ void store_part(__amdgpu_buffer_rsrc_t rs, uint32_t offset, floatx4_t v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), rs, offset, 0, 16);
}
__device__ __forceinline__ floatx4_t load_part(__amdgpu_buffer_rsrc_t rs, uint32_t offset) {
  return __builtin_bit_cast(floatx4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, offset, 0, 16));
}
// called by all threads, after store_part; word: an LDS word nothing else uses meanwhile
__device__ __forceinline__ bool last_to_arrive(uint32_t* count, uint32_t n, uint32_t* word) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *word = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const bool last = __builtin_amdgcn_readfirstlane(*word) == n - 1;
  if (last && threadIdx.x == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return last;
}
