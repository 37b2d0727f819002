// Device helpers shared by the library's HIP sources (gfx950 only): vector
// types, 16-byte register loads and stores, the global -> LDS copy, explicit
// vector-memory counter waits, the bf16 MFMA and bf16 packing.  Internal
// header; the definitions live in namespace ssa_dev.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssa_dev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(void* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// D = A B + C on one 16x16 tile, K = 32 (v_mfma_f32_16x16x32_bf16).
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Two fp32 values to packed bf16, round to nearest even.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// One wave-wide global -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4):
// lane i's 16 bytes from g land at LDS address l + 16 i (l wave-uniform).  It
// is inline assembly, so the compiler's memory-counter tracking does not make
// reads of other LDS buffers wait for it; every reader of the destination
// waits explicitly (vm_wait, then the barrier that publishes the buffer).
// The copy reads M0, and on this architecture a scalar write of M0 and a
// global -> LDS load that reads it need one wait state between them.  The
// compiler inserts it for its own instructions but does not look inside inline
// assembly, so the s_nop is part of every copy (here and in ssa_gemm.hip).
// COHERENT: a device-scope read (sc1), for rows written in the same launch.
template <bool COHERENT = false>
__device__ __forceinline__ void dma16(const void* g, const char* l) {
  const uint32_t a = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)l;
  if (COHERENT)
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off sc1" ::"v"(g), "{m0}"(a) : "memory");
  else
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "{m0}"(a) : "memory");
}

// dma16 with the non-temporal hint (nt), for rows a workgroup reads once: they
// should not displace what the caches hold for other workgroups.
__device__ __forceinline__ void dma16_stream(const void* g, const char* l) {
  const uint32_t a = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)l;
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(g), "{m0}"(a) : "memory");
}

// s_waitcnt vmcnt(N): all but this wave's N most recent vector-memory
// operations (LDS copies included) have completed.
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void lds_dma_wait() { vm_wait<0>(); }

// Split partials that cross workgroups (and XCDs, whose L2s are not coherent with
// each other) are written through to the device coherence point: 16-byte buffer
// stores with the device-coherent cache policy (sc1), the instruction of a
// device-scope store.  A wave's store then covers whole lines; as two 8-byte
// device-scope atomics, each instruction wrote half of every 16 bytes.
// us with 8-byte and with 16-byte stores: 250 rows on 3001 cached (32/8 heads, key
// ranges in 4 pieces) 42.0 and 39.2; a Llama-3-8B layer of 640 tokens (split
// projections) 498.5 and 489; of 128 decodes 274.3 and 272.2.
// base is wave-uniform; offsets are bytes from it.
constexpr int kCachePolicySc1 = 16;
struct PartWriter {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ explicit PartWriter(float* base) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<float*>((uintptr_t)(((uint64_t)hi << 32) | lo)), (short)0, 0x7fffffff,
        0x00020000);
  }
  __device__ void operator()(int byte_off, u32x4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, byte_off, 0, kCachePolicySc1);
  }
};

}  // namespace ssa_dev
