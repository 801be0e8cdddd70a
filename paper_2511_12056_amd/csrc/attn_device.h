// Device-side vector types and wavefront helpers shared by the attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

namespace pda {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T) T __attribute__((address_space(3)))*
#define GLOBAL_PTR(T) T __attribute__((address_space(1)))*

// Lanes l and l^32 hold the two halves of one query's keys.  v_permlane32_swap hands every lane
// both halves' values (one in each result register), so max and sum need no select.
__device__ __forceinline__ float pair_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    f32x2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);     // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(unsigned, h);
}

// 16 bytes per lane from global memory (scalar base + per-lane byte offset) straight into LDS:
// lane l's data lands at lds_addr + 16*l (lds_addr wave-uniform, passed in M0).  Inline assembly
// on purpose: the compiler's wait-count insertion then does not see an LDS write that it cannot
// tell apart from the operand reads that follow (it would drain the whole prefetch before every
// LDS read); completion is tracked by hand with s_waitcnt vmcnt before the barrier.
// M0 is not restored; it is declared clobbered.
// The compiler does not see into the assembly, so the wait states it would insert are up to us: one
// between the write of M0 and the load, and five between a VALU write of the base registers (the
// v_readlane that restores a spilled pointer) and the load.  Copying the base through VCC is both: an
// instruction in between, and a scalar write, which the hardware interlocks.
__device__ __forceinline__ void lds_dma16(const void* sbase, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 vcc, %2\n\tglobal_load_lds_dwordx4 %1, vcc"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(sbase)
                 : "memory", "m0", "vcc");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// Row-dependent XOR applied to the index of a row's 16-byte granules in an LDS tile, chosen so that
// the operand reads are free of bank conflicts (64 banks of 4 bytes).  With 256-byte rows (d = 128)
// every row starts at bank 0: the K reads (16 rows, one granule each) need 16 different granules,
// the transposing V reads (4 rows, 4 granules each) 4 different groups of 4.  With 128-byte rows
// (d = 64) even and odd rows already lie in different halves of the banks, so the XOR is taken
// from the row index without its lowest bit.
template <int D>
__device__ __forceinline__ constexpr int swz_k(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int D>
__device__ __forceinline__ constexpr int swz_v(int row) { return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2); }

// Streaming (non-temporal) 16- and 8-byte accesses for data that is touched once: they leave the
// caches to data that is reused and measurably raise the rate of the HBM-bound kernels.
__device__ __forceinline__ float4 nt_load4(const float4* p) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void nt_store4(float4* p, const float4& a) {
    const f32x4 v = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}
__device__ __forceinline__ void nt_store2(uint2* p, unsigned lo, unsigned hi) {
    const u32x2 v = {lo, hi};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x2*>(p));
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [I0, N).
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

}  // namespace pda
