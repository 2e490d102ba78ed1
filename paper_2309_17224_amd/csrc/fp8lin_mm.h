// Device helpers shared by the matmul kernels of libfp8lin.so: the FP8 MFMA,
// LDS copies and waits, operand fragments, tile order, output stores and the
// in-launch amax / bias.  Internal, not part of the ABI.
#pragma once

#include "fp8lin_fp8.h"
#include "fp8lin_internal.h"

namespace fp8lin {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// MFMA operand format selectors: 0 = fp8 (E4M3), 1 = bf8 (E5M2).
template <int F0, int F1>
__device__ __forceinline__ v4f mfma16(v8i a, v8i b, v4f c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, F0, F1, 0, 0, 0, 0);
}

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
    return v;
}

// 32-bit LDS address of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// Wait until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Wait until every LDS read of this wave has returned its data.
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// Workgroup barrier with no memory fence: the main loop orders its LDS
// traffic itself (wait_vmcnt for the copies, wait_lgkmcnt0 for the reads).
__device__ __forceinline__ void ws_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// The two 16-byte pieces of an MFMA operand fragment, as one 8-register vector.
__device__ __forceinline__ v8i ld_frag(const uint8_t* p, int fo0, int fo1) {
    const uint4 p0 = *(const uint4*)(p + fo0);
    const uint4 p1 = *(const uint4*)(p + fo1);
    return v8i{(int)p0.x, (int)p0.y, (int)p0.z, (int)p0.w, (int)p1.x, (int)p1.y, (int)p1.z, (int)p1.w};
}

// Physical 16-byte chunk of logical chunk c in LDS operand row r is
// c ^ chunk_swz(r).  A fragment read has lane l on row r = l % 16 (row bit 0
// picks the half of a 256-byte bank line) and logical chunk 2 (l / 16) + piece.
// Within one phase (fixed lane bit 5 and parity of lane bits 2..4) the map
// (r1, r2, r3) -> (r1 ^ piece, parity ^ r3, bit 5 ^ r2) of the three chunk bits
// is one-to-one, so the 16 lanes hit 16 distinct bank groups.
__device__ __forceinline__ int chunk_swz(int r) { return ((r >> 1) & 1) | (((r >> 2) & 1) << 2); }

// Contiguous tile ranges per XCD, then grouped row-major order inside.
__device__ __forceinline__ void tile_of(int b, int nb, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int x = b & 7, l = b >> 3;
    const int per = nb >> 3, rem = nb & 7;
    const int t = x * per + min(x, rem) + l;
    constexpr int G = 8;
    const int group = G * tiles_n;
    const int gid = t / group;
    const int first = gid * G;
    const int gm = min(tiles_m - first, G);
    const int r = t - gid * group;
    tm = first + r % gm;
    tn = r / gm;
}

// 16-byte store with the non-temporal hint: outputs are not read again by the
// kernel and should not displace cached operands.
__device__ __forceinline__ void st_stream(void* p, uint4 v) {
    __builtin_nontemporal_store(u32x4_any{v.x, v.y, v.z, v.w}, (u32x4_any*)p);
}

// Store 4 consecutive outputs of row m starting at column n (unscaled by
// 2^-sh); returns the largest output magnitude pattern (as fp32 bits).
template <int OUT_DT>
__device__ __forceinline__ uint32_t store4(void* C, int64_t ldc, int64_t m, int64_t n, int64_t M,
                                           int64_t N, v4f acc, int sh) {
    float y[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) y[v] = ldexpf(acc[v], sh);
    uint32_t mx = 0;
    if (OUT_DT == FP8_DT_BF16) {
        uint32_t h[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            h[v] = f32_to_bf16_rne(y[v]);
            mx = max(mx, (h[v] & 0x7FFFu) << 16);
        }
        if (m < M) {
            uint16_t* p = (uint16_t*)C + m * ldc + n;
            if (n + 3 < N) {
                st8_any(p, h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            } else {
                for (int v = 0; v < 4; ++v)
                    if (n + v < N) p[v] = (uint16_t)h[v];
            }
        }
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) mx = max(mx, __float_as_uint(y[v]) & 0x7FFFFFFFu);
        if (m < M) {
            float* p = (float*)C + m * ldc + n;
            if (n + 3 < N) {
                st16_any(p, make_uint4(__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])));
            } else {
                for (int v = 0; v < 4; ++v)
                    if (n + v < N) p[v] = y[v];
            }
        }
    }
    return m < M ? mx : 0u;
}

// Unscale exponent of output row m (of M): -(ba + bb), with ba of row m when
// ba_rows (per-row activation biases, one per data sample or segment).
__device__ __forceinline__ int row_shift(const int32_t* ba_p, int ba_rows, int bb, int64_t m, int64_t M) {
    return -((ba_rows ? ba_p[min(m, M - 1)] : ba_p[0]) + bb);
}

// Direct L2 -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4, the
// form with a wave-uniform 64-bit base in SGPRs and a 32-bit lane offset):
// lane i's 16 bytes land at lds_row + 16 i; lds_row must be wave-uniform.
// The instruction is issued from inline assembly so that the compiler does
// not treat every later LDS read as dependent on it (it cannot tell the two
// halves of the double buffer apart and would wait for the prefetch before
// each read); completion is tracked with wait_vmcnt.
__device__ __forceinline__ void lds_dma16_s(const uint8_t* sbase, uint32_t voff, uint32_t lds_row) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_row), "v"(voff), "s"(sbase)
                 : "memory");
}

// The same copy with the non-temporal hint (a stream read once).
__device__ __forceinline__ void lds_dma16_nt(const uint8_t* sbase, uint32_t voff, uint32_t lds_row) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :
                 : "s"(lds_row), "v"(voff), "s"(sbase)
                 : "memory");
}

__device__ __forceinline__ int32_t bias_of_fmt(int fmt, uint32_t a, int32_t margin, uint32_t* fl) {
    switch (fmt) {
        case FP8_E4M3: return bias_of<FP8_E4M3>(a, margin, fl);
        case FP8_E5M2: return bias_of<FP8_E5M2>(a, margin, fl);
        case FP8_E4_A: return bias_of<FP8_E4_A>(a, margin, fl);
        default: return bias_of<FP8_E5_A>(a, margin, fl);
    }
}

// The share of one workgroup (called by one of its threads, once per
// workgroup of the launch) in the output's amax: bc, its largest |Y| as a
// canonical fp32 pattern, goes to *amax_out (zeroed beforehand) or, with
// bo.ws, into the running maximum of the launch, whose last workgroup writes
// amax, bias and flags.
__device__ __forceinline__ void fold_amax(uint32_t bc, uint32_t* amax_out, const BiasOut& bo) {
    if (!bo.ws) {
        atomicMax(amax_out, bc);
        return;
    }
    // The fold is a returning device-scope atomic whose result is consumed by
    // an asm statement that also clobbers memory: the compiler cannot move the
    // count above it, and the hardware has performed the fold (the wait for
    // its return) before the count is issued.  The workgroup that counts last
    // therefore finds every fold in ws[0].  A release/acquire count would say
    // the same in the language's terms, but at agent scope its release writes
    // back the XCD's L2 in every workgroup's epilogue (2-6 % slower on
    // launches of several rounds).
    const uint32_t prev = __hip_atomic_fetch_max(bo.ws, bc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("; fold returned %0" : : "v"(prev) : "memory");
    const uint32_t done = __hip_atomic_fetch_add(bo.ws + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done == gridDim.x - 1) {
        const uint32_t a = __hip_atomic_exchange(bo.ws, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(bo.ws + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t fl;
        *bo.bias = bias_of_fmt(bo.fmt, a, bo.margin, &fl);
        if (amax_out) *amax_out = a;
        if (bo.flags) *bo.flags = fl;
    }
}

}  // namespace
}  // namespace fp8lin
