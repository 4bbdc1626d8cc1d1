// Pieces shared by the register-decode GEMM kernels: fragment decode, direct
// buffer -> LDS loads that the kernels count themselves, wait and scheduling
// helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fp4_decode.hpp"

namespace ue5m3 {
namespace {

// The large output tile, and how tiles are dealt to the XCDs.
constexpr int BM = 256, BN = 256;
constexpr int kXcds = 8;
constexpr int kGroupM = 4;

// Origin of logical tile t: workgroups are dispatched round-robin over the
// XCDs, so logical tiles are remapped to give each XCD a contiguous range,
// walked in groups of kGroupM tile rows (column-major inside a group) so
// that tiles running together on one XCD share A and B rows in its L2.
__device__ __forceinline__ void tile_origin(int t, int tiles_m, int tiles_n, int64_t& m0, int64_t& n0) {
    const int ntiles = tiles_m * tiles_n;
    if (ntiles % kXcds == 0) t = (t % kXcds) * (ntiles / kXcds) + t / kXcds;
    const int group_tiles = kGroupM * tiles_n;
    const int g = t / group_tiles;
    const int first_m = g * kGroupM;
    const int gm = min(tiles_m - first_m, kGroupM);
    const int rr = t - g * group_tiles;
    m0 = (int64_t)(first_m + rr % gm) * BM;
    n0 = (int64_t)(rr / gm) * BN;
}

// Instruction classes for the scheduling-group builtins.
constexpr int kSgValu = 0x002, kSgMfma = 0x008, kSgVmemRead = 0x020, kSgDsRead = 0x100;

typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) void* glb_void_ptr;

__device__ __forceinline__ uint32_t half_scales(uint32_t word, uint32_t sel) {
    return __builtin_amdgcn_perm(0u, word, sel) << 7;
}

template <int HSEL>
__device__ __forceinline__ f16x8_t decode_frag(uint32_t w, uint32_t s2) {
    const f16x2_t sp = __builtin_bit_cast(f16x2_t, s2);
    const f16x2_t sc = __builtin_shufflevector(sp, sp, HSEL, HSEL);   // op_sel picks the half
    const f16x2_t v0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 0.125f, 0) * sc;
    const f16x2_t v1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 0.125f, 1) * sc;
    const f16x2_t v2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 0.125f, 2) * sc;
    const f16x2_t v3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 0.125f, 3) * sc;
    return f16x8_t{v0[0], v0[1], v1[0], v1[1], v2[0], v2[1], v3[0], v3[1]};
}

// Direct global->LDS loads written as instructions the compiler does not
// model: it would otherwise wait for every outstanding direct load before any
// LDS read (it cannot tell the stage arrays apart), which would remove the
// overlap.  The kernel counts them itself with vmcnt.  The LDS destination of
// lane l is m0 + 16 l.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_ptr)p);
}

// Calls f(integral_constant<int, i>) for i in [I0, I1).
template <int I0, int I1, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I0 < I1) {
        f(std::integral_constant<int, I0>{});
        static_for<I0 + 1, I1>(f);
    }
}

// Buffer resource of a raw byte range [base, base + bytes): loads whose
// per-lane offset falls outside it are dropped by the hardware.
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4_t buffer_rsrc(const void* base, uint32_t bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)base;
    i32x4_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));   // stride 0
    r[2] = (int)bytes;
    r[3] = 0x00020000;                                                   // 32-bit data format
    return r;
}

// 16 bytes per lane from rsrc at voff + soff into LDS at lds + OFF + 16 lane
// (the LDS offset is added inside the instruction sequence so that the
// compiler does not keep one register per destination).
template <int OFF>
__device__ __forceinline__ void dma_buf_x4(i32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :: "v"(voff), "s"(rsrc), "s"(soff), "s"(lds), "i"(OFF) : "memory", "m0", "scc");
}

// vmcnt(n) with expcnt and lgkmcnt left at their maxima (n < 64).
template <int n>
__device__ __forceinline__ void wait_vmem() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x0F70);
}

// Orders a wave's LDS writes before its own later LDS reads of what other
// lanes wrote (and those reads before the next writes): the LDS serves one
// wave's instructions in order, so the compiler only must not move memory
// accesses across this point and the data must have landed.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0)
    asm volatile("" ::: "memory");
}

}  // namespace
}  // namespace ue5m3
