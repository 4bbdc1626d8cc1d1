// Decoded-operand FP4 GEMM for few output rows (decoding and other small
// batches): C[m, n] = alpha * sum_k A_hat[m, k] * B_hat[n, k] with M <= 64.
// Same operands, decode and result contract as the kernels of gemm.hip; any
// K % 16 == 0, any size of operand (64-bit addresses) with N < 2^29.
//
// Bound: reading B, the quantized weight, once (N K / 2 bytes); with more than
// 32 rows the decode of A (skinny_gemm).  A 256 x 256
// output tile gives a weight of N rows only N / 256 workgroups that each walk
// all of K; here a workgroup owns 16 (NT = 1) or 32 (NT = 2) weight rows and
// its waves split K among themselves, so that every CU streams its share of
// the weight with many loads in flight, and the partial sums meet in LDS
// (added in wave order: the result does not depend on timing, and no
// workspace is needed).  Measured against the 256 x 256 tiles: 1 x 6144 x
// 4096 72.5 -> 5.9 us, 1 x 21504 x 4096 72.8 -> 10.9 us (4.1 TB/s of
// payload), 24 x 21504 x 4096 72.6 -> 17.7 us, 64 x 6144 x 4096 72.6 ->
// 12.8 us, 32 x 4096 x 21504 349 -> 27 us.
//
// v_mfma_f32_16x16x32_f16 with the weight as the row operand: lane l supplies
// 8 k-elements of weight row l % 16 and of A row l % 16, k group l / 16.  A
// step covers 128 k = 64 payload bytes of each row: group g takes the row's
// 16 bytes g (blocks 2g, 2g + 1), whose four words feed four products.  The
// k order inside a step is thus permuted, identically for both operands.
// Weight rows go straight from memory to registers (each is used once), four
// steps of loads ahead of the products; the A rows come from L2.  A wave's
// steps come in pairs that cover a whole 128-byte line of each row: single
// steps dealt over the waves had every line fetched by two waves, and L1 is
// too small for the lines in flight (24 x 21504 x 4096 20.0 -> 17.7 us).  A
// reload of each step's registers right after its products (in place of whole
// groups of four steps) took 30% more registers and was no faster.
#include "codec.hpp"
#include "fp4_decode.hpp"
#include "launch.hpp"

#include <type_traits>

namespace ue5m3 {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr int kSkAhead = 4;                      // steps whose loads are in flight together
constexpr int kSkBlocks = 8;                     // 16-element blocks per step

// One step's share of a lane: 16 payload bytes (two blocks) and their codes.
struct SkLoad {
    uint32_t w[4];
    uint32_t c0, c1;
};

// Blocks kb, kb + 1 of the row at pay / sc (kbt blocks).  FULL: kbt % 8 == 0
// and kb < kbt, so both exist, the payload is 16-byte and the pair of codes
// 2-byte aligned.  Otherwise blocks at or past kbt read block kbt - 1 and
// take code 0 (value 0).
template <bool FULL>
__device__ __forceinline__ void sk_load(SkLoad& r, const uint8_t* __restrict__ pay,
                                        const uint8_t* __restrict__ sc, int64_t kb, int64_t kbt) {
    if (FULL) {
        const uint4 v = *reinterpret_cast<const uint4*>(pay + kb * 8);
        r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.w[3] = v.w;
        const uint32_t c = *reinterpret_cast<const uint16_t*>(sc + kb);
        r.c0 = c & 0xFFu;
        r.c1 = c >> 8;
    } else {
        const int64_t k0 = min(kb, kbt - 1), k1 = min(kb + 1, kbt - 1);
        const uint2 a = *reinterpret_cast<const uint2*>(pay + k0 * 8);
        const uint2 b = *reinterpret_cast<const uint2*>(pay + k1 * 8);
        r.w[0] = a.x; r.w[1] = a.y; r.w[2] = b.x; r.w[3] = b.y;
        const uint32_t c0 = sc[k0], c1 = sc[k1];
        r.c0 = kb < kbt ? c0 : 0u;
        r.c1 = kb + 1 < kbt ? c1 : 0u;
    }
}

// Word j (8 elements) of a lane's 32 into an MFMA fragment.
template <int J>
__device__ __forceinline__ f16x8_t sk_frag(const SkLoad& r) {
    uint32_t o[4];
    decode8(r.w[J], scale_factors(J < 2 ? r.c0 : r.c1), o);
    const uint4 v = make_uint4(o[0], o[1], o[2], o[3]);
    return __builtin_bit_cast(f16x8_t, v);
}

// MT, NT: 16-row groups of A and of the weight per workgroup of W waves.
template <int BMODE, int MT, int NT, int W, bool FULL>
__global__ __launch_bounds__(64 * W) void gemm_fp4_skinny_kernel(
    int M, int64_t N, int64_t K, const uint8_t* __restrict__ A, const uint8_t* __restrict__ As,
    const float* __restrict__ a_dec, const uint8_t* __restrict__ B, const uint8_t* __restrict__ Bs,
    const float* __restrict__ b_dec, void* __restrict__ C, float amul, bool out_bf16) {
    __shared__ f32x4_t part[W][MT * NT][64];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * (16 * NT);
    const int64_t kbt = K / 16;
    const int64_t steps = (kbt + kSkBlocks - 1) / kSkBlocks;

    // row sources; rows past the matrix read its last row (their outputs are
    // not stored)
    const uint8_t *ap[MT], *as[MT], *bp[NT], *bs[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int64_t m = min(16 * i + r, M - 1);
        ap[i] = A + m * (kbt * 8);
        as[i] = As + m * kbt;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int64_t n = min(n0 + 16 * j + r, N - 1);
        bp[j] = B + n * (kbt * 8);
        bs[j] = Bs + (BMODE == (int)BScale::Row ? n : (n >> 4)) * kbt;
    }

    f32x4_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // Wave w takes step pairs w, w + W, ...: a pair is one whole 128-byte
    // line of every row.  kSkAhead steps are in flight.  A step past the last
    // one re-reads it with code 0 for the weight.
    for (int64_t s0 = 2 * wave; s0 < steps; s0 += W * kSkAhead) {
        SkLoad b[kSkAhead][NT], a[kSkAhead][MT];
#pragma unroll
        for (int u = 0; u < kSkAhead; ++u) {
            const int64_t s = s0 + (u & 1) + (u >> 1) * 2 * W;
            const int64_t kb = min(s, steps - 1) * kSkBlocks + 2 * g;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                sk_load<FULL>(b[u][j], bp[j], bs[j], kb, kbt);
                if (s >= steps) b[u][j].c0 = b[u][j].c1 = 0u;
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) sk_load<FULL>(a[u][i], ap[i], as[i], kb, kbt);
        }
#pragma unroll
        for (int u = 0; u < kSkAhead; ++u) {
            auto word = [&](auto jc) {
                constexpr int J = decltype(jc)::value;
                f16x8_t fb[NT], fa[MT];
#pragma unroll
                for (int j = 0; j < NT; ++j) fb[j] = sk_frag<J>(b[u][j]);
#pragma unroll
                for (int i = 0; i < MT; ++i) fa[i] = sk_frag<J>(a[u][i]);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[j], fa[i], acc[i][j], 0, 0, 0);
            };
            word(std::integral_constant<int, 0>{});
            word(std::integral_constant<int, 1>{});
            word(std::integral_constant<int, 2>{});
            word(std::integral_constant<int, 3>{});
        }
    }

    // ---- the waves' partial sums, in wave order -----------------------------
    // 16 x 16 accumulator: lane l holds column l % 16 (an A row) and rows
    // 4 (l / 16) .. + 3 (adjacent output columns n).
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) part[wave][i * NT + j][lane] = acc[i][j];
    __syncthreads();
    const float alpha = (a_dec[0] * b_dec[0]) * amul;      // operands were decoded times 2^-3
    for (int q = tid; q < MT * NT * 64; q += 64 * W) {
        const int ij = q >> 6, l = q & 63;
        f32x4_t v = part[0][ij][l];
#pragma unroll
        for (int w = 1; w < W; ++w) v += part[w][ij][l];
        const int m = 16 * (ij / NT) + (l & 15);
        const int64_t n = n0 + 16 * (ij % NT) + 4 * (l >> 4);
        if (m >= M) continue;
        const float y[4] = {alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]};
        const bool vec = (N & 3) == 0 && n + 3 < N;
        if (out_bf16) {
            uint16_t* d = reinterpret_cast<uint16_t*>(C) + m * N + n;
            if (vec) {
                *reinterpret_cast<uint2*>(d) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) d[e] = (uint16_t)pack_bf16x2(y[e], 0.0f);
            }
        } else {
            float* d = reinterpret_cast<float*>(C) + m * N + n;
            if (vec) {
                *reinterpret_cast<float4*>(d) = make_float4(y[0], y[1], y[2], y[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) d[e] = y[e];
            }
        }
    }
}

template <int BMODE, int MT, int NT, int W>
hipError_t launch_skinny_t(int64_t M, int64_t N, int64_t K, const uint8_t* a, const uint8_t* as, const float* ad,
                           const uint8_t* b, const uint8_t* bs, const float* bd, void* c, bool c_bf16, float amul,
                           hipStream_t s) {
    const dim3 grid((unsigned)((N + 16 * NT - 1) / (16 * NT)));
    if (K % (16 * kSkBlocks) == 0)
        hipLaunchKernelGGL((gemm_fp4_skinny_kernel<BMODE, MT, NT, W, true>), grid, dim3(64 * W), 0, s, (int)M, N, K,
                           a, as, ad, b, bs, bd, c, amul, c_bf16);
    else
        hipLaunchKernelGGL((gemm_fp4_skinny_kernel<BMODE, MT, NT, W, false>), grid, dim3(64 * W), 0, s, (int)M, N, K,
                           a, as, ad, b, bs, bd, c, amul, c_bf16);
    return hipGetLastError();
}

template <int BMODE, int MT>
hipError_t launch_skinny_m(int64_t M, int64_t N, int64_t K, const uint8_t* a, const uint8_t* as, const float* ad,
                           const uint8_t* b, const uint8_t* bs, const float* bd, void* c, bool c_bf16, float amul,
                           hipStream_t s) {
#define UE5M3_SKINNY(NT, W) launch_skinny_t<BMODE, MT, NT, W>(M, N, K, a, as, ad, b, bs, bd, c, c_bf16, amul, s)
    // 32 weight rows per workgroup halve the reads and decodes of A per weight
    // row: worth it once that still gives about every CU a workgroup, and
    // earlier with four A groups, whose decode dominates (24 x 21504 x 4096:
    // 17.6 us, with 16 rows 25.7; 64 x 6144 x 4096: 12.5 and 19.5; 24 x 2048 x
    // 2048: 5.1 and 4.5; 32 x 4096 x 21504: 34 and 27).
    if (N >= (MT == 4 ? 4096 : 8192)) return UE5M3_SKINNY(2, 4);
    // Eight waves on a long K (32 x 4096 x 21504: 27.1 us, with four 30.5);
    // four on a short one, where the sum over waves costs more than it gains
    // (24 x 2048 x 2048: 6.5 and 4.5 us; even at 12 x 4096 x 4096).
    return K > 4096 ? UE5M3_SKINNY(1, 8) : UE5M3_SKINNY(1, 4);
#undef UE5M3_SKINNY
}

template <int BMODE>
hipError_t launch_skinny_b(int64_t M, int64_t N, int64_t K, const uint8_t* a, const uint8_t* as, const float* ad,
                           const uint8_t* b, const uint8_t* bs, const float* bd, void* c, bool c_bf16, float amul,
                           hipStream_t s) {
    if (M <= 16) return launch_skinny_m<BMODE, 1>(M, N, K, a, as, ad, b, bs, bd, c, c_bf16, amul, s);
    if (M <= 32) return launch_skinny_m<BMODE, 2>(M, N, K, a, as, ad, b, bs, bd, c, c_bf16, amul, s);
    return launch_skinny_m<BMODE, 4>(M, N, K, a, as, ad, b, bs, bd, c, c_bf16, amul, s);
}

}  // namespace

bool skinny_gemm(int64_t M, int64_t N, int64_t K, int cus) {
    // a launch dimension holds less than 2^32 work-items: N / 32 workgroups of 256
    if (M <= 0 || M > 64 || K <= 0 || N <= 0 || N > ((int64_t)1 << 29) - 32) return false;
    // Up to 32 rows the weight's bytes bound the call.  Above, the decode of A,
    // which every workgroup repeats, does: the small tiles are ahead once the
    // workgroups of 32 weight rows outnumber the CUs, and where K is so short
    // that a wave's four steps in flight (2048 k of the workgroup) reach past
    // it.  Measured on 256 CUs, here / small tiles, us: 64 x 21504 x 4096 30.5
    // / 22, 33 x 21504 x 8192 45.5 / 39.8, 64 x 12288 x 8192 39.9 / 28.4, 33 x
    // 12288 x 2048 9.9 / 9.7, 64 x 65536 x 4096 89 / 46; 64 x 8192 x 4096 13.0
    // / 15.7, 64 x 8192 x 2048 8.3 / 9.6, 33 x 2048 x 4096 11.5 / 15.1; 64 x
    // 1024 x 512 5.9 / 4.5, 33 x 256 x 1024 6.5 / 6.2, 64 x 4096 x 1024 7.7 /
    // 6.3, 64 x 1024 x 1536 7.7 / 8.0.  At 17 to 32 rows the two cross over only
    // far out (32 x 21504 x 4096 19.5 / 22, 17 x 32768 x 4096 20.5 / 22.8, 24 x
    // 32768 x 4096 23.5 / 22.8, 32 x 65536 x 4096 54.7 / 42.9).
    return M <= 32 || (N <= 32 * (int64_t)cus && K > 1024) || !mid_gemm_fits(M, N, K);
}

hipError_t launch_gemm_skinny(BScale bmode, float amul, int64_t M, int64_t N, int64_t K, const uint8_t* a,
                              const uint8_t* a_scales, const float* a_dec, const uint8_t* b,
                              const uint8_t* b_scales, const float* b_dec, void* c, bool c_bf16, hipStream_t s) {
    return bmode == BScale::Row
               ? launch_skinny_b<(int)BScale::Row>(M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16, amul, s)
               : launch_skinny_b<(int)BScale::Tile>(M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16, amul,
                                                    s);
}

}  // namespace ue5m3
