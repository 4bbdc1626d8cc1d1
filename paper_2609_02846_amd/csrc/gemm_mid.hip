// Decoded-operand FP4 GEMM in tiles of 64 or 128 rows and columns, any
// K % 16 == 0: the calls whose 256 x 256 tiles (gemm_fp4_reg_kernel) would
// leave most CUs idle, and the leftover tiles of large products whose K is
// not a multiple of 256 (reg_plan).
//
// The decode is the register decode of gemm_fp4_reg_kernel: the packed rows
// and their scale codes are staged in LDS 256 k at a time, double buffered,
// and each wave decodes its own fragments.  A wave covers (32 TM) x (32 TN)
// outputs, a group of four waves (2 x 2) a tile of (64 TM) x (64 TN), and KS
// groups of one workgroup share the tile's K and add up in LDS (in group
// order: deterministic, no workspace).
//
// Bound: the decode.  A k-step of a wave has TM TN products and 8 (TM + TN)
// conversions and multiplies; about four of them hide behind a product of 32
// cycles, so 2 x 2 (8 per product) costs about 52 cycles per product where
// the 4 x 4 of gemm_fp4_reg_kernel (4.35) costs 39.  Small tiles win where
// large ones leave CUs without work (mid_plan, reg_time).  Measured against
// the kernels that ran before, us: 300 x 4096 x 4096 72 -> 22, 777 x 4096 x
// 21504 352 -> 151, dgrad 2000 x 4096 x 6144 109 -> 97; K not a multiple of
// 256: 1520 x 1360 x 3408 178 -> 29, 1520 x 3408 x 1360 71 -> 26.
#include "codec.hpp"
#include "fp4_decode.hpp"
#include "gemm_regs.hpp"
#include "launch.hpp"

namespace ue5m3 {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

constexpr int kMidK = 256;                       // k per stage
constexpr int kMidRow = kMidK / 2;               // payload bytes of a stage row
constexpr int kMidSc = kMidK / 16;               // scale bytes of a stage row
constexpr int kMidXcds = 8, kMidGroupM = 4;

// One slice (64 k) of a lane's operands: rows 32 i + l % 32 of its wave's A
// rows (groups 0 .. TM-1) and B rows (TM ..): four payload words and the
// row's scale word (see decode order in gemm_fp4_reg_kernel).
template <int G>
struct MidSlice {
    uint32_t w[G][4];
    uint32_t s[G];
};

template <int TM, int TN>
struct MidFrags {
    f16x8_t a[TM], b[TN];
};

template <int TM, int TN, int KK>
__device__ __forceinline__ void mid_decode(MidFrags<TM, TN>& f, MidSlice<TM + TN>& R, uint32_t sel) {
    if (KK == 0) {
#pragma unroll
        for (int g = 0; g < TM + TN; ++g) {
            R.s[g] = half_scales(R.s[g], sel);
            asm("" : "+v"(R.s[g]));              // keep the half selection in op_sel
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = decode_frag<KK / 2>(R.w[i][KK], R.s[i]);
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = decode_frag<KK / 2>(R.w[TM + j][KK], R.s[TM + j]);
}

// The products of one k-step, issued as B x A^T: element e of lane l is row
// l % 32, column 8 (e / 4) + 4 (l / 32) + e % 4 of accumulator (i, j).
template <int TM, int TN>
__device__ __forceinline__ void mid_mfma(f32x16_t (&acc)[TM][TN], const MidFrags<TM, TN>& f) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
}

// Origin of tile t: contiguous ranges of tiles per XCD (workgroups are dealt
// round-robin over the XCDs), walked in groups of kMidGroupM tile rows.
__device__ __forceinline__ void mid_origin(int t, int tiles_m, int tiles_n, int bm, int bn, int64_t& m0,
                                           int64_t& n0) {
    const int ntiles = tiles_m * tiles_n;
    const int x = t % kMidXcds, q = ntiles / kMidXcds, rem = ntiles % kMidXcds;
    t = x * q + min(x, rem) + t / kMidXcds;
    const int group_tiles = kMidGroupM * tiles_n;
    const int g = t / group_tiles;
    const int first_m = g * kMidGroupM;
    const int gm = min(tiles_m - first_m, kMidGroupM);
    const int rr = t - g * group_tiles;
    m0 = (int64_t)(first_m + rr % gm) * bm;
    n0 = (int64_t)(rr / gm) * bn;
}

// Scale codes kb0 .. kb0 + 15 of a row of kbt codes; codes at or past kbt
// are 0, so the payload bytes staged beside them (the next row's, or stale)
// count as zeros.
__device__ __forceinline__ uint4 mid_scales(const uint8_t* __restrict__ row, int kb0, int kbt) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (kb0 + kMidSc <= kbt) {
        __builtin_memcpy(&v, row + kb0, 16);     // rows of kbt bytes: any alignment
    } else {
        uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int b = 0; b < kMidSc; ++b)
            if (kb0 + b < kbt) d[b >> 2] |= (uint32_t)row[kb0 + b] << (8 * (b & 3));
        v = make_uint4(d[0], d[1], d[2], d[3]);
    }
    return v;
}

template <int BMODE, int TM, int TN, int KS, bool OUT_BF16>
__global__ __launch_bounds__(256 * KS, KS == 1 ? 2 : 1) void gemm_fp4_mid_kernel(
    int M, int N, int K, int tiles_m, int tiles_n, int tail, const uint8_t* __restrict__ A, const uint8_t* __restrict__ As,
    const float* __restrict__ a_dec, const uint8_t* __restrict__ B, const uint8_t* __restrict__ Bs,
    const float* __restrict__ b_dec, void* __restrict__ C, float amul) {
    constexpr int G = TM + TN;
    constexpr int kRows = 64 * G;                                  // stage rows: A, then B
    constexpr int kPay = kRows * kMidRow, kScl = kRows * kMidSc;
    constexpr int kStage = kPay + kScl;
    __shared__ __attribute__((aligned(16))) uint8_t smem[KS * 2 * kStage];

    const int tid = threadIdx.x & 255;                             // within the K group
    const int lane = threadIdx.x & 63;
    const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 31, hi = lane >> 5;
    uint8_t* const buf0 = smem + kg * 2 * kStage;
    uint8_t* const buf1 = buf0 + kStage;

    int64_t m0, n0;
    if (tail < 0) {
        mid_origin(blockIdx.x, tiles_m, tiles_n, 64 * TM, 64 * TN, m0, n0);
    } else {
        // the large tiles from `tail` on (tiles_m x tiles_n of them), in pieces
        constexpr int kPieces = (BN / (64 * TN)) * (BM / (64 * TM));
        const int q = blockIdx.x % kPieces;
        tile_origin(tail + blockIdx.x / kPieces, tiles_m, tiles_n, m0, n0);
        m0 += q / (BN / (64 * TN)) * 64 * TM;
        n0 += q % (BN / (64 * TN)) * 64 * TN;
        if (m0 >= M || n0 >= N) return;              // the whole workgroup
    }

    const int kbt = K / 16;
    const int slices = (kbt + 3) / 4, stages = (kbt + kMidSc - 1) / kMidSc;
    // this group's stages [g0, g0 + nst); the last group has the most
    const int g0 = stages * kg / KS, nst = stages * (kg + 1) / KS - g0;
    const int iters = stages - stages * (KS - 1) / KS;

    // ---- loads -----------------------------------------------------------------
    // Payload: instruction i of wave w brings stage rows 8 (4 i + w) .. + 7 of
    // 128 bytes; lane l covers row l / 8, position l % 8, which holds chunk
    // (l % 8) ^ (l / 8) (so that the 8 lanes the LDS serves together hit
    // different banks).  The whole offset is in the per-lane operand, which
    // the buffer's range check covers, each 4-byte word on its own (measured:
    // 16-byte direct loads across the end of a range bring the words inside
    // it and zeros): rows past the matrix give zeros, and the last row's last
    // chunk, of which K % 32 == 16 leaves half, reads nothing past the end.
    const uint32_t rowb = (uint32_t)kbt * 8u;
    const i32x4_t ra = buffer_rsrc(A, (uint32_t)M * rowb), rb = buffer_rsrc(B, (uint32_t)N * rowb);
    const uint32_t chunk16 = (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
    const uint32_t offa = (uint32_t)(m0 + 8 * wave + (lane >> 3)) * rowb + chunk16;
    const uint32_t offb = (uint32_t)(n0 + 8 * wave + (lane >> 3)) * rowb + chunk16;
    const uint32_t l0 = lds_addr(buf0) + 1024u * wave, l1 = lds_addr(buf1) + 1024u * wave;
    auto issue = [&](uint32_t dst, int g) {
        const uint32_t gp = (uint32_t)(g0 + g) * kMidRow;
        static_for<0, 2 * TM>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            dma_buf_x4<i * 4096>(ra, offa + (gp + (uint32_t)(32 * i) * rowb), 0u, dst);
        });
        static_for<0, 2 * TN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            dma_buf_x4<(2 * TM + i) * 4096>(rb, offb + (gp + (uint32_t)(32 * i) * rowb), 0u, dst);
        });
    };
    // Scales: thread t < kRows carries stage row t's 16 codes through
    // registers (rows of kbt bytes have no alignment).
    const uint8_t* srow;
    if (tid < 64 * TM) {
        srow = As + min(m0 + tid, (int64_t)M - 1) * kbt;
    } else {
        const int64_t n = min(n0 + tid - 64 * TM, (int64_t)N - 1);
        srow = Bs + (BMODE == (int)BScale::Row ? n : (n >> 4)) * kbt;
    }
    const bool has_row = kRows == 256 || tid < kRows;
    uint4 sreg = make_uint4(0u, 0u, 0u, 0u);
    auto load_scales = [&](int g) {
        if (has_row) sreg = mid_scales(srow, (g0 + g) * kMidSc, kbt);
    };
    auto put_scales = [&](uint8_t* buf) {
        if (has_row) *reinterpret_cast<uint4*>(buf + kPay + tid * kMidSc) = sreg;
    };

    // ---- fragment reads ----------------------------------------------------------
    const int pa = (wm * 32 * TM + r) * kMidRow, pb = (64 * TM + wn * 32 * TN + r) * kMidRow;
    const int x0 = ((0 + hi) ^ (r & 7)) * 16, x1 = ((2 + hi) ^ (r & 7)) * 16;
    const int x2 = ((4 + hi) ^ (r & 7)) * 16, x3 = ((6 + hi) ^ (r & 7)) * 16;
    const uint32_t sel = hi ? 0x0C030C02u : 0x0C010C00u;
    auto read_slice = [&](MidSlice<G>& R, const uint8_t* buf, int sl, int xo) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int off = (g < TM ? pa : pb - TM * 32 * kMidRow) + g * 32 * kMidRow;
            const uint4 v = *reinterpret_cast<const uint4*>(buf + off + xo);
            R.w[g][0] = v.x; R.w[g][1] = v.y; R.w[g][2] = v.z; R.w[g][3] = v.w;
            R.s[g] = *reinterpret_cast<const uint32_t*>(buf + kPay + off / kMidRow * kMidSc + sl * 4);
        }
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // ---- pipeline ----------------------------------------------------------------
    // Stage g is in buffer g & 1.  During its last slice (after the barrier
    // that follows the arrival of stage g + 1) the loads of stage g + 2 go
    // into the buffer just consumed.
    issue(l0, 0);
    load_scales(0);
    wait_vmem<0>();
    put_scales(buf0);
    if (nst > 1) {
        issue(l1, 1);
        load_scales(1);
    }
    __syncthreads();

    MidSlice<G> R0, R1;
    MidFrags<TM, TN> F0, F1;
    if (nst > 0) {
        read_slice(R0, buf0, 0, x0);
        mid_decode<TM, TN, 0>(F0, R0, sel);
    }
    // Each product is followed by VALU slots: a k-step has TM TN products and
    // 8 (TM + TN) decode instructions.  Two slots fewer than their quotient
    // measured best (6 for 2 x 2: 777 x 4096 x 21504 157 us, 8 slots 163,
    // none 177).
    constexpr int kValu = (8 * G + TM * TN - 1) / (TM * TN) - 2;
    auto sched = [&]() {
#pragma unroll
        for (int q = 0; q < TM * TN; ++q) {
            __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kSgValu, kValu, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // k-steps 1 (decoded before) .. 3 of slice Rc; the first k-step of Rn
    auto products = [&](MidSlice<G>& Rc, MidSlice<G>& Rn) {
        mid_decode<TM, TN, 2>(F0, Rc, sel);
        mid_mfma<TM, TN>(acc, F1);
        sched();
        mid_decode<TM, TN, 3>(F1, Rc, sel);
        mid_mfma<TM, TN>(acc, F0);
        sched();
        mid_decode<TM, TN, 0>(F0, Rn, sel);
        mid_mfma<TM, TN>(acc, F1);
        sched();
    };
    // Stage `it` of the group from buffer `cur`.  The tile's last stage may
    // hold fewer than four slices; it is the last one of the group with the
    // most stages, so no barrier follows it.  Groups with fewer stages meet
    // the same barriers: each iteration but the last of `iters` has one.
    auto stage = [&](int it, const uint8_t* cur, uint8_t* nxt, uint32_t lcur) {
        const int left = slices - 4 * (g0 + it);
        auto slice = [&](int sl, int xo, MidSlice<G>& Rc, MidSlice<G>& Rn) {
            mid_decode<TM, TN, 1>(F1, Rc, sel);
            mid_mfma<TM, TN>(acc, F0);
            sched();
            read_slice(Rn, cur, sl + 1, xo);
            products(Rc, Rn);
        };
        slice(0, x1, R0, R1);
        if (left <= 1) return;
        slice(1, x2, R1, R0);
        if (left <= 2) return;
        slice(2, x3, R0, R1);
        if (left <= 3) return;
        mid_decode<TM, TN, 1>(F1, R1, sel);
        mid_mfma<TM, TN>(acc, F0);
        sched();
        if (it + 1 < iters) {
            wait_vmem<0>();
            put_scales(nxt);
            __syncthreads();
            if (it + 1 < nst) read_slice(R0, nxt, 0, x0);
            if (it + 2 < nst) {
                issue(lcur, it + 2);
                load_scales(it + 2);
            }
        }
        products(R1, R0);
    };
    for (int it = 0; it < nst; it += 2) {
        stage(it, buf0, buf1, l0);
        if (it + 1 < nst) stage(it + 1, buf1, buf0, l1);
    }

    // ---- sum over the K groups, store ------------------------------------------------
    // the stage buffers are free after the barrier; group 0 adds and stores
    __syncthreads();
    if (KS > 1) {
        f32x4_t* ex = reinterpret_cast<f32x4_t*>(smem) + wave * (TM * TN * 4 * 64) + lane;
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        ex[((i * TN + j) * 4 + q) * 64] = f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1],
                                                                 acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4_t v = ex[((i * TN + j) * 4 + q) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
                }
    }
    const float alpha = (a_dec[0] * b_dec[0]) * amul;              // operands were decoded times 2^-3
    constexpr int esz = OUT_BF16 ? 2 : 4;
    const int64_t mw = m0 + wm * 32 * TM, nw = n0 + wn * 32 * TN;
    // Through LDS, 32 rows at a time, so that the stores write whole runs of
    // a row: rows of 32 TN values, padded by 16 bytes (KS > 1: placed past
    // the exchanged partials).
    constexpr int kRowB = 32 * TN * esz + 16;
    constexpr int kChunks = 32 * TN * esz / 16;                    // 16-byte chunks per row
    constexpr int kPer = 64 / kChunks;                             // rows per store instruction
    uint8_t* const ep = smem + (KS > 1 ? TM * TN * 16384 : 0) + wave * (32 * kRowB);
    static_assert((KS > 1 ? TM * TN * 16384 : 0) + 4 * 32 * kRowB <= KS * 2 * kStage, "epilogue fits the stages");
    const bool vec = (N * esz) % 16 == 0;                          // runs of 16 bytes wholly inside or outside C
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v0 = alpha * acc[i][j][4 * q], v1 = alpha * acc[i][j][4 * q + 1];
                const float v2 = alpha * acc[i][j][4 * q + 2], v3 = alpha * acc[i][j][4 * q + 3];
                uint8_t* d = ep + r * kRowB + (32 * j + 8 * q + 4 * hi) * esz;
                if (OUT_BF16)
                    *reinterpret_cast<u32x2_t*>(d) = u32x2_t{pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
                else
                    *reinterpret_cast<f32x4_t*>(d) = f32x4_t{v0, v1, v2, v3};
            }
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < 32 / kPer; ++t) {
            const int row = t * kPer + lane / kChunks, ch = lane % kChunks;
            const u32x4_t d = *reinterpret_cast<const u32x4_t*>(ep + row * kRowB + ch * 16);
            const int64_t m = mw + 32 * i + row, n = nw + ch * (16 / esz);
            if (m < M && n < N) {
                uint8_t* o = reinterpret_cast<uint8_t*>(C) + (m * N + n) * esz;
                if (vec) {
                    *reinterpret_cast<u32x4_t*>(o) = d;
                } else {
#pragma unroll
                    for (int e = 0; e < 16 / esz; ++e)
                        if (n + e < N) {
                            if (OUT_BF16)
                                reinterpret_cast<uint16_t*>(o)[e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
                            else
                                reinterpret_cast<uint32_t*>(o)[e] = d[e];
                        }
                }
            }
        }
        wave_lds_sync();
    }
}

template <int BMODE, int TM, int TN, int KS>
hipError_t launch_mid_t(int blocks, int tiles_m, int tiles_n, int tail, int64_t M, int64_t N, int64_t K, const uint8_t* a,
                        const uint8_t* as, const float* ad, const uint8_t* b, const uint8_t* bs, const float* bd, void* c,
                        bool c_bf16, float amul, hipStream_t s) {
    if (c_bf16)
        hipLaunchKernelGGL((gemm_fp4_mid_kernel<BMODE, TM, TN, KS, true>), dim3((unsigned)blocks), dim3(256 * KS), 0, s,
                           (int)M, (int)N, (int)K, tiles_m, tiles_n, tail, a, as, ad, b, bs, bd, c, amul);
    else
        hipLaunchKernelGGL((gemm_fp4_mid_kernel<BMODE, TM, TN, KS, false>), dim3((unsigned)blocks), dim3(256 * KS), 0, s,
                           (int)M, (int)N, (int)K, tiles_m, tiles_n, tail, a, as, ad, b, bs, bd, c, amul);
    return hipGetLastError();
}

// Modelled time (us) of one configuration: the busiest CU runs `per` tiles,
// each with a fixed part (prologue, epilogue) and tau ns per k.
double mid_time(int64_t tiles, int64_t K, int cus, double fixed, double tau, double tau1) {
    const int64_t per = (tiles + cus - 1) / cus;
    return 3.0 + per * (fixed + 1e-3 * K * (per == 1 ? tau1 : tau));
}
struct MidPlan {
    int tm, tn, ks;
    double us;
};

// The configuration with the smallest modelled time.  Constants fitted to
// launches on a 256-CU device (model / measured, us): 300 x 4096 x 4096
// 1x2x2 23 / 22 (2x2x2 31 / 30, 1x1x2 29 / 25), 777 x 4096 x 21504 2x2x2
// 153 / 151 (2x2x1 169 / 164, 1x2x1 205 / 190), 100 x 6144 x 4096 1x1x2
// 17 / 15.5, 1520 x 1360 x 3408 2x2x2 30 / 29, 1520 x 3408 x 1360 2x2x1
// 27 / 26, 6144 x 4096 x 8000 2x2x1 361 / 365.  Two K groups (ks = 2) help a CU that has only one tile: with one
// wave per SIMD its decode and products do not overlap fully.
template <typename Tiles>
MidPlan mid_plan(Tiles tiles, int64_t K, int cus) {
    const MidPlan c[6] = {
        {2, 2, 1, mid_time(tiles(2, 2), K, cus, 2.0, 7.2, 7.6)}, {2, 2, 2, mid_time(tiles(2, 2), K, cus, 3.5, 7.2, 6.8)},
        {1, 2, 1, mid_time(tiles(1, 2), K, cus, 1.7, 4.6, 5.1)}, {1, 2, 2, mid_time(tiles(1, 2), K, cus, 2.8, 4.6, 4.2)},
        {1, 1, 1, mid_time(tiles(1, 1), K, cus, 1.0, 2.9, 3.4)}, {1, 1, 2, mid_time(tiles(1, 1), K, cus, 2.0, 2.9, 2.8)},
    };
    MidPlan best = c[0];
    for (int i = 1; i < 6; ++i)
        if (c[i].us < best.us) best = c[i];
    return best;
}

// The whole product; `large` tiles of 256 x 256 cut into smaller ones.
MidPlan mid_plan(int64_t M, int64_t N, int64_t K, int cus) {
    return mid_plan([=](int tm, int tn) { return ((M + 64 * tm - 1) / (64 * tm)) * ((N + 64 * tn - 1) / (64 * tn)); }, K,
                    cus);
}
MidPlan mid_tail_plan(int64_t K, int64_t large, int cus) {
    return mid_plan([=](int tm, int tn) { return large * (BM / (64 * tm)) * (BN / (64 * tn)); }, K, cus);
}

// tail < 0: the whole product; otherwise its large tiles from `tail` on.
template <int BMODE>
hipError_t launch_mid_b(const MidPlan& p, int tail, int64_t M, int64_t N, int64_t K, const uint8_t* a, const uint8_t* as,
                        const float* ad, const uint8_t* b, const uint8_t* bs, const float* bd, void* c, bool c_bf16,
                        float amul, hipStream_t s) {
    const int bm = tail < 0 ? 64 * p.tm : BM, bn = tail < 0 ? 64 * p.tn : BN;
    const int tm = (int)((M + bm - 1) / bm), tn = (int)((N + bn - 1) / bn);
    const int blocks = tail < 0 ? tm * tn : (tm * tn - tail) * (BM / (64 * p.tm)) * (BN / (64 * p.tn));
#define UE5M3_MID_ARGS (blocks, tm, tn, tail, M, N, K, a, as, ad, b, bs, bd, c, c_bf16, amul, s)
#define UE5M3_MID(TM, TN) (p.ks == 1 ? launch_mid_t<BMODE, TM, TN, 1> UE5M3_MID_ARGS : launch_mid_t<BMODE, TM, TN, 2> UE5M3_MID_ARGS)
    if (p.tm == 2) return UE5M3_MID(2, 2);
    if (p.tn == 2) return UE5M3_MID(1, 2);
    return UE5M3_MID(1, 1);
#undef UE5M3_MID
#undef UE5M3_MID_ARGS
}

}  // namespace

bool mid_gemm_fits(int64_t M, int64_t N, int64_t K) {
    const int64_t lim = (int64_t)1 << 31;
    return K > 0 && K < lim && M * (K / 2) < lim && N * (K / 2) < lim && M < lim - 256 && N < lim - 256 &&
           ((M + 63) / 64) * ((N + 63) / 64) < lim;
}

double mid_gemm_time(int64_t M, int64_t N, int64_t K, int cus) { return mid_plan(M, N, K, cus).us; }

hipError_t launch_gemm_mid(BScale bmode, float amul, int64_t M, int64_t N, int64_t K, int cus, const uint8_t* a,
                           const uint8_t* a_scales, const float* a_dec, const uint8_t* b, const uint8_t* b_scales,
                           const float* b_dec, void* c, bool c_bf16, hipStream_t s) {
    const MidPlan p = mid_plan(M, N, K, cus);
    return bmode == BScale::Row
               ? launch_mid_b<(int)BScale::Row>(p, -1, M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16, amul,
                                                s)
               : launch_mid_b<(int)BScale::Tile>(p, -1, M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16,
                                                 amul, s);
}

double mid_tail_time(int64_t K, int64_t large, int cus) { return mid_tail_plan(K, large, cus).us; }

hipError_t launch_gemm_mid_tail(BScale bmode, float amul, int64_t M, int64_t N, int64_t K, int cus, int first,
                                const uint8_t* a, const uint8_t* a_scales, const float* a_dec, const uint8_t* b,
                                const uint8_t* b_scales, const float* b_dec, void* c, bool c_bf16, hipStream_t s) {
    const int64_t large = ((M + BM - 1) / BM) * ((N + BN - 1) / BN) - first;
    const MidPlan p = mid_tail_plan(K, large, cus);
    return bmode == BScale::Row
               ? launch_mid_b<(int)BScale::Row>(p, first, M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16,
                                                amul, s)
               : launch_mid_b<(int)BScale::Tile>(p, first, M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, c, c_bf16,
                                                 amul, s);
}

}  // namespace ue5m3
