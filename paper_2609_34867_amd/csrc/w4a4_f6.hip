// W4A4 linear for large M on the 6-bit matrix instructions.
//
// gfx950 multiplies 6-bit floats (v_mfma_f32_16x16x128_f8f6f4, both operands
// 6 bits wide) at twice the rate of int8.  Every int4 code -8..7 is exactly
// representable in the E3M2 format (3 exponent and 2 mantissa bits: the
// integers up to 8), every product is an integer of magnitude <= 64, and
// every partial sum an integer of magnitude <= 64 K_in <= 2^23 for K_in <=
// 131072, so the fp32 accumulators hold the exact integers that int8 MFMA
// gives, in any order of summation (checked at K = 131072 with all codes at
// the extremes): the same y and acc, bit for bit.
//
// Two launches: k_codes_f6 rewrites both operands' packed codes as 6-bit
// fragments (1.25 bytes of traffic per code) and k_w4a4_gemm_f6 contracts
// them.  Unpacking inside the GEMM instead (as the int8 kernels do) does not
// fit: a 6-bit MFMA leaves too few VALU slots per operand value.
#include "gemm_device.h"
#include "p4q_internal.h"

#include <algorithm>
#include <type_traits>

namespace p4q {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 v32h __attribute__((ext_vector_type(32)));

// Fragment layout of an operand [R][K]: row blocks of 256 rows, each a run of
// stages of 128 k; a stage holds 16 fragments of 16 rows.  A fragment is one
// MFMA operand: lane l's 24 bytes are the 32 codes of row l % 16, k chunk
// l / 16, as a plane of 16 bytes per lane and a plane of 8 bytes per lane.
// So a stage is one linear 24 KB copy into LDS, every fragment read is free
// of bank conflicts, and its two loads fill six consecutive registers (three
// 16-byte loads for two fragments cost register moves).
constexpr int F_BM = 256, F_BN = 256;
constexpr int F_KS = 128;                        // k per stage
constexpr int kFragBytes = 1536;                 // 16 rows x 128 k
constexpr int kPairBytes = 2 * kFragBytes;
constexpr int kOpStage = 8 * kPairBytes;         // one operand's stage: 24 KB
constexpr int kStageF = 2 * kOpStage;
constexpr int kRing = 3;
constexpr int kScaleBuf = (F_BM + F_BN) * 4;
constexpr int kScaleRing = 3;

// 32 packed int4 codes (16 bytes) -> 32 6-bit floats (24 bytes).  Nibbles
// become fp16 1024 + (code + 8) by masking, minus 1032 is the code; the
// conversion instruction packs 32 of them.  The order of the 32 values is
// permuted, the same way for both operands, which the contraction over k
// does not see.
__device__ __forceinline__ v6i codes_to_f6(uint4 c) {
    union {
        v32h v;
        h2 p[16];
    } u;
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t o = w[i] ^ 0x88888888u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t q = ((o >> (4 * j)) & 0x000F000Fu) | 0x64006400u;
            u.p[4 * i + j] = __builtin_bit_cast(h2, q) - h2{(_Float16)1032.0f, (_Float16)1032.0f};
        }
    }
    return __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(u.v, 1.0f);
}

// One wavefront rewrites 32 rows x kConvK stages: lane l reads row l % 16
// (and + 16), k chunk l / 16.  Bound by its memory traffic; the stores are
// whole planes.  Rows past R are not written (what lies there reaches
// only output rows that are not stored); k past K is zero.
constexpr int kConvK = 4;

__global__ __launch_bounds__(256) void k_codes_f6(const uint8_t *__restrict__ a, int Ra,
                                                  uint8_t *__restrict__ fa, int itemsA,
                                                  const uint8_t *__restrict__ w, int Rw,
                                                  uint8_t *__restrict__ fw, int items, int Kb,
                                                  int KT, int segs) {
    const int lane = threadIdx.x & 63;
    int item = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (item >= items) return;
    const bool isw = item >= itemsA;
    if (isw) item -= itemsA;
    const uint8_t *src = isw ? w : a;
    uint8_t *dst = isw ? fw : fa;
    const int R = isw ? Rw : Ra;
    const int pair = item / segs, kt0 = (item - pair * segs) * kConvK;
    const int r0 = 32 * pair + (lane & 15), r1 = r0 + 16;
    const int n = min(kConvK, KT - kt0);
    uint4 c0[kConvK], c1[kConvK];
#pragma unroll
    for (int i = 0; i < kConvK; ++i) {
        const int kb = (kt0 + i) * (F_KS / 2) + 16 * (lane >> 4);
        c0[i] = c1[i] = make_uint4(0, 0, 0, 0);
        if (i < n && kb < Kb) {
            if (r0 < R) c0[i] = *reinterpret_cast<const uint4 *>(src + (int64_t)r0 * Kb + kb);
            if (r1 < R) c1[i] = *reinterpret_cast<const uint4 *>(src + (int64_t)r1 * Kb + kb);
        }
    }
    uint8_t *out = dst + ((int64_t)(pair >> 3) * KT + kt0) * kOpStage + (pair & 7) * kPairBytes;
#pragma unroll
    for (int i = 0; i < kConvK; ++i) {
        if (i >= n) break;
        const v6i f0 = codes_to_f6(c0[i]), f1 = codes_to_f6(c1[i]);
        uint8_t *o = out + (int64_t)i * kOpStage;
        *reinterpret_cast<v4i *>(o + 16 * lane) = v4i{f0[0], f0[1], f0[2], f0[3]};
        *reinterpret_cast<v2i *>(o + 1024 + 8 * lane) = v2i{f0[4], f0[5]};
        *reinterpret_cast<v4i *>(o + kFragBytes + 16 * lane) = v4i{f1[0], f1[1], f1[2], f1[3]};
        *reinterpret_cast<v2i *>(o + kFragBytes + 1024 + 8 * lane) = v2i{f1[4], f1[5]};
    }
}

// acc += w a^T, both operands E3M2.  Inline assembly, so that the 256
// accumulators stay in the accumulation registers: with the builtin the
// register allocator moved them through the other half of the register file
// at every stage (263 spills).  The compiler knows no hazards of it: the
// caller keeps the distances to the writes before the first and the reads after
// the last one, and holds the accumulators behind them (hold_acc).
__device__ __forceinline__ void mfma_f6(v6i w, v6i a, v4f &acc) {
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:3 blgp:3" : "+a"(acc) : "v"(w), "v"(a));
}

// No instruction: every use of acc before it stays before, every one after it
// after, in the order of the other volatile statements.
template <int NF>
__device__ __forceinline__ void hold_acc(v4f (&acc)[NF][NF]) {
    static_assert(NF == 8, "operands");
#pragma unroll
    for (int i = 0; i < NF; ++i)
        asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]), "+a"(acc[i][2]), "+a"(acc[i][3]),
                     "+a"(acc[i][4]), "+a"(acc[i][5]), "+a"(acc[i][6]), "+a"(acc[i][7]));
}

// 256 x 256 tile on 4 wavefronts of 128 x 128 (one per SIMD: 256 accumulator
// and 192 operand registers), persistent work-groups, one per CU, with one
// DMA ring of 3 stages running on across tile boundaries.
//  * LDS traffic is what bounds the shape: per stage a wavefront reads 24 KB
//    for 64 MFMAs of 16 cycles; four of them read 96 KB (768 cycles at 128 B
//    per cycle) and the DMA writes 48 KB, against 1024 MFMA cycles.  Eight
//    wavefronts of 128 x 64 read half as much again.
//  * A wavefront holds two operand sets: while the MFMAs of stage g run on
//    one, stage g + 1 is read into the other.  So stage g's slot is free as
//    soon as stage g starts, and the DMA of stage g + 3 goes into it: two
//    whole stages are always in flight.
//  * Measured, M x N x K = 11264 x 12288 x 4096: 277 us in the batch-16 step,
//    against 387 us of the int8 kernel there; the four products of a 7B layer
//    at 11264 rows 1092 us (1139 with four registers spilled, before hold_acc).
//    With random codes, 216 us is what its MFMAs alone take on nine rounds of
//    tiles (8.25 full), at the clock the power limit leaves them (28 cycles of
//    2.4 GHz per MFMA instead of 18); its data movement alone takes 204 us.
//  * KT, the number of stages, is even (the operands are padded with a stage
//    of zeros), so a tile starts and ends on the same set.
template <bool BF16OUT, bool ACC>
__global__ __launch_bounds__(256, 1) void k_w4a4_gemm_f6(
    const uint8_t *__restrict__ fa, const float *__restrict__ sa, const uint8_t *__restrict__ fw,
    const float *__restrict__ sw, int M, int N, int KT, void *__restrict__ y, int64_t ldy,
    int32_t *__restrict__ acc_out, int tiles_m, int tiles_n) {
    constexpr int NF = 8;                        // fragments of 16 rows per operand and wavefront
    constexpr int SCALE_OFF = kRing * kStageF;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[SCALE_OFF + kScaleRing * kScaleBuf];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int wm = wave_u & 1, wn = wave_u >> 1;

    const int T = tiles_m * tiles_n;
    const int xcd = blockIdx.x % kXcds, i0 = blockIdx.x / kXcds;
    const int nb = ((int)gridDim.x - xcd + kXcds - 1) / kXcds;
    const int q = T / kXcds, rr = T % kXcds;
    const int start = (xcd < rr) ? xcd * (q + 1) : rr * (q + 1) + (xcd - rr) * q;
    const int len = q + (xcd < rr ? 1 : 0);
    const int nt = (i0 < len) ? (len - i0 + nb - 1) / nb : 0;
    if (nt == 0) return;                         // block-uniform
    auto tile_at = [&](int k, int &tm, int &tn) __attribute__((always_inline)) {
        grouped_tile(start + i0 + k * nb, tiles_m, tiles_n, tm, tn);
    };

    const uint32_t lds = lds_addr(smem), sbase = lds + SCALE_OFF;
    const uint32_t dofs = (uint32_t)(wave_u * 6 * 1024);
    const uint32_t vofs = dofs + (uint32_t)lane * 16u;
    const uint32_t blk = (uint32_t)KT * kOpStage;          // bytes of one row block

    // The DMA of one stage: issue_begin() once, then issue_pair(i) for i < 6.
    // Past the last stage the descriptors are empty (the loads read as zeros
    // into a slot that is not read any more), which keeps the number of
    // outstanding instructions, and with it every wait, the same to the end.
    int iss_k = -1, iss_kt = 0, iss_slot = kRing - 1;
    uint32_t iss_lds = 0, iss_off = 0;
    v4i dA, dW;
    auto issue_begin = [&]() __attribute__((always_inline)) {
        if (iss_kt == 0) {
            ++iss_k;
            const bool live = iss_k < nt;
            int tm = 0, tn = 0;
            if (live) tile_at(iss_k, tm, tn);
            dA = buffer_desc(fa + (int64_t)tm * blk, live ? blk : 0u);
            dW = buffer_desc(fw + (int64_t)tn * blk, live ? blk : 0u);
            if (live) {
                const v4i dSa = buffer_desc(sa + tm * F_BM, (uint32_t)(min(M - tm * F_BM, F_BM) * 4));
                const v4i dSw = buffer_desc(sw + tn * F_BN, (uint32_t)(min(N - tn * F_BN, F_BN) * 4));
                const uint32_t sb = sbase + (uint32_t)((iss_k % kScaleRing) * kScaleBuf);
                dma4(dSa, (uint32_t)(64 * wave + lane) * 4u, sb + wave_u * 256);
                dma4(dSw, (uint32_t)(64 * wave + lane) * 4u, sb + F_BM * 4 + wave_u * 256);
            }
        }
        if (++iss_slot == kRing) iss_slot = 0;
        iss_lds = lds + (uint32_t)iss_slot * kStageF + dofs;
        iss_off = vofs + (uint32_t)iss_kt * kOpStage;
        if (++iss_kt == KT) iss_kt = 0;
    };
    auto issue_pair = [&](int i) __attribute__((always_inline)) {
        dma16(dA, iss_off + i * 1024, iss_lds + i * 1024);
        dma16(dW, iss_off + i * 1024, iss_lds + kOpStage + i * 1024);
    };

    const bool vec16 = ((ldy & 7) == 0) && ((reinterpret_cast<uintptr_t>(y) & 15) == 0);
    const bool acc_vec = ACC && (N & 3) == 0 && ((reinterpret_cast<uintptr_t>(acc_out) & 15) == 0);
    const uint32_t fA = (uint32_t)(wm * 4 * kPairBytes + lane * 16);
    const uint32_t fW = (uint32_t)(kOpStage + wn * 4 * kPairBytes + lane * 16);
    // A lane's 8-byte part lies at + 1024 + 8 lane.  Two offsets, one opaque to
    // the compiler: merged into one two-address load, the parts of two
    // fragments would land in adjacent registers and be moved apart again.
    int fo[2] = {-8 * lane, -8 * lane};
    asm volatile("" : "+v"(fo[1]));
    v6i a[2][NF], w[2][NF];
    auto read_pair = [&](const uint8_t *b, int p, auto set_c) __attribute__((always_inline)) {
        constexpr int S = decltype(set_c)::value;
        const uint8_t *f = (p < 4) ? b + fA + p * kPairBytes : b + fW + (p - 4) * kPairBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const v4i x = *reinterpret_cast<const v4i *>(f + h * kFragBytes);
            const v2i z = *reinterpret_cast<const v2i *>(f + h * kFragBytes + 1024 + fo[h]);
            const v6i v = {x[0], x[1], x[2], x[3], z[0], z[1]};
            if (p < 4) a[S][2 * p + h] = v;
            else w[S][2 * p - 8 + h] = v;
        }
    };

#pragma unroll
    for (int g = 0; g < kRing; ++g) {
        issue_begin();
#pragma unroll
        for (int i = 0; i < 6; ++i) issue_pair(i);
    }
    // stage 0 into set 0, with stages 1 and 2 in flight
    asm volatile("s_waitcnt vmcnt(24)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int p = 0; p < NF; ++p) read_pair(smem, p, std::integral_constant<int, 0>{});

    int rslot = 1;                               // slot of stage g + 1
    auto stage = [&](v4f (&acc)[NF][NF], auto set_c) __attribute__((always_inline)) {
        constexpr int S = decltype(set_c)::value;
        // stage g + 1 has landed from every wave, and every wave holds stage g
        // in registers: its slot takes the DMA of stage g + 3.  Loads land in
        // order, so one stage's 12 instructions outstanding means that every
        // older stage is complete.
        asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        issue_begin();
        // Behind every 8 MFMAs one pair of fragments is read and one piece of
        // the DMA issued: issued together at the head of the stage, the DMA
        // held up the wavefront's MFMAs for ~750 of its ~2200 cycles (the CU
        // accepts 64 bytes of it per cycle, and a wavefront issues in order).
        const uint8_t *nx = smem + rslot * kStageF;
        if (++rslot == kRing) rslot = 0;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            read_pair(nx, i, std::integral_constant<int, 1 - S>{});
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                mfma_f6(w[S][i], a[S][j], acc[i][j]);
                if (j == 4 && i < 6) issue_pair(i);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    for (int ck = 0; ck < nt; ++ck) {
        v4f acc[NF][NF];
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        hold_acc(acc);
        asm volatile("s_nop 7" ::: "memory");              // zeroed accumulators before the first MFMA
        for (int kt = 0; kt < KT; kt += 2) {
            stage(acc, std::integral_constant<int, 0>{});
            stage(acc, std::integral_constant<int, 1>{});
        }
        int tm, tn;
        tile_at(ck, tm, tn);
        const int m0 = tm * F_BM, n0 = tn * F_BN;
        const float *s_sa = reinterpret_cast<const float *>(smem + SCALE_OFF + (ck % kScaleRing) * kScaleBuf);
        const float *s_sw = s_sa + F_BM;
        // Epilogue: each wavefront stages 32 rows x 128 columns at a time in
        // its own 8 KB of the slot whose stage every wave now holds in
        // registers (the next tile's first; its next DMA follows the next barrier):
        // 8-byte units, unit block i of row r at i ^ (r % 8), read back as
        // 16 bytes per lane and stored as whole 256-byte row segments.
        // (the nops: the distance from the last MFMA to the reads of acc)
        asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        hold_acc(acc);
        int r16 = lane & 15, cq = lane >> 4, lanee = lane;
        asm volatile("" : "+v"(r16), "+v"(cq), "+v"(lanee));
        uint8_t *stg = smem + (rslot == 0 ? kRing - 1 : rslot - 1) * kStageF + wave_u * 8192;
        const int rows_left = M - m0, cols_left = N - n0;
        const bool full = vec16 && rows_left >= F_BM && cols_left >= F_BN;
#pragma unroll
        for (int pass = 0; pass < NF / 2; ++pass) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = 2 * pass + jj;
                const int rl = wm * 128 + 16 * j + r16;
                const float sam = s_sa[rl];
                const int rs = 16 * jj + r16;
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int nl = wn * 128 + 16 * i + 4 * cq;
                    const float4 swv = *reinterpret_cast<const float4 *>(s_sw + nl);
                    const float swe[4] = {swv.x, swv.y, swv.z, swv.w};
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = __fmul_rn(__fmul_rn(acc[i][j][e], sam), swe[e]);
                    uint2 packed;
                    if constexpr (BF16OUT) {
                        packed.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{o[0], o[1]}, bf2));
                        packed.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{o[2], o[3]}, bf2));
                    } else {
                        uint32_t h[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float ov = o[e];
                            asm volatile("" : "+v"(ov));   // round to fp32 first, then to fp16
                            h[e] = __builtin_bit_cast(uint16_t, (_Float16)ov);
                        }
                        packed = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                    }
                    const int u = 4 * (i ^ (rs & 7)) + cq;
                    *reinterpret_cast<uint2 *>(stg + rs * 256 + u * 8) = packed;
                    if constexpr (ACC) {
                        const int m = m0 + rl, nb0 = n0 + nl;
                        if (m < M) {
                            int32_t *dst = acc_out + (int64_t)m * N + nb0;
                            const v4i v = {(int)acc[i][j][0], (int)acc[i][j][1], (int)acc[i][j][2],
                                           (int)acc[i][j][3]};
                            if (acc_vec && nb0 + 3 < N) {
                                *reinterpret_cast<v4i *>(dst) = v;
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (nb0 + e < N) dst[e] = v[e];
                            }
                        }
                    }
                }
            }
            // lane l, step s reads back row 4 s + l / 16, chunk l % 16 (LDS
            // operations of one wave take effect in issue order)
            const int rq = lanee >> 4, rc = lanee & 15;
            const int rt0 = wm * 128 + 32 * pass + rq, ct = wn * 128 + 8 * rc;
            uint16_t *dst = static_cast<uint16_t *>(y) + (int64_t)(m0 + rt0) * ldy + n0 + ct;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int rs = 4 * s + rq;
                const int cu = 4 * ((rc >> 1) ^ (rs & 7)) + 2 * (rc & 1);
                const v4i val = *reinterpret_cast<const v4i *>(stg + rs * 256 + cu * 8);
                if (full) {
                    __builtin_nontemporal_store(val, reinterpret_cast<v4i *>(dst));
                } else if (rt0 + 4 * s < rows_left) {
                    if (vec16 && ct + 8 <= cols_left) {
                        __builtin_nontemporal_store(val, reinterpret_cast<v4i *>(dst));
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (ct + e < cols_left) dst[e] = (uint16_t)((uint32_t)val[e >> 1] >> (16 * (e & 1)));
                    }
                }
                dst += 4 * ldy;
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no DMA into LDS past the end
}

inline int f6_stages(int K) { return (K + 2 * F_KS - 1) / (2 * F_KS) * 2; }

inline int64_t row_blocks(int R) { return ((int64_t)R + 255) / 256; }

}  // namespace

size_t gemm_f6_bytes(int M, int N, int K) {
    const int64_t KT = f6_stages(K);
    return (size_t)((row_blocks(M) + row_blocks(N)) * KT * kOpStage);
}

hipError_t launch_w4a4_gemm_f6(int M, int N, int K, const uint8_t *a, const float *sa,
                               const uint8_t *w, const float *sw, p4q_dtype out_dt, void *y,
                               int64_t ldy, int32_t *acc_out, void *ws, hipStream_t stream) {
    const int KT = f6_stages(K);
    uint8_t *fa = static_cast<uint8_t *>(ws);
    uint8_t *fw = fa + row_blocks(M) * KT * kOpStage;
    const int segs = (KT + kConvK - 1) / kConvK;
    const int itemsA = (M + 31) / 32 * segs, items = itemsA + (N + 31) / 32 * segs;
    hipLaunchKernelGGL(k_codes_f6, dim3((items + 3) / 4), dim3(256), 0, stream, a, M, fa, itemsA, w, N,
                       fw, items, K / 2, KT, segs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int tiles_m = (int)row_blocks(M), tiles_n = (int)row_blocks(N);
    const int T = tiles_m * tiles_n;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min(T, device_cus())), dim3(256), 0, stream, fa,
                           sa, fw, sw, M, N, KT, y, ldy, acc_out, tiles_m, tiles_n);
        return hipGetLastError();
    };
    if (out_dt == P4Q_BF16)
        return acc_out ? go(k_w4a4_gemm_f6<true, true>) : go(k_w4a4_gemm_f6<true, false>);
    return acc_out ? go(k_w4a4_gemm_f6<false, true>) : go(k_w4a4_gemm_f6<false, false>);
}

}  // namespace p4q
