// Attention prefill on the pruned sequence with FP16 (or BF16) Q, K, V --
// the decoder step after the q/k/v linears (P4Q Appendix B.3: W4A4 with the
// key and value caches kept in FP16):
//     O[t, h] = sum_j softmax_j(<q_t, k_j> / sqrt(D)) v_j,  j <= t when causal.
//
// One work-group of 4 wavefronts per (128 queries, head, sample); each
// wavefront owns 32 queries and walks the key tiles of 64 keys:
//  * S^T = K Q^T on v_mfma_f32_32x32x16 (K from LDS, Q^T held in registers):
//    lane l ends up with query l%32 and 16 keys of each 32-key half, so the
//    softmax statistics of a query need its registers and one exchange with
//    lane l^32;
//  * online softmax in fp32 with exp2 (log2(e)/sqrt(D) folded in); the
//    running maximum is raised only when a tile exceeds it by more than 2^8
//    in exp2 units, so the output accumulators are rescaled rarely (the
//    weights stay below 2^8, well inside the 16-bit range);
//  * O^T += V^T P^T: P^T is the softmax of S^T converted to 16 bits, used as
//    the MFMA's B operand straight from the S^T registers.  The key order it
//    implies (register r of lane group g holds key 8(r/4) + 4g + r%4 of a
//    32-key half) is the one in which the transposing LDS reads
//    (ds_read_b64_tr_b16) fetch V^T from V as it lies in memory: a 16-lane
//    group reads 4 keys x 16 d, and lane j gets the four keys of d = j.
//  * K and V tiles go straight to LDS (buffer_load ... lds; rows past L read
//    as zeros), two buffers, the next tile's loads issued in pieces between
//    the steps of the current one; one barrier per tile.
//  * Operand reads are issued ahead of the MFMAs that use them (the first K
//    steps, and V's first half before the softmax): left to itself the
//    compiler reads each operand just before its MFMA and waits out the LDS
//    latency 32 times per tile.
//  * Work-groups of one (sample, head) are neighbours on one XCD, longest
//    first, so K and V come from its L2 after the first of them.
// At 16 x 704 tokens and 32 heads a call takes 123 us (the kernel 121),
// against 166 us for the form that staged K and V^T through registers, read
// operands as needed and masked through a branch per score; one sample of 371
// tokens, 40 heads: 13.0 (12.6) against 16.6 us.  Per SIMD its vector instructions take 39 us, its MFMAs 28
// us; q, k, v and the output take 73 us at the rate of a copy.  Reading Q
// and writing the output of 128 queries alone (no tiles) takes 42 us, each
// tile of the two work-groups on a CU 2 us, most of it waiting: two
// wavefronts per SIMD (224 registers, 64 KB of LDS per work-group) do not
// cover the chain S^T -> maximum -> exp2 -> P V.  Work-groups of two
// wavefronts: 172 us; neighbouring samples instead of neighbouring query
// tiles on an XCD: 148 us.
// Output layout of the 32x32 MFMA: register r of lane l holds row
// 8(r/4) + 4(l/32) + r%4, column l%32.
#include "gemm_device.h"
#include "p4q_internal.h"

#include <algorithm>
#include <type_traits>

namespace p4q {
namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s *lds_v4s_t;

constexpr int kD = 128;                 // head dimension
constexpr int kNW = 4;                  // wavefronts per work-group
constexpr int kQW = 32;                 // queries per wavefront
constexpr int kQB = kNW * kQW;          // queries per work-group
constexpr int kKT = 64;                 // keys per tile
constexpr int kRow = kD * 2;            // bytes of a K or V row
constexpr int kOperand = kKT * kRow;    // 16 KB
constexpr int kTile = 2 * kOperand;     // K, then V
constexpr float kRescale = 8.0f;        // raise the running max past this margin (exp2 units)

// LDS placement of 16-byte chunk c of row r.  K: the rows that a fragment
// read takes together (16 of them, one chunk) fall in distinct banks; V: the
// four keys of a transposing read (64-byte pieces) fall in distinct banks.
__device__ __forceinline__ int k_slot(int r, int c) { return c ^ (r & 15); }
__device__ __forceinline__ int v_slot(int r, int c) { return c ^ ((r & 3) << 2); }

template <bool BF16>
__device__ __forceinline__ v16f mfma(uint4 a, uint4 b, v16f c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}

// two fp32 -> two 16-bit values (nearest, ties to even), low half first
template <bool BF16>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    if constexpr (BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2bf));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2h));
}

// the same of lo * c and hi * c.  In fp16 the product is rounded once, straight
// to 16 bits (v_fma_mixlo_f16), which takes a conversion of its own for each: the
// packed one is handed products that are already rounded to fp32.
template <bool BF16>
__device__ __forceinline__ uint32_t pack2_scaled(float lo, float hi, float c) {
    if constexpr (BF16) return pack2<true>(lo * c, hi * c);
    else {
        const _Float16 a = (_Float16)(lo * c), b = (_Float16)(hi * c);
        return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
    }
}

template <bool BF16, bool CAUSAL>
__global__ __launch_bounds__(64 * kNW, 2) void k_attention(const uint16_t *__restrict__ q,
                                                          const uint16_t *__restrict__ k,
                                                          const uint16_t *__restrict__ v, int64_t ld,
                                                          int L, int H, uint16_t *__restrict__ o,
                                                          int64_t ldo, float c2, int total) {
    constexpr int NI = 16 / kNW;            // 1 KB DMA instructions per operand and wavefront
    __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * kTile];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, c32 = lane & 31;
    const int nqt = (L + kQB - 1) / kQB;
    const int wg = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (wg >= total) return;
    const int logical = xcd_logical(wg, total);
    const int bh = logical / nqt, qi = logical - bh * nqt;
    const int qt = CAUSAL ? nqt - 1 - qi : qi;             // longest (causal) first
    const int b = bh / H, h = bh - b * H;
    const int q0 = qt * kQB;
    const int64_t base = (int64_t)b * L * ld + (int64_t)h * kD;

    const int qw0 = q0 + kQW * wave;                       // first query of the wavefront
    const int tq = qw0 + c32;                              // this lane's query

    // DMA of a tile: instruction n of a wavefront fills rows 4 (NI wave + n)
    // + lane / 16 of the operand; slot lane % 16 takes the chunk that k_slot /
    // v_slot place there (both are their own inverses).  Offsets have 32 bits:
    // L ld2 < 2^31, but (with L <= 62 and rows of many MB) not 63 ld2, so rows past
    // L of the first tile get an offset past any span.  Those of a later tile lie
    // below 2 L ld2.
    const uint32_t span = (uint32_t)((int64_t)L * ld * 2);
    const v4i dK = buffer_desc(k + base, span), dV = buffer_desc(v + base, span);
    const uint32_t ld2 = (uint32_t)(ld * 2);
    const int drow = 4 * NI * wave + (lane >> 4);
    uint32_t vok[NI], vov[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int r = drow + 4 * n;
        const uint32_t row = r < L ? (uint32_t)r * ld2 : 0x80000000u;
        vok[n] = row + 16u * (uint32_t)k_slot(r, lane & 15);
        vov[n] = row + 16u * (uint32_t)v_slot(r, lane & 15);
    }
    const uint32_t lds0 = lds_addr(smem) + (uint32_t)(wave * NI * 1024);
    // (no tile kt: empty descriptors, nothing is read)
    const int kend = CAUSAL ? min(L, q0 + kQB) : L;
    const int ntiles = (kend + kKT - 1) / kKT;
    auto issue = [&](bool isv, int kt, int n0, int n1) __attribute__((always_inline)) {
        v4i d = isv ? dV : dK;
        d[2] = (kt < ntiles) ? d[2] : 0;
#pragma unroll
        for (int n = n0; n < n1; ++n)
            dma16(d, (isv ? vov[n] : vok[n]) + (uint32_t)(kt * kKT) * ld2,
                  lds0 + (kt & 1) * kTile + (isv ? kOperand : 0) + n * 1024);
    };

    issue(false, 0, 0, NI);
    issue(true, 0, 0, NI);
    // The query's Q^T operands (8 k-steps of 16 d; a query past L takes the
    // last row's, its output is not stored).  The wait for them is placed here,
    // behind the first tile's loads: one that the compiler puts inside the loop
    // would also wait for the next tile's, which it cannot tell apart.
    uint4 qf[8];
    const uint16_t *qrow = q + base + (int64_t)min(tq, L - 1) * ld + 8 * g;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const uint4 *>(qrow + 16 * s);
#pragma unroll
    for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[s].x), "+v"(qf[s].y), "+v"(qf[s].z), "+v"(qf[s].w));

    v16f acc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db) acc[db] = v16f{};
    float m = -__builtin_huge_valf(), lsum = 0.0f;

    // lanes l and l ^ 32 hold the two halves of a query's keys: their
    // combination through a permlane swap (no LDS round trip)
    auto xmax32 = [](float x) __attribute__((always_inline)) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return __builtin_fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    };
    auto xsum32 = [](float x) __attribute__((always_inline)) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    };
    // K fragment addresses: row 32 hf + c32 (its k_slot depends on c32 only)
    const uint32_t kofs = (uint32_t)(c32 * kRow);
    const uint32_t kx = (uint32_t)(c32 & 15);
    // V^T: lane reads 8 bytes of key 16 s + 8 e + 4 g + (lane % 16) / 4, d =
    // 32 db + 16 ((lane / 16) % 2) + 4 (lane % 4)
    const int vkey = 4 * g + ((lane & 15) >> 2);
    const uint32_t vofs = (uint32_t)(kOperand + vkey * kRow + 8 * (lane & 1));
    const uint32_t vc = (uint32_t)(2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)), vx = (uint32_t)((vkey & 3) << 2);

    // One tile of 64 keys from LDS buffer kt & 1, both 32-key halves at once:
    // their S^T products are two independent MFMA chains, and one softmax
    // update (one max, one rescale decision, one sum) covers the 64 keys.
    // NH = 1: only the first half has keys at or before this wavefront's last
    // query (causal diagonal); the second is skipped, since weights of 0 would
    // still turn a non-finite row of V into NaN.  The next tile's loads are
    // issued on the way.
    auto tile_keys = [&](int kt, auto nh_c) __attribute__((always_inline)) {
        constexpr int NH = decltype(nh_c)::value;
        const uint8_t *sb = smem + (kt & 1) * kTile;
        const int k0 = kt * kKT;
        auto k_read = [&](int hf, int s) __attribute__((always_inline)) {
            return *reinterpret_cast<const uint4 *>(sb + 32 * hf * kRow + kofs + 16u * ((uint32_t)(2 * s + g) ^ kx));
        };
        auto v_read = [&](int db, int s) __attribute__((always_inline)) {
            const uint8_t *p = sb + vofs + 16 * s * kRow + 16u * ((uint32_t)(4 * db) + vc ^ vx);
            const v4s x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t)(p));
            const v4s y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t)(p + 8 * kRow));
            const uint2 a = __builtin_bit_cast(uint2, x), c = __builtin_bit_cast(uint2, y);
            return make_uint4(a.x, a.y, c.x, c.y);
        };
        // S^T = K Q^T: lane holds query c32, keys k0 + 32 hf + 8(r/4) + 4g + r%4
        v16f st[NH];
#pragma unroll
        for (int hf = 0; hf < NH; ++hf) st[hf] = v16f{};
        // K steps in batches of two, read two batches ahead
        uint4 kf[2][2][NH];
        auto k_batch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) kf[i & 1][j][hf] = k_read(hf, 2 * i + j);
        };
        k_batch(0);
        k_batch(1);
        issue(false, kt + 1, 0, NI);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) st[hf] = mfma<BF16>(kf[i & 1][j][hf], qf[2 * i + j], st[hf]);
            if (i + 2 < 4) k_batch(i + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        // V^T of d 0..63: in flight during the softmax
        uint4 vf[2][2 * NH];
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int s = 0; s < 2 * NH; ++s) vf[db][s] = v_read(db, s);
        issue(true, kt + 1, 0, NI);
        __builtin_amdgcn_sched_barrier(0);
        // mask (only where the tile reaches the diagonal or the end; one
        // wave-uniform branch)
        if (k0 + 32 * NH > L || (CAUSAL && k0 + 32 * NH - 1 > qw0)) {
#pragma unroll
            for (int hf = 0; hf < NH; ++hf)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kk = k0 + 32 * hf + 8 * (r >> 2) + 4 * g + (r & 3);
                    const bool ok = (kk < L) & (!CAUSAL | (kk <= tq));
                    st[hf][r] = ok ? st[hf][r] : -__builtin_huge_valf();
                }
        }
        float tmax = -__builtin_huge_valf();
#pragma unroll
        for (int hf = 0; hf < NH; ++hf)
#pragma unroll
            for (int r = 0; r < 16; ++r) tmax = __builtin_fmaxf(tmax, st[hf][r]);
        tmax = xmax32(tmax);
        // raise the running max only past the margin (wave-uniform rescale)
        const bool raise = (tmax - m) * c2 > kRescale || m == -__builtin_huge_valf();
        if (__any((int)raise)) {
            const float mnew = raise ? tmax : m;
            const float mref = (mnew == -__builtin_huge_valf()) ? 0.0f : mnew;
            const float alpha = (m == -__builtin_huge_valf()) ? 0.0f : __builtin_amdgcn_exp2f((m - mref) * c2);
            m = mnew;
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
        }
        const float mc = (m == -__builtin_huge_valf()) ? 0.0f : m * c2;
        float psum = 0.0f;
        uint4 pb[NH][2];
#pragma unroll
        for (int hf = 0; hf < NH; ++hf) {
            uint32_t pw[8];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[hf][r], c2, -mc));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[hf][r + 1], c2, -mc));
                psum += p0 + p1;
                pw[r >> 1] = pack2<BF16>(p0, p1);
            }
            pb[hf][0] = make_uint4(pw[0], pw[1], pw[2], pw[3]);
            pb[hf][1] = make_uint4(pw[4], pw[5], pw[6], pw[7]);
        }
        lsum += xsum32(psum);
        __builtin_amdgcn_sched_barrier(0);
        // O^T += V^T P^T (steps of 16 keys), each d block's operands read two
        // blocks ahead
#pragma unroll
        for (int db = 0; db < 4; ++db) {
#pragma unroll
            for (int s = 0; s < 2 * NH; ++s) acc[db] = mfma<BF16>(vf[db & 1][s], pb[s >> 1][s & 1], acc[db]);
            if (db + 2 < 4)
#pragma unroll
                for (int s = 0; s < 2 * NH; ++s) vf[db & 1][s] = v_read(db + 2, s);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // tiles past this wavefront's last query hold only masked keys: it loads
    // its share of them and keeps the barriers (one per tile either way)
    const int nlive = qw0 >= L ? 0 : CAUSAL ? min(ntiles, (qw0 + kQW - 1) / kKT + 1) : ntiles;
    // tile kt has landed from every wavefront, and every wavefront is done
    // with tile kt - 1, whose buffer the loads of tile kt + 1 overwrite
    auto arrive = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); };
    // a wavefront whose queries are the first half of its last tile's keys
    const bool half = CAUSAL && nlive > 0 && (qw0 & (kKT - 1)) == 0;
    int kt = 0;
    for (; kt < nlive - (int)half; ++kt) {
        arrive();
        tile_keys(kt, std::integral_constant<int, 2>{});
    }
    if (half) {
        arrive();
        tile_keys(kt, std::integral_constant<int, 1>{});
        ++kt;
    }
    for (; kt < ntiles; ++kt) {
        arrive();
        issue(false, kt + 1, 0, NI);
        issue(true, kt + 1, 0, NI);
    }

    // O[tq][d] = acc / lsum; register r of d-block db holds d = 32 db + 8(r/4) +
    // 4g + r%4.  The wavefront's 32 rows pass through 8 KB of LDS (8-byte unit
    // u of row r at u ^ 2 (r % 16)) and leave as whole 256-byte rows.
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // every wavefront is done with the tiles
    const float inv = 1.0f / lsum;
    uint8_t *stg = smem + wave * (kQW * kRow);
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int u = 8 * db + 2 * j + g;
            const uint2 w = make_uint2(pack2_scaled<BF16>(acc[db][4 * j], acc[db][4 * j + 1], inv),
                                       pack2_scaled<BF16>(acc[db][4 * j + 2], acc[db][4 * j + 3], inv));
            *reinterpret_cast<uint2 *>(stg + c32 * kRow + 8 * (u ^ ((c32 & 15) << 1))) = w;
        }
    const bool vec16 = (ldo & 7) == 0 && (reinterpret_cast<uintptr_t>(o) & 15) == 0;
    uint16_t *ob = o + (int64_t)b * L * ldo + (int64_t)h * kD + 8 * (lane & 15);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int r = 4 * s + (lane >> 4), t = qw0 + r;
        const uint4 w = *reinterpret_cast<const uint4 *>(stg + r * kRow + 16 * ((lane & 15) ^ (r & 15)));
        if (t < L) {
            uint16_t *dst = ob + (int64_t)t * ldo;
            if (vec16) {
                __builtin_nontemporal_store(__builtin_bit_cast(v4i, w), reinterpret_cast<v4i *>(dst));
            } else {
                *reinterpret_cast<uint2 *>(dst) = make_uint2(w.x, w.y);
                *reinterpret_cast<uint2 *>(dst + 4) = make_uint2(w.z, w.w);
            }
        }
    }
}

}  // namespace

hipError_t launch_attention(p4q_dtype dt, int B, int L, int H, const void *q, const void *k,
                            const void *v, int64_t ld, void *o, int64_t ldo, int causal,
                            hipStream_t stream) {
    const float c2 = 1.4426950408889634f / __builtin_sqrtf((float)kD);   // log2(e) / sqrt(D)
    const uint16_t *qq = static_cast<const uint16_t *>(q), *kk = static_cast<const uint16_t *>(k),
                   *vv = static_cast<const uint16_t *>(v);
    uint16_t *oo = static_cast<uint16_t *>(o);
    auto go = [&](auto kern) {
        // a launch dimension holds fewer than 2^32 threads: many very short
        // samples wrap into the second one
        const int64_t total = (int64_t)B * H * ((L + kQB - 1) / kQB), wrap = 1 << 20;
        if (total > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
        const dim3 grid((unsigned)std::min(total, wrap), (unsigned)((total + wrap - 1) / wrap));
        hipLaunchKernelGGL(kern, grid, dim3(64 * kNW), 0, stream, qq, kk, vv, ld, L, H, oo, ldo, c2,
                           (int)total);
        return hipGetLastError();
    };
    if (dt == P4Q_BF16) return causal ? go(k_attention<true, true>) : go(k_attention<true, false>);
    return causal ? go(k_attention<false, true>) : go(k_attention<false, false>);
}

}  // namespace p4q
