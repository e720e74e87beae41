// Loop 3 of Algorithm 1 (Lavin & Gray): the alpha^2 independent products
// M^(xi,nu) = U^(xi,nu) V^(xi,nu) (Eq. (13)), K x C by C x P each, on the MFMA units.
#include <stdlib.h>

#include "wino_internal.h"
#include "bf16x3.h"

namespace wino {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Maps the hardware workgroup id to a logical block id so that logically consecutive blocks run
// on the same XCD.  Workgroups are dealt to the 8 XCDs round-robin (id % 8) and each XCD has
// its own L2; consecutive logical blocks share an operand panel, so they should share an L2.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks)
{
    constexpr int XCDS = 8;
    const int per = nblocks / XCDS;            // blocks in the evenly divisible part
    if (bid >= per * XCDS) return bid;         // ragged remainder keeps its id
    return (bid % XCDS) * per + bid / XCDS;
}

// fp32 operands on the bf16 matrix units (bf16x3.h: every value in three exact parts, six products, fp32 sums).
// A workgroup of four wavefronts (2 x 2) owns a BM x BN block of one M^(e); every wavefront TM x TN tiles of 32 x 32.
// Both operands are stored reduction-index-major (U[e][c][k], V[e][c][b]); the matrix instruction wants eight
// channels of one row per lane.  So a thread fetches eight channels of one column with eight 4-byte loads (each 256
// contiguous bytes per wavefront, which the vector memory path takes at the same 64 bytes per cycle as wider ones),
// splits them once and stores the parts as 16-byte words [channels / 8][part][column]: LDS accesses are contiguous
// both ways, and the values that two wavefronts share are split only once.
//
// Pipeline: two slabs of BK channels in flight in registers, two slabs in LDS, one barrier per slab (which orders LDS
// traffic only: requests stay in flight across it).  While a slab is multiplied, the next one is split.
//
// Blocks that overhang Kp or Pp load from clamped (valid) addresses: rows/columns of a product are independent, so
// whatever is loaded there only reaches outputs that are never stored.  Channels past the end of this share lie
// behind the buffers' ends and read as 0.
//
// What bounds it is energy: on N(0,1) data back-to-back v_mfma_f32_32x32x16_bf16 alone pull the clock from 2.4 to
// 1.77 GHz (18.7 ns each per SIMD); four vector instructions, half an LDS read and a quarter of an LDS store beside
// each make it 25 ns, this kernel runs at 30 (matrix pipes 60 % busy).  36 products of 256 x 256 by 256 x 12544:
// 118 TFLOP/s with v_mfma_f32_32x32x2_f32 (501 us), 184 so (320 us); 512 -> 512 channels at 28 x 28, batch 8: multiply
// 83 -> 53 us.  Single-buffered slabs of 32 channels on v_mfma_f32_16x16x32_bf16, which takes an eighth less energy,
// but with two barriers and no split between the matrix instructions: 355 us (matrix pipes 46 % busy).  (Operands were
// split as they are then.  The multiplication by 2^24, for the whole range of fp32, costs 4 %: the same 36 products on
// another box 364 -> 377 us, 479 with fp32 instructions; that layer 84.1 -> 86.7 us.)
__device__ __forceinline__ void gemm_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Byte offset of a float in a buffer of less than 4 GiB; what lies behind 4 GiB stays there (rows past the last channel).
__device__ __forceinline__ unsigned gemm_offset(unsigned long long floats)
{
    return floats < 0x3fffffffull ? (unsigned)floats * 4u : 0xffffffffu;
}

// ONE: the share is one slab.  Then there is nothing to overlap within a workgroup and what bounds the launch is writing
// M: no second slab, half the LDS, twice the workgroups per CU, and no matrix instructions for the empty half of a
// slab (64 products of 32 x 16 by 16 x 3600: layer 32.8 -> 30.3 us).
// LONG: the share is longer than BF16_LONG channels, so its sums are set aside now and then (bf16x3.h), where M will be.
enum { ONE, USUAL, LONG };
template <int BM, int BN, int BK, int DEPTH>
__global__ __launch_bounds__(256, DEPTH == ONE && BM * BN < 128 * 128 ? 4 : 2) void gemm_f32_kernel(
    const float *__restrict__ U, const float *__restrict__ V, float *__restrict__ Mo, int Kp, int Cp, int Pp, int tiles_m,
    int tiles_n, int a2, int c_share, int c_real)
{
    constexpr int TM = BM / 64, TN = BN / 64;
    constexpr int G8 = BK / 8;                                   // groups of eight channels per slab
    constexpr int AG = G8 * BM / 256, BG = G8 * BN / 256;        // groups a thread fetches
    static_assert(G8 * BM % 256 == 0 && G8 * BN % 256 == 0 && BK % 16 == 0, "a slab divides evenly among the threads");
    __shared__ uintx4_b As[DEPTH == ONE ? 1 : 2][G8 * 3 * BM];
    __shared__ uintx4_b Bs[DEPTH == ONE ? 1 : 2][G8 * 3 * BN];

    int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int tm_i = bid % tiles_m;
    bid /= tiles_m;
    const int tn_i = bid % tiles_n;
    bid /= tiles_n;
    const int e = bid % a2;
    const int z = bid / a2;   // which share of the channel loop (layers with few blocks split it)
    const int k0 = tm_i * BM, p0 = tn_i * BN;
    const int c_first = z * c_share, c_rows = min(c_share, Cp - c_first);
    const int nk = (c_rows + BK - 1) / BK;      // slabs, >= 1 by construction of the launch

    const float *Ue = U + ((size_t)e * Cp + c_first) * Kp;
    const float *Ve = V + ((size_t)e * Cp + c_first) * Pp;
    float *Me = Mo + ((size_t)z * a2 + e) * Kp * Pp;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lh = lane >> 5;

    // Operands are fetched through buffers that hold this share's channel rows of U^(e) and V^(e) (one component's
    // Cp x Kp or Cp x Pp floats stay below 4 GB: see the launcher).  A group of eight rows lies inside the buffer or
    // behind it as a whole, and its vector offset alone tells which: sums of offsets saturate, they must not wrap around
    // into the buffer.
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void *)Ue, 0, (unsigned)((size_t)c_rows * Kp * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void *)Ve, 0, (unsigned)((size_t)c_rows * Pp * 4), 0x00020000);
    unsigned oa[AG], ob[BG];
#pragma unroll
    for (int j = 0; j < AG; ++j) {
        const int id = tid + j * 256;
        oa[j] = gemm_offset((unsigned long long)(id / BM * 8) * Kp + min(k0 + id % BM, Kp - 1));
    }
#pragma unroll
    for (int j = 0; j < BG; ++j) {
        const int id = tid + j * 256;
        ob[j] = gemm_offset((unsigned long long)(id / BN * 8) * Pp + min(p0 + id % BN, Pp - 1));
    }
    float ra[2][AG][8], rb[2][BG][8];
    auto request = [&](int slot, int slab) {
        const unsigned past = slab < nk ? 0u : 0xffffffffu;
        const unsigned sa = (unsigned)(slab * BK) * (unsigned)Kp * 4u | past, sb = (unsigned)(slab * BK) * (unsigned)Pp * 4u | past;
#pragma unroll
        for (int j = 0; j < AG; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                ra[slot][j][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                rsrc_a, __builtin_elementwise_add_sat(oa[j], sa),
                                                                (unsigned)(i * Kp) * 4u, 0));
#pragma unroll
        for (int j = 0; j < BG; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                rb[slot][j][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                rsrc_b, __builtin_elementwise_add_sat(ob[j], sb),
                                                                (unsigned)(i * Pp) * 4u, 0));
    };
    // group id = (channels / 8) * extent + column -> word (channels / 8) * 3 * extent + part * extent + column
    auto store = [&](int slot, int buf) {
        uintx4_b p[3];
#pragma unroll
        for (int j = 0; j < AG; ++j) {
            const int id = tid + j * 256, w = id / BM * 3 * BM + id % BM;
            bf16_split8(ra[slot][j], p, BF16_SCALE);
#pragma unroll
            for (int q = 0; q < 3; ++q) As[buf][w + q * BM] = p[q];
        }
#pragma unroll
        for (int j = 0; j < BG; ++j) {
            const int id = tid + j * 256, w = id / BN * 3 * BN + id % BN;
            bf16_split8(rb[slot][j], p, BF16_SCALE);
#pragma unroll
            for (int q = 0; q < 3; ++q) Bs[buf][w + q * BN] = p[q];
        }
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int a_off = lh * 3 * BM + wm * (TM * 32) + li, b_off = lh * 3 * BN + wn * (TN * 32) + li;
    auto multiply = [&](int buf, int depth = BK / 16) {      // (depth in units of 16 channels, the rest of the slab is zeros)
#pragma unroll
        for (int t = 0; t < BK / 16; ++t) {
            if (t >= depth) break;
            uintx4_b a[3][TM], b[3][TN];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; i < TM; ++i) a[q][i] = As[buf][(t * 6 + q) * BM + a_off + i * 32];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[q][j] = Bs[buf][(t * 6 + q) * BN + b_off + j * 32];
            }
#pragma unroll
            for (int n = 0; n < BF16_PRODUCTS; ++n)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[bf16_part_a(n)][i]),
                                                                            __builtin_bit_cast(bf16x8, b[bf16_part_b(n)][j]),
                                                                            acc[i][j], 0, 0, 0);
        }
    };

    // Accumulator register r of lane (li, lh) is row 8*(r/4) + 4*lh + r%4, column li of its tile; Kp and Pp are multiples of
    // 32, so a 32 x 32 tile is entirely inside or entirely outside.
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int ct = p0 + wn * (TN * 32) + j * 32, rt = k0 + wm * (TM * 32) + i * 32;
                if (ct < Pp && rt < Kp) {
                    float *dst = Me + (size_t)(rt + 4 * lh) * Pp + ct + li;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = f(acc[i][j][r], dst[(size_t)(8 * (r / 4) + (r % 4)) * Pp]);
                }
            }
    };
    // a tile's sums over the first `rows` channels with fp32 instructions
    auto fp32_tile = [&](int i, int j, int rows) {
        const float *a = Ue + min(k0 + wm * (TM * 32) + i * 32 + li, Kp - 1) + (size_t)lh * Kp;
        const float *b = Ve + min(p0 + wn * (TN * 32) + j * 32 + li, Pp - 1) + (size_t)lh * Pp;
        floatx16 sums;
#pragma unroll
        for (int r = 0; r < 16; ++r) sums[r] = 0.0f;
#pragma unroll 8
        for (int c = 0; c < rows; c += 2)
            sums = __builtin_amdgcn_mfma_f32_32x32x2f32(a[(size_t)c * Kp], b[(size_t)c * Pp], sums, 0, 0, 0);
        return sums;
    };

    if (DEPTH == ONE && c_real <= 2) {
        // (one or two products are rounded once that way; their six parts are not always rounded to nearest: 2.5e-8 and
        // 3.1e-8 of the product against 3.5e-8 and 3.3e-8.  From three on the parts are the more precise)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = fp32_tile(i, j, 2);
        each([](float sum, float &m) { return m = sum; });
        return;
    }
    if constexpr (DEPTH == ONE) {
        request(0, 0);
        store(0, 0);
        gemm_lds_barrier();
        multiply(0, c_rows <= 16 ? 1 : BK / 16);
    } else {
    // Requests past the last slab are made all the same (they fetch nothing: every row lies behind the buffers), so
    // that the number of loads in flight does not depend on the path taken.
#pragma unroll
    for (int s = 0; s < 2; ++s) request(s, s);
    store(0, 0);
    gemm_lds_barrier();
    // slab kt sits in LDS buffer kt & 1 and came through register slot kt & 1, both known at compile time.  The order
    // of a trip is laid down, because the compiler would move the requests to where their registers are read: the
    // requests of slab kt + 2 first, then the operand reads, then matrix instructions with the split of slab kt + 1
    // (13 vector instructions per pair of values, four to five per matrix instruction) between them.
    auto slab = [&](int kt, int odd) {
        request(odd, kt + 2);                   // (the slot of slab kt, which is in LDS)
        multiply(odd);
        store(odd ^ 1, odd ^ 1);                // (past the last slab: zeros, read by nobody)
        __builtin_amdgcn_sched_group_barrier(0x2, AG + BG, 0);       // (their offsets)
        __builtin_amdgcn_sched_group_barrier(0x20, 8 * (AG + BG), 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 3 * (TM + TN), 0);
        constexpr int NM = BF16_PRODUCTS * TM * TN * (BK / 16), NV = (52 * (AG + BG) + NM - 1) / NM;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, NV, 0);
            if (BK == 32 && i == NM / 2 - 2) __builtin_amdgcn_sched_group_barrier(0x100, 3 * (TM + TN), 0);
        }
        gemm_lds_barrier();
    };
    int kt = 0;
    for (; kt + 2 < nk; kt += 2) {
        slab(kt, 0);
        slab(kt + 1, 1);
        if (DEPTH == LONG && (kt + 2) % (BF16_RUN / BK) == 0) {
            if (kt + 2 == BF16_RUN / BK)
                each([](float sum, float &m) { m = sum; return 0.0f; });
            else
                each([](float sum, float &m) { m += sum; return 0.0f; });
        }
    }
    // the last slab is multiplied only, and only as deep as it is filled (384 filters, 48 channels, 216 tiles, F(6x6,3x3):
    // layer 33.5 -> 32.1 us; 12 channels of 20 images at 40 x 40, F(2x2,3x3): 31.7 -> 30.0)
    const int depth = c_rows - (nk - 1) * BK <= 16 ? 1 : BK / 16;
    if (kt + 1 < nk) {
        slab(kt, 0);
        multiply(1, depth);
    } else {
        multiply(0, depth);
    }
    }

    if (DEPTH == LONG) each([](float sum, float &m) { return m + sum; });
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float t = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                acc[i][j][r] *= BF16_UNSCALE, acc[i][j][r + 1] *= BF16_UNSCALE;
                t = bf16_look(acc[i][j][r], acc[i][j][r + 1], t);
            }
            if (!__any(!bf16_finite(t))) continue;
            // the sums that are not finite, with fp32 instructions (bf16x3.h)
            const floatx16 exact = fp32_tile(i, j, c_rows);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!bf16_finite(acc[i][j][r])) acc[i][j][r] = exact[r];
        }

    each([](float sum, float &m) { return m = sum; });
}

template <int BM, int BN, int BK>
static hipError_t launch_f32(const Geo &g, const float *U, const float *V, float *M, int splits, hipStream_t s)
{
    const int tiles_m = (g.Kp + BM - 1) / BM, tiles_n = (g.Pp + BN - 1) / BN;
    const int c_share = (g.Cp / 16 + splits - 1) / splits * 16;
    if ((g.Cp + c_share - 1) / c_share != splits) return hipErrorInvalidValue;   // every share gets at least 16 channels
    const long long blocks = (long long)tiles_m * tiles_n * g.a2 * splits;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // 32-bit byte offsets inside one component of U and of V
    if ((unsigned long long)g.Cp * g.Pp * 4ull >= (1ull << 32) || (unsigned long long)g.Cp * g.Kp * 4ull >= (1ull << 32))
        return hipErrorNotSupported;
    const dim3 grid((unsigned)blocks), block(256);
    if (c_share <= BK)
        gemm_f32_kernel<BM, BN, BK, ONE><<<grid, block, 0, s>>>(U, V, M, g.Kp, g.Cp, g.Pp, tiles_m, tiles_n, g.a2, c_share, g.C);
    else if (c_share <= BF16_LONG)
        gemm_f32_kernel<BM, BN, BK, USUAL><<<grid, block, 0, s>>>(U, V, M, g.Kp, g.Cp, g.Pp, tiles_m, tiles_n, g.a2, c_share, g.C);
    else
        gemm_f32_kernel<BM, BN, BK, LONG><<<grid, block, 0, s>>>(U, V, M, g.Kp, g.Cp, g.Pp, tiles_m, tiles_n, g.a2, c_share, g.C);
    return hipGetLastError();
}

// fp16 operands, fp32 accumulation, v_mfma_f32_32x32x16_f16.  Operands are stored as
// [e][c/8][row][c%8]: the 8 reduction values a lane feeds to one MFMA are one 16-byte word, a
// BK=32 slab is 4 contiguous runs of 16-byte words per operand, and LDS keeps the same order.
// Lanes 0-31 take the even 8-channel group of a 16-deep MFMA step, lanes 32-63 the odd one,
// for both operands alike, so every product pairs equal channels.
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

template <int BM, int BN>
__global__ __launch_bounds__(256) void gemm_f16_kernel(const uint4 *__restrict__ U, const uint4 *__restrict__ V,
                                                       float *__restrict__ Mo, int Kp, int Cp, int Pp, int tiles_m,
                                                       int tiles_n)
{
    constexpr int BK = 32, G8 = BK / 8;
    constexpr int TM = BM / 64, TN = BN / 64;
    constexpr int A4 = G8 * BM, B4 = G8 * BN;                  // 16-byte words per slab
    constexpr int AL = (A4 + 255) / 256, BL = (B4 + 255) / 256;
    __shared__ uint4 As[2][A4];
    __shared__ uint4 Bs[2][B4];

    int bid = xcd_remap(blockIdx.x, gridDim.x);   // the filter blocks that share a run of V meet in one L2
    const int tm_i = bid % tiles_m;
    bid /= tiles_m;
    const int tn_i = bid % tiles_n;
    const int e = bid / tiles_n;
    const int k0 = tm_i * BM, p0 = tn_i * BN;
    const int C8 = Cp / 8;

    const uint4 *Ue = U + (size_t)e * C8 * Kp;
    const uint4 *Ve = V + (size_t)e * C8 * Pp;
    float *Me = Mo + (size_t)e * Kp * Pp;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lg = lane >> 5;

    uint4 ra[AL], rb[BL];
    auto load_global = [&](int g0) {
#pragma unroll
        for (int j = 0; j < AL; ++j) {
            const int idx = tid + j * 256;
            const int grp = idx / BM, col = idx % BM;
            ra[j] = make_uint4(0, 0, 0, 0);
            if (idx < A4 && k0 + col < Kp) ra[j] = Ue[(size_t)(g0 + grp) * Kp + k0 + col];
        }
#pragma unroll
        for (int j = 0; j < BL; ++j) {
            const int idx = tid + j * 256;
            const int grp = idx / BN, col = idx % BN;
            rb[j] = make_uint4(0, 0, 0, 0);
            if (idx < B4 && p0 + col < Pp) rb[j] = Ve[(size_t)(g0 + grp) * Pp + p0 + col];
        }
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int j = 0; j < AL; ++j) {
            const int idx = tid + j * 256;
            if (idx < A4) As[buf][idx] = ra[j];
        }
#pragma unroll
        for (int j = 0; j < BL; ++j) {
            const int idx = tid + j * 256;
            if (idx < B4) Bs[buf][idx] = rb[j];
        }
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int nk = Cp / BK;
    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) load_global((kt + 1) * G8);
        const uint4 *as = &As[cur][wm * (BM / 2) + li];
        const uint4 *bs = &Bs[cur][wn * (BN / 2) + li];
#pragma unroll
        for (int kk = 0; kk < G8 / 2; ++kk) {
            halfx8 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const uint4 t = as[(2 * kk + lg) * BM + i * 32];
                a[i] = *reinterpret_cast<const halfx8 *>(&t);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const uint4 t = bs[(2 * kk + lg) * BN + j * 32];
                b[j] = *reinterpret_cast<const halfx8 *>(&t);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_lds(cur ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = p0 + wn * (BN / 2) + j * 32 + li;
            const int rbase = k0 + wm * (BM / 2) + i * 32 + 4 * lg;
            if (col < Pp) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = rbase + 8 * (r / 4) + (r % 4);
                    if (row < Kp) Me[(size_t)row * Pp + col] = acc[i][j][r];
                }
            }
        }
}

template <int BM, int BN>
static hipError_t launch_f16(const Geo &g, const void *U, const void *V, float *M, hipStream_t s)
{
    const int tiles_m = (g.Kp + BM - 1) / BM, tiles_n = (g.Pp + BN - 1) / BN;
    const long long blocks = (long long)tiles_m * tiles_n * g.a2;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    gemm_f16_kernel<BM, BN><<<dim3((unsigned)blocks), dim3(256), 0, s>>>((const uint4 *)U, (const uint4 *)V, M, g.Kp,
                                                                         g.Cp, g.Pp, tiles_m, tiles_n);
    return hipGetLastError();
}

// Launch shape of the fp32 multiply: block tile and number of shares of the channel loop.
// Large problems use 128 x 128 blocks and no split.  A problem with few blocks (small batch,
// small images) would leave most of the 256 CUs idle while each block runs a long serial loop,
// so it gets 64-wide blocks and, if that is still short of one block per CU, its reduction over
// C is spread over 2, 4 or 8 groups of blocks, each writing its own partial M (the inverse
// transform adds the partials while gathering).  More than one round of blocks per CU does not
// pay: every block has a fixed prologue and epilogue.
struct GemmShape { int bm, bn, splits; };

static GemmShape gemm_shape(const Geo &g)
{
    GemmShape sh;
    sh.bm = g.Kp >= 128 ? 128 : 64;
    sh.bn = g.Pp >= 128 ? 128 : 64;
    sh.splits = 1;
    if (g.dt != WINO_F32) return sh;
    auto blocks = [&](int bm, int bn) {
        return (long long)((g.Kp + bm - 1) / bm) * ((g.Pp + bn - 1) / bn) * g.a2;
    };
    {
        // Every CU works through blocks / 256 blocks; when that is a small number with a large fractional part, the
        // CUs that get one block more set the time (conv5.x at N = 64: 1600 blocks, 6.25 per CU, 7 rounds).  Halving
        // the block along the tiles doubles the count and brings the loss under 6 % (measured at N = 64: 28 x 28
        // layers 0.621 -> 0.604 ms, 14 x 14 layers 0.272 -> 0.260 ms); U, the operand that is then read twice as
        // often, is the small one.
        auto loss = [&](long long b) { return (double)((b + 255) / 256) / ((double)b / 256.0); };
        if (sh.bm == 128 && sh.bn == 128 && blocks(128, 128) >= 1024 && loss(blocks(128, 128)) > 1.06 &&
            loss(blocks(128, 64)) < loss(blocks(128, 128)) - 0.02)
            sh.bn = 64;
    }
    // Fewer than three 128 x 128 blocks per CU leave the fourth slot of most CUs empty and, with few tiles, pad the
    // last block column heavily (512 -> 512 channels at 28 x 28, batch 8, F(4x4,3x3): 576 blocks for 416 tile
    // columns; 128 x 64 blocks: 1008 blocks, 0.136 -> 0.122 ms for the layer).  From about 900 blocks on the wide
    // block is as fast or faster.
    if (blocks(sh.bm, sh.bn) < 768 && sh.bn == 128) sh.bn = 64;
    if (blocks(sh.bm, sh.bn) < 512 && sh.bm == 128) sh.bm = 64;
    const int nk = g.Cp / 16;
    const long long b = blocks(sh.bm, sh.bn);
    while (sh.splits < 8 && b * sh.splits * 2 <= 256 && nk % (sh.splits * 2) == 0 && nk / (sh.splits * 2) >= 2)
        sh.splits *= 2;
    return sh;
}

int gemm_splits(const Geo &g) { return gemm_shape(g).splits; }

void gemm_launch_shape(const Geo &g, int *bm, int *bn, int *splits)
{
    const GemmShape sh = gemm_shape(g);
    *bm = sh.bm, *bn = sh.bn, *splits = sh.splits;
}

hipError_t launch_batched_gemm(const Geo &g, const void *U, const void *V, float *M, int splits, hipStream_t s)
{
    if (g.dt == WINO_F16) {
        const bool wide_m = g.Kp >= 128, wide_n = g.Pp >= 128;
        if (splits != 1) return hipErrorInvalidValue;
        if (wide_m && wide_n) return launch_f16<128, 128>(g, U, V, M, s);
        if (wide_m) return launch_f16<128, 64>(g, U, V, M, s);
        if (wide_n) return launch_f16<64, 128>(g, U, V, M, s);
        return launch_f16<64, 64>(g, U, V, M, s);
    }
    const float *u = (const float *)U, *v = (const float *)V;
    const GemmShape sh = gemm_shape(g);
    if (sh.bm == 128 && sh.bn == 128) return launch_f32<128, 128, 16>(g, u, v, M, splits, s);
    if (sh.bm == 128) return launch_f32<128, 64, 32>(g, u, v, M, splits, s);
    if (sh.bn == 128) return launch_f32<64, 128, 32>(g, u, v, M, splits, s);
    return launch_f32<64, 64, 32>(g, u, v, M, splits, s);
}

}  // namespace wino
