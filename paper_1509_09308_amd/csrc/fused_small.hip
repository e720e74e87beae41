// All four loops of Algorithm 1 (Lavin & Gray) in one launch for small layers: F(2x2,3x3), F(4x4,3x3) and F(6x6,3x3), fp32,
// any padding and width, untransformed filters or U.  Layers that keep the chip busy for some microseconds only are bound
// by the launches of the other forms (three, each filling and draining the chip) and by the trips of U, V and M through
// memory between them; here a workgroup repeats both transforms for what it multiplies, which costs little where most
// CUs would idle.
//
// Workgroup = 4 wavefronts owning 16 filters x 16 tiles of all components.  Per step of CS channels
//   transform: F(4x4) and F(6x6): wavefronts 0 and 1 one (tile, channel) pair per lane, 2 and 3 one (filter, channel) pair;
//     F(2x2) every wavefront both, of twice the channels.  Rows of a tile come as a whole (16- and 8-byte requests: one
//     request per tap was 1.5 times as slow).  Rows outside the image and channels past the last lie behind the buffers'
//     ends and read as 0.  Results go to one of two LDS buffers as [e][channel group][row][channel], both operands alike.
//   multiply: a quarter of the components each, v_mfma_f64_16x16x4_f64: a lane reads the CS / 4 channels of its group of a
//     filter and of a tile at once and feeds them to that many instructions.
// One barrier per step.  Products are formed and added in 64 bits: fp32 matrix instructions round more than the forms on the
// bf16 units do (32 channels, F(2x2): 2.0e-7 of the result against 1.5e-7; so 1.1e-7, what the transforms round), and three
// bf16 parts would be split once per 16 filters or tiles.
//
// Bound by its chain: a step of F(4x4) takes 1.5 us (18 matrix instructions of a wavefront, 250 vector instructions, a
// barrier), whether one step or two are in flight.  32 -> 32 channels at 56 x 56, N = 1, F(2x2): three launches 11.9 us, 6.6 so;
// 64 -> 64, 13.9 and 8.8; 32 -> 16 at 84 x 84, N = 6, F(4x4): 22.1 and 10.8.  32 filters
// per workgroup: 10-50 % slower.
#include <type_traits>

#include "wino_internal.h"
#include "transforms.h"

namespace wino {

typedef float floatx4_m __attribute__((ext_vector_type(4)));
typedef float floatx2_m __attribute__((ext_vector_type(2)));
typedef double doublex4_m __attribute__((ext_vector_type(4)));

constexpr unsigned SM_OOB = 0x80000000u;                              // an offset behind every buffer
constexpr unsigned SM_MAX_BYTES = 0x40000000u;                        // longest stretch of D one workgroup's buffer covers
constexpr int sm_cs(int m) { return m == 2 ? 16 : 8; }                // channels per step
constexpr int SM_ROW = 20;                                            // floats of a filter's 16 tiles in the epilogue's LDS

__device__ __forceinline__ void sm_lds_barrier()                      // orders LDS traffic only: loads stay in flight across it
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

enum { SM_FWD, SM_BWD, SM_U };         // filters: G, G of the exchanged layer (rotated by 180 degrees), transformed

// TILES, FILTERS: what this wavefront transforms.
template <int M, int SRC, bool TILES, bool FILTERS>
__device__ __forceinline__ void fused_small_body(const float *__restrict__ D, const float *__restrict__ F, float *__restrict__ Y,
                                                 const Geo &g, int n_tb, unsigned f_bytes, float *lds, int wave)
{
    constexpr int A = M + 2, NE = A * A, CS = sm_cs(M), Q = CS / 4;
    constexpr int NC = NE / 4;                                 // components of a wavefront
    constexpr int DEPTH = M == 2 ? 2 : 1;                      // steps in flight
    constexpr int T_FLOATS = NE * CS * 16, BUF = 2 * T_FLOATS;
    constexpr int NF = SRC == SM_U ? NE : 9;                   // values of a (filter, channel) pair
    static_assert(NE * 16 * SM_ROW <= 2 * BUF, "the epilogue reuses the two buffers");
    // logically consecutive workgroups share filters and run on one XCD
    const int per = gridDim.x / 8;
    const int bid = blockIdx.x < per * 8 ? (blockIdx.x % 8) * per + blockIdx.x / 8 : blockIdx.x;
    const int k0 = bid / n_tb * 16, b0 = bid % n_tb * 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int steps = (g.C + CS - 1) / CS;
    // row i of channel group h lies at i ^ swizzle(h): the filters' writes, channels first, then meet two to a bank
    auto swizzle = [](int h) { return CS == 8 ? (h & 1) * 8 : h * 4; };

    // ---- tiles: lane's tile b0 + tid % 16, channel tid / 16 of the step ----
    const int tiles_per_image = g.Th * g.Tw, img0 = b0 / tiles_per_image;
    const unsigned plane = (unsigned)(g.H * g.W) * 4u;
    const size_t image = (size_t)g.C * g.H * g.W, left = ((size_t)g.N - img0) * image * 4;
    const __amdgpu_buffer_rsrc_t rsrc_d = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(D + (size_t)img0 * image - 1), 0, (unsigned)(left < SM_MAX_BYTES ? left : SM_MAX_BYTES) + 4u, 0x00020000);
    const int cl = tid >> 4 & (CS - 1);
    // A tile's rows are fetched whole, A columns from y0 on.  The column left of the image is the element in front (the buffer
    // begins one element early; it is zeroed afterwards), but for the very first row of D, which is fetched from its first
    // column on and moved: there is nothing in front.  The last tile of a row is fetched from column W - A on and moved
    // `over` columns: nothing behind a row is fetched.
    unsigned at[A];
    const int over = max(M * (g.Tw - 1) - g.pad + A - g.W, 0);
    bool left_out, cut;
    {
        const int b = b0 + (tid & 15);
        const int ty = b % g.Tw, t2 = b / g.Tw, tx = t2 % g.Th;
        const int x0 = M * tx - g.pad, y0 = M * ty - g.pad;
        left_out = y0 < 0, cut = over > 0 && ty == g.Tw - 1;
        const unsigned first = (unsigned)((t2 / g.Th - img0) * g.C + cl) * plane + 4u;
#pragma unroll
        for (int p = 0; p < A; ++p)
            at[p] = b < g.P && x0 + p >= 0 && x0 + p < g.H ? first + (unsigned)((x0 + p) * g.W + y0 - (cut ? over : 0)) * 4u : SM_OOB;
    }
    const bool head = left_out && b0 + (tid & 15) == 0 && cl == 0;         // (its row 0 of the image is row `pad` of the tile)
    if (head) at[1] += 4u;
    // ---- filters: G[k][c] lies together by channel, so lanes run along channels; the others by filter ----
    const __amdgpu_buffer_rsrc_t rsrc_f = __builtin_amdgcn_make_buffer_rsrc((void *)F, 0, f_bytes, 0x00020000);
    const int ft = CS == 16 ? tid : tid & 127;
    const int fc = SRC == SM_FWD ? ft % CS : ft / 16, fk = SRC == SM_FWD ? ft / CS : ft % 16;

    float d[DEPTH][A][A], f[DEPTH][NF];
    auto request = [&](auto sc, int step) {
        constexpr int S = decltype(sc)::value % DEPTH;
        if constexpr (TILES) {
            const unsigned so = step < steps ? (unsigned)step * CS * plane : 0u;
            const unsigned none = step * CS + cl < g.C ? 0u : SM_OOB;
#pragma unroll
            for (int p = 0; p < A; ++p) {
                const unsigned o = at[p] | none;
#pragma unroll
                for (int q = 0; q < A; q += 4) {
                    if (q + 4 <= A) {
                        const floatx4_m x = __builtin_bit_cast(floatx4_m, __builtin_amdgcn_raw_buffer_load_b128(rsrc_d, o + 4u * q, so, 0));
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[S][p][(q + i) % A] = x[i];
                    } else {
                        const floatx2_m x = __builtin_bit_cast(floatx2_m, __builtin_amdgcn_raw_buffer_load_b64(rsrc_d, o + 4u * q, so, 0));
#pragma unroll
                        for (int i = 0; i < 2; ++i) d[S][p][(q + i) % A] = x[i];
                    }
                }
            }
        }
        if constexpr (FILTERS) {
            const int c = step * CS + fc;
            {
                const int k = k0 + fk;
                if constexpr (SRC == SM_U) {
                    const unsigned o = k < g.Kp && c < g.Cp ? ((unsigned)c * g.Kp + k) * 4u : SM_OOB;
#pragma unroll
                    for (int e = 0; e < NE; ++e)
                        f[S][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_f, o, (unsigned)(e * g.Cp) * g.Kp * 4u, 0));
                } else {
                    const unsigned o = k < g.K && c < g.C ? (SRC == SM_FWD ? (unsigned)k * g.C + c : (unsigned)c * g.K + k) * 36u : SM_OOB;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const floatx4_m x = __builtin_bit_cast(floatx4_m, __builtin_amdgcn_raw_buffer_load_b128(rsrc_f, o + 16u * h, 0, 0));
#pragma unroll
                        for (int i = 0; i < 4; ++i) f[S][SRC == SM_BWD ? 8 - (4 * h + i) : 4 * h + i] = x[i];
                    }
                    f[S][SRC == SM_BWD ? 0 : 8] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_f, o + 32u, 0, 0));
                }
            }
        }
    };
    // taps fetched from another column than they belong to
    auto prepare = [&](auto sc) {
        constexpr int S = decltype(sc)::value % DEPTH;
        if constexpr (TILES) {
            if (b0 == 0 && wave == 0) {
#pragma unroll
                for (int q = A - 1; q > 0; --q) {
                    float here = d[S][1][q], before = d[S][1][q - 1];
                    asm("" : "+v"(here), "+v"(before));     // (or the choice is made between addresses, and the array stays in memory)
                    d[S][1][q] = head ? before : here;
                }
            }
            if (__any(cut)) {
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    if (!(over >> n & 1)) continue;
#pragma unroll
                    for (int p = 0; p < A; ++p)
#pragma unroll
                        for (int q = 0; q < A; ++q) {
                            float here = d[S][p][q], further = d[S][p][(q + (1 << n)) % A];
                            asm("" : "+v"(here), "+v"(further));
                            d[S][p][q] = cut ? (q + (1 << n) < A ? further : 0.0f) : here;
                        }
                }
            }
        }
    };
    auto transform = [&](auto sc, int buf) {
        constexpr int S = decltype(sc)::value % DEPTH;
        if constexpr (TILES) {
            const int h = cl / Q;
            float *const to = lds + buf * BUF + (h * 16 + ((tid & 15) ^ swizzle(h))) * Q + cl % Q;
            float t[A][A];
#pragma unroll
            for (int p = 0; p < A; ++p) {
                const float first = d[S][p][0];
                d[S][p][0] = left_out ? 0.0f : first;
                bt_mul<M>(d[S][p], t[p]);
            }
#pragma unroll
            for (int q = 0; q < A; ++q) {
                float in[A], o[A];
#pragma unroll
                for (int p = 0; p < A; ++p) in[p] = t[p][q];
                bt_mul<M>(in, o);
#pragma unroll
                for (int p = 0; p < A; ++p) to[(p * A + q) * (CS * 16)] = o[p];
            }
        }
        if constexpr (FILTERS) {
            const int h = fc / Q;
            {
                float *const to = lds + buf * BUF + T_FLOATS + (h * 16 + (fk ^ swizzle(h))) * Q + fc % Q;
                if constexpr (SRC == SM_U) {
#pragma unroll
                    for (int e = 0; e < NE; ++e) to[e * (CS * 16)] = f[S][e];
                } else {
                    float t[A][3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const float in[3] = {f[S][q], f[S][3 + q], f[S][6 + q]};
                        float o[A];
                        g_mul<M>(in, o);
#pragma unroll
                        for (int p = 0; p < A; ++p) t[p][q] = o[p];
                    }
#pragma unroll
                    for (int p = 0; p < A; ++p) {
                        float o[A];
                        g_mul<M>(t[p], o);
#pragma unroll
                        for (int q = 0; q < A; ++q) to[(p * A + q) * (CS * 16)] = o[q];
                    }
                }
            }
        }
    };

    // ---- multiply: components NC wave ..; lane (i, h): filter resp. tile i, channels of group h ----
    const int li = lane & 15, lh = lane >> 4;
    doublex4_m acc[NC];
#pragma unroll
    for (int e = 0; e < NC; ++e) acc[e] = doublex4_m{0.0, 0.0, 0.0, 0.0};
    typedef std::conditional_t<Q == 4, floatx4_m, floatx2_m> op_t;
    const float *const ops = lds + wave * NC * (CS * 16) + (lh * 16 + (li ^ swizzle(lh))) * Q;
    auto multiply = [&](int buf) {
#pragma unroll
        for (int e = 0; e < NC; ++e) {
            const op_t b = *reinterpret_cast<const op_t *>(ops + buf * BUF + e * (CS * 16));
            const op_t a = *reinterpret_cast<const op_t *>(ops + buf * BUF + T_FLOATS + e * (CS * 16));
#pragma unroll
            for (int t = 0; t < Q; ++t) acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[t], (double)b[t], acc[e], 0, 0, 0);
        }
    };
    constexpr std::integral_constant<int, 0> even;
    constexpr std::integral_constant<int, 1> odd;
    request(even, 0);
    if constexpr (DEPTH == 2) request(odd, 1);
    prepare(even);
    transform(even, 0);
    request(even, DEPTH);
    sm_lds_barrier();
    auto step = [&](auto bc, int s) {
        constexpr int B = decltype(bc)::value;
        constexpr std::integral_constant<int, B ^ 1> next;
        prepare(next);
        multiply(B);
        transform(next, B ^ 1);                // (past the last step: of nothing, read by nobody)
        request(next, s + 1 + DEPTH);          // (past the last step: nothing is fetched)
        sm_lds_barrier();
    };
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        step(even, s);
        step(odd, s + 1);
    }
    if (s < steps) step(even, s);

    // ---- inverse transform: register r of lane (i, h) is filter 4 r + h, tile i ----
#pragma unroll
    for (int e = 0; e < NC; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) lds[((wave * NC + e) * 16 + 4 * r + lh) * SM_ROW + li] = (float)acc[e][r];
    sm_lds_barrier();
    const int b = b0 + (tid & 15);
    const int ty = b % g.Tw, t2 = b / g.Tw, tx = t2 % g.Th;
    const int xo = M * tx, yo = M * ty;
    const bool wide = g.Wo % (M == 4 ? 4 : 2) == 0;            // rows of a tile in whole units of 16 or 8 bytes
    const int k = k0 + (tid >> 4);
    const float *const from = lds + (tid >> 4) * SM_ROW + (tid & 15);
    float t[M][A], y[M][M];
#pragma unroll
    for (int q = 0; q < A; ++q) {
        float in[A], o[M];
#pragma unroll
        for (int p = 0; p < A; ++p) in[p] = from[(p * A + q) * (16 * SM_ROW)];
        at_mul<M>(in, o);
#pragma unroll
        for (int p = 0; p < M; ++p) t[p][q] = o[p];
    }
#pragma unroll
    for (int p = 0; p < M; ++p) at_mul<M>(t[p], y[p]);
    if (b >= g.P || k >= g.K) return;
    float *const dst = Y + (((size_t)(t2 / g.Th) * g.K + k) * g.Ho + xo) * g.Wo + yo;
#pragma unroll
    for (int p = 0; p < M; ++p) {
        if (xo + p >= g.Ho) break;
        float *const at = dst + (size_t)p * g.Wo;
        if (wide) {
            if constexpr (M == 4) {
                *reinterpret_cast<floatx4_m *>(at) = floatx4_m{y[p][0], y[p][1], y[p][2], y[p][3]};
            } else {
#pragma unroll
                for (int q = 0; q < M; q += 2)
                    if (yo + q < g.Wo) *reinterpret_cast<floatx2_m *>(at + q) = floatx2_m{y[p][q], y[p][q + 1]};
            }
        } else {
#pragma unroll
            for (int q = 0; q < M; ++q)
                if (yo + q < g.Wo) at[q] = y[p][q];
        }
    }
}

template <int M, int SRC>
__global__ __launch_bounds__(256) void fused_small_kernel(const float *__restrict__ D, const float *__restrict__ F,
                                                          float *__restrict__ Y, Geo g, int n_tb, unsigned f_bytes)
{
    __shared__ __attribute__((aligned(16))) float lds[2 * (M + 2) * (M + 2) * sm_cs(M) * 16 * 2];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (sm_cs(M) == 16)
        fused_small_body<M, SRC, true, true>(D, F, Y, g, n_tb, f_bytes, lds, wave);
    else if (wave < 2)
        fused_small_body<M, SRC, true, false>(D, F, Y, g, n_tb, f_bytes, lds, wave);
    else
        fused_small_body<M, SRC, false, true>(D, F, Y, g, n_tb, f_bytes, lds, wave);
}

bool fused_small_eligible(const Geo &g)
{
    if (g.dt != WINO_F32 || g.W < g.alpha) return false;
    // the tiles of one item span at most `span` images; their byte offsets from the first must stay below 2^30
    const unsigned long long tiles = (unsigned long long)g.Th * g.Tw, span = (16 + tiles - 2) / tiles + 1;
    if (span * g.C * g.H * g.W * 4ull + 65536 >= SM_MAX_BYTES) return false;
    if ((unsigned long long)g.a2 * g.Cp * g.Kp * 4ull >= SM_OOB) return false;
    return ((long long)g.P + 15) / 16 * ((g.K + 15) / 16) <= 0x7fffffffLL;
}

// Small enough: estimates of both forms' time in microseconds, fitted to 2300 layers of up to 50 000 items: for the stages so that
// 85-95 % of the layers take longer, for this form so that 90 % take less.  The four stages: a fixed part and what V, M (padded, and
// once more the filters that exist) and D take through the caches (MB); the input gradient's filter transform is a launch of its
// own.  This form: up to one workgroup per CU a fixed part and its steps; beyond, rounds of two workgroups per CU (F(6x6): one),
// between as many as they fill and as many as they begin, each a fixed part and its steps; and Y.  Transformed filters are fetched
// value by value.  Of 1500 other layers that the rule sends here none took longer than the four stages.
// Measured, stages / this form: F(2x2), 64 -> 64 channels at 56 x 56: 13.9 / 8.8 us (from U 13.0 / 9.6); 5 -> 98 at 53 x 53, N = 19, 6062
// items: 46 / 51 (45 / 54); 2 -> 129 at 197 x 11, N = 24, 6615 items: 47 / 57 (45 / 61); 31 -> 22 at 120 x 120, N = 13: 63 / 70 (63 /
// 78); 109 -> 44 at 17 x 17: 12.1 / 12.1 (11.6 / 13.0); F(4x4), 32 -> 16 at 84 x 84, N = 6: 22.1 / 10.8; F(6x6), 39 -> 16 at 150 x 147,
// N = 4: 34 / 23; 5 -> 20 at 64 x 97, N = 49: 49 / 59.
bool fused_small_preferred(const Geo &g, int filters)
{
    if (!fused_small_eligible(g)) return false;
    const double items = (double)((g.P + 15) / 16) * ((g.K + 15) / 16), steps = (g.C + sm_cs(g.m) - 1) / sm_cs(g.m);
    const double row = 4e-6 * g.a2 * g.Pp, D = 4e-6 * g.N * g.C * g.H * g.W, Y = 4e-6 * g.N * g.K * g.Ho * g.Wo;
    const bool u = filters == WINO_FILTERS_U;
    const double resident = g.m == 6 ? 256.0 : 512.0;
    const double rounds = 0.5 * (items / resident + (double)(long long)((items + resident - 1.0) / resident));
    const double past = row * ((double)g.Cp + g.Kp) > 256.0 ? row * ((double)g.Cp + g.Kp) - 256.0 : 0.0;     // MB that the last-level cache does not hold
    double stages, us;
    if (g.m == 2) {
        stages = 8.8 + row * (0.09 * g.Cp + 0.1 * g.Kp + 0.22 * g.K) + 1.15 * D + 0.1 * past;
        us = items <= 256 ? 4.8 + (u ? 1.2 : 1.0) * steps + 0.7 * Y : 3.5 + rounds * (1.8 + (u ? 2.1 : 1.78) * steps) + 0.26 * Y;
    } else if (g.m == 4) {
        stages = 10.2 + row * (0.08 * g.Cp + 0.13 * g.Kp + 0.27 * g.K) + 0.88 * D + 0.1 * past;
        us = items <= 256 ? 5.5 + 1.5 * steps + 0.35 * Y : 4.1 + rounds * ((u ? 3.4 : 2.7) + 2.5 * steps) + 0.24 * Y;
    } else {
        stages = 13.2 + row * (0.16 * g.Cp + 0.055 * g.Kp + 0.43 * g.K) + 0.58 * D + 0.1 * past;
        us = items <= 256 ? 7.1 + 3.2 * steps + 0.65 * Y : 6.6 + rounds * (3.5 + 3.4 * steps) + 0.54 * Y;
    }
    if (filters == WINO_FILTERS_G_BWD) stages += 2.5;
    return us < stages;
}

template <int M>
static hipError_t sm_launch(const Geo &g, const float *D, const float *G, const float *U, float *Y, bool bwd, hipStream_t s)
{
    const int n_tb = (g.P + 15) / 16;
    const dim3 grid((unsigned)(n_tb * ((g.K + 15) / 16))), block(256);
    if (U != nullptr)
        fused_small_kernel<M, SM_U><<<grid, block, 0, s>>>(D, U, Y, g, n_tb, (unsigned)((size_t)g.a2 * g.Cp * g.Kp * 4));
    else if (bwd)
        fused_small_kernel<M, SM_BWD><<<grid, block, 0, s>>>(D, G, Y, g, n_tb, (unsigned)((size_t)g.K * g.C * 36));
    else
        fused_small_kernel<M, SM_FWD><<<grid, block, 0, s>>>(D, G, Y, g, n_tb, (unsigned)((size_t)g.K * g.C * 36));
    return hipGetLastError();
}

// G (`bwd`: of the exchanged layer) or U given.
hipError_t launch_fused_small(const Geo &g, const float *D, const float *G, const float *U, float *Y, bool bwd, hipStream_t s)
{
    if (g.m == 2) return sm_launch<2>(g, D, G, U, Y, bwd, s);
    return g.m == 4 ? sm_launch<4>(g, D, G, U, Y, bwd, s) : sm_launch<6>(g, D, G, U, Y, bwd, s);
}

}  // namespace wino
