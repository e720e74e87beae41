// Direct evaluation of the layer definition, Eq. (1) of Lavin & Gray (2-D correlation summed
// over channels), for layers the fast algorithm does not cover: other filter sizes, strides,
// and layers with very few channels such as the 3-channel first layer of Table 3.
#include "wino_internal.h"
#include "bf16x3.h"

namespace wino {

template <typename T> __device__ __forceinline__ float ld_d(const T *p);
template <> __device__ __forceinline__ float ld_d<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ld_d<__half>(const __half *p) { return __half2float(*p); }
template <typename T> __device__ __forceinline__ void st_d(T *p, float v);
template <> __device__ __forceinline__ void st_d<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void st_d<__half>(__half *p, float v) { *p = __float2half_rn(v); }

// The general form, for the little that the matrix units do not take (see the launcher): one thread per output pixel, KB
// filters at a time held in registers.  The filter block is
// staged in LDS as [c][u][v][k] so a thread fetches 4 filters per LDS read (all lanes read the
// same address: broadcast).  Loads of D and stores of Y are contiguous across a wavefront.
constexpr int DC_KB = 16;
constexpr int DC_LDS_FLOATS = 8192;

template <typename T>
__global__ __launch_bounds__(256) void direct_conv_kernel(const T *__restrict__ D, const T *__restrict__ G,
                                                          T *__restrict__ Y, int N, int C, int H, int W, int K, int R,
                                                          int S, int pad, int stride, int Ho, int Wo, int CC)
{
    __shared__ float gs[DC_LDS_FLOATS];
    const int pix = blockIdx.x * 256 + threadIdx.x;
    const int k0 = blockIdx.y * DC_KB;
    const int i = blockIdx.z;
    const bool live = pix < Ho * Wo;
    const int ox = live ? pix / Wo : 0, oy = live ? pix % Wo : 0;
    const int RS = R * S;
    float acc[DC_KB];
#pragma unroll
    for (int kk = 0; kk < DC_KB; ++kk) acc[kk] = 0.0f;
    const T *Di = D + (size_t)i * C * H * W;
    for (int c0 = 0; c0 < C; c0 += CC) {
        const int cn = min(CC, C - c0);
        __syncthreads();
        for (int idx = threadIdx.x; idx < cn * RS * DC_KB; idx += 256) {
            const int kk = idx % DC_KB, j = idx / DC_KB;  // j = cc*RS + uv
            const int k = k0 + kk;
            gs[idx] = (k < K) ? ld_d<T>(G + ((size_t)k * C + c0) * RS + j) : 0.0f;
        }
        __syncthreads();
        if (live) {
            for (int cc = 0; cc < cn; ++cc) {
                const T *Dc = Di + (size_t)(c0 + cc) * H * W;
                for (int u = 0; u < R; ++u) {
                    const int x = ox * stride + u - pad;
                    if (x < 0 || x >= H) continue;
                    for (int v = 0; v < S; ++v) {
                        const int y = oy * stride + v - pad;
                        if (y < 0 || y >= W) continue;
                        const float d = ld_d<T>(Dc + (size_t)x * W + y);
                        const float4 *w = reinterpret_cast<const float4 *>(&gs[((cc * R + u) * S + v) * DC_KB]);
#pragma unroll
                        for (int q = 0; q < DC_KB / 4; ++q) {
                            const float4 f = w[q];
                            acc[4 * q + 0] = fmaf(d, f.x, acc[4 * q + 0]);
                            acc[4 * q + 1] = fmaf(d, f.y, acc[4 * q + 1]);
                            acc[4 * q + 2] = fmaf(d, f.z, acc[4 * q + 2]);
                            acc[4 * q + 3] = fmaf(d, f.w, acc[4 * q + 3]);
                        }
                    }
                }
            }
        }
    }
    if (live) {
#pragma unroll
        for (int kk = 0; kk < DC_KB; ++kk)
            if (k0 + kk < K) st_d<T>(Y + (((size_t)i * K + k0 + kk) * Ho + ox) * Wo + oy, acc[kk]);
    }
}

typedef float floatx4_dc __attribute__((ext_vector_type(4)));

// four consecutive elements from an address aligned to four elements, widened to fp32
template <typename T> __device__ __forceinline__ floatx4_dc ld4_d(const T *p);
template <> __device__ __forceinline__ floatx4_dc ld4_d<float>(const float *p)
{
    return *reinterpret_cast<const floatx4_dc *>(p);
}
template <> __device__ __forceinline__ floatx4_dc ld4_d<__half>(const __half *p)
{
    const uint2 raw = *reinterpret_cast<const uint2 *>(p);
    const __half2 a = *reinterpret_cast<const __half2 *>(&raw.x), b = *reinterpret_cast<const __half2 *>(&raw.y);
    return floatx4_dc{__low2float(a), __high2float(a), __low2float(b), __high2float(b)};
}
// store that does not keep the line in the caches (an output plane is written once and is far larger than they are)
template <typename T> __device__ __forceinline__ void st_nt_d(T *p, float v);
template <> __device__ __forceinline__ void st_nt_d<float>(float *p, float v) { __builtin_nontemporal_store(v, p); }
template <> __device__ __forceinline__ void st_nt_d<__half>(__half *p, float v)
{
    __builtin_nontemporal_store(__builtin_bit_cast(unsigned short, __float2half_rn(v)), reinterpret_cast<unsigned short *>(p));
}

// 3 x 3, stride 1 with at most 4 channels (the first layer of Table 3) on the matrix units.  Eq. (1) for one
// output row is a product of the K x 9C matrix of filter taps with the 9C x Wo matrix whose column y holds the
// 3 x 3 x C window of output y: v_mfma_f32_32x32x2_f32 takes 32 filters x 2 taps x 32 neighbouring outputs of a
// row.  A workgroup owns DM_RB output rows of one image (one per wavefront) and 64 filters: the DM_RB + 2 input
// rows of every channel are staged in LDS once (fp32, zero halo = the padding), the taps of the 64 filters stay in
// registers as A operands for the whole kernel, and lane (y, h) fetches the B operand of step t -- tap 2t + h of
// window y -- with one LDS read at a per-lane offset fixed for the kernel.  Per 32 outputs: ceil(9C/2) LDS reads,
// 2 ceil(9C/2) MFMAs, and stores of 32 neighbouring outputs per filter (tried and slower: two outputs per lane
// with a lane swap, 64 neighbouring outputs per store).  The layer is bound by writing Y (C = 3,
// K = 64: 21 output values per input value), which this form approaches because the arithmetic no longer competes
// with the stores for the vector ALU.  A small problem (rb = 1) gives every workgroup a single output row, whose
// 32-output blocks the four wavefronts share, so that a batch of one still has a few hundred workgroups.
typedef float floatx16_dc __attribute__((ext_vector_type(16)));
constexpr int DM_RB = 4;

template <typename T, int CT>
__global__ __launch_bounds__(64 * DM_RB) void direct_conv3x3_mfma_kernel(const T *__restrict__ D,
                                                                         const T *__restrict__ G, T *__restrict__ Y,
                                                                         int H, int W, int K, int pad, int Ho, int Wo,
                                                                         int WS, int rb)
{
    constexpr int J = 9 * CT, NT = (J + 1) / 2;                   // taps, MFMA steps
    const int PR = rb + 2;                                        // staged rows per channel
    extern __shared__ float patch[];                              // [c][row][WS]; input column y sits at index y + 4
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, li = lane & 31, lg = lane >> 5;
    const int x0 = blockIdx.x * rb;                               // first output row of the workgroup
    const int k0 = blockIdx.y * 64;
    const int i = blockIdx.z;

    // A operands: filter k0 + 32 g + li, tap 2 t + lg (0 beyond the filters and beyond the 9C taps)
    float a[2][NT];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int k = k0 + 32 * g + li, j = 2 * t + lg;
            a[g][t] = (k < K && j < J) ? ld_d<T>(G + (size_t)k * J + j) : 0.0f;
        }
    // LDS offset of tap 2 t + lg relative to (row of the output, column of the output); a tap past 9C repeats
    // tap 0 (its A operand is 0; the B operand only has to be a number the window really contains)
    int off[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int j = (2 * t + lg < J) ? 2 * t + lg : 0;
        const int c = j / 9, u = (j % 9) / 3, v = j % 3;
        off[t] = (c * PR + u) * WS + v + 4 - pad;
    }

    // stage input rows x0 - pad .. x0 - pad + PR - 1 of every channel: 16-byte loads, zeros outside the image
    const T *Di = D + (size_t)i * CT * H * W;
    const int W4 = W / 4;
    for (int idx = tid; idx < CT * PR * W4; idx += 64 * DM_RB) {
        const int q = idx % W4, r = (idx / W4) % PR, c = idx / (W4 * PR);
        const int x = x0 - pad + r;
        floatx4_dc v = {0.f, 0.f, 0.f, 0.f};
        if (x >= 0 && x < H) v = ld4_d<T>(Di + ((size_t)c * H + x) * W + 4 * q);
        *reinterpret_cast<floatx4_dc *>(&patch[(c * PR + r) * WS + 4 + 4 * q]) = v;
    }
    for (int idx = tid; idx < CT * PR; idx += 64 * DM_RB) {       // the columns left and right of the image
        patch[idx * WS + 3] = 0.0f;
        patch[idx * WS + 4 + W] = 0.0f;
    }
    __syncthreads();

    const int xl = rb == 1 ? 0 : wave;                             // this wavefront's output row within the workgroup's
    const int x = x0 + xl;
    if (x >= Ho) return;
    const float *prow = patch + xl * WS + li;
    T *yrow = Y + (((size_t)i * K + k0 + 4 * lg) * Ho + x) * Wo + li;
    const size_t kstride = (size_t)Ho * Wo;
    for (int yb = rb == 1 ? 32 * wave : 0; yb < Wo; yb += rb == 1 ? 32 * DM_RB : 32) {
        floatx16_dc acc[2];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][r] = 0.0f;
        float b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = prow[yb + off[t]];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int g = 0; g < 2; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g][t], b[t], acc[g], 0, 0, 0);
        // accumulator register r of lane (li, lg) is filter 32 g + 8 (r / 4) + 4 lg + r % 4, output yb + li
        if (yb + li < Wo) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kk = 32 * g + 8 * (r / 4) + (r % 4);
                    if (k0 + 4 * lg + kk < K) st_nt_d<T>(yrow + (size_t)kk * kstride + yb, acc[g][r]);
                }
        }
    }
}

template <typename T, int CT>
static hipError_t launch_direct_mfma(int N, int H, int W, int K, int pad, int Ho, int Wo, const void *D, const void *G,
                                     void *Y, hipStream_t s)
{
    const int WS = (Wo + 31) / 32 * 32 + 8;   // a lane past the last output still reads inside its row
    const long long wgs = (long long)((Ho + DM_RB - 1) / DM_RB) * ((K + 63) / 64) * N;
    const int rb = wgs < 512 ? 1 : DM_RB;     // one output row per workgroup when bands of rows would not fill the chip
    const size_t lds = (size_t)CT * (rb + 2) * WS * sizeof(float);
    dim3 grid((Ho + rb - 1) / rb, (K + 63) / 64, N);
    direct_conv3x3_mfma_kernel<T, CT><<<grid, dim3(64 * DM_RB), lds, s>>>((const T *)D, (const T *)G, (T *)Y, H, W, K, pad,
                                                                        Ho, Wo, WS, rb);
    return hipGetLastError();
}

// The matrix-unit form serves 3 x 3, stride 1, 1-4 channels, rows that are a whole number of 16-byte units, and
// an LDS patch within the 64 KB a launch gets without asking.
static bool direct_mfma_ok(int C, int H, int W, int K, int R, int S, int pad, int stride, int Ho, int Wo, int N)
{
    if (R != 3 || S != 3 || stride != 1 || C < 1 || C > 4 || W % 4 != 0 || pad < 0 || pad > 1) return false;
    const long long WS = (Wo + 31) / 32 * 32 + 8;
    if ((long long)C * (DM_RB + 2) * WS * 4 > 65536) return false;
    return (Ho + DM_RB - 1) / DM_RB <= 0x7fffffff && (K + 63) / 64 <= 65535 && N <= 65535;
}

// Any filter, stride and padding as a matrix product on the matrix units: Y[k][pixel] = sum over taps j = (c, u, v) of
// G[k][j] D[pixel's window][j], the K x CRS matrix of filters as it lies in memory times the CRS x N Ho Wo matrix of
// windows, which is never built: a thread fetches its elements from D with one bounds check each.  fp32 goes through the
// bf16 units in three exact parts (bf16x3.h), fp16 directly; sums are fp32.
// A workgroup of four wavefronts owns BM filters x BN pixels.  Per step of 16 taps every thread fetches quads of four
// taps of one filter or pixel, splits them and stores the parts to LDS as 8-byte halves of the 16-byte words (eight taps
// of one row) that the matrix instruction takes; two steps are in flight in registers, two in LDS, one barrier per step.
// A step is a chain of fetch, split, barrier, LDS reads and six dependent matrix instructions, about 1 500 cycles for a
// workgroup alone on its CU, so KS groups of four wavefronts share the steps of the same block, each taking a run of them,
// and add their sums in LDS at the end: four groups where there are no more blocks than CUs, two up to twice as many.
// 64 x 128 blocks spare a third of the fetches per product where there are 512 of them.  (Fetching a filter's taps with
// lanes along the filters: 64 cache lines per request, 50 us for the first layer below.)
// Where a tap lies is looked up in LDS: (u, v) and offset repeat every 16 R S taps, 16 channels on.  Counting (c, u, v) up in
// scalars took 85 scalar instructions per step and wavefront, which the SIMDs of a CU take turns at: that, and not the
// chain, set the pace of CUs with two workgroups.  The check is three instructions: the part of a window inside the image
// is a rectangle of (u, v), its corners packed in 16-bit halves.
// One thread per pixel and 16 filters on the vector ALUs / scalars counted up / this: 64 -> 128 channels at 56 x 56, stride
// 2, N = 16: 151 / 34 / 29 us in fp32 (call after call into one output 26), 127 / 28 / 22 in fp16 (N = 1, fp32: 115 / 18 / 16);
// 512 -> 512 at 14 x 14, stride 2, N = 1: 807 / 99 / 72; 1 x 1, 256 -> 512 at 28 x 28, stride 2, N = 8: 120 / 15.4 / 14.9; 7 x 7,
// 3 -> 64 at 224 x 224, stride 2, N = 8: 84 / 36 / 28; 5 x 5, 48 -> 128 at 27 x 27, N = 4: 210 / 31 / 24; 512 -> 512 at 28 x 28,
// stride 2, N = 64: - / 659 / 541.  Error against float64: 25-60 % less than the first form's.
constexpr int DG_STEP = 16;

typedef _Float16 halfx8_dc __attribute__((ext_vector_type(8)));
typedef unsigned uintx2_d __attribute__((ext_vector_type(2)));
typedef unsigned short ushortx2_dc __attribute__((ext_vector_type(2)));

// Barrier that orders LDS traffic only: global loads requested earlier stay in flight across it.
__device__ __forceinline__ void dg_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct DgGeo {
    int C, H, W, K, R, S, pad, stride, Ho, Wo;
    int J, P;                    // taps, pixels of all images
    int tiles_m;
    int period;                  // taps after which (u, v) repeat at the same place of a step, or all
    unsigned ahead;              // bytes of D from one period to the next
};

// LONG: more than BF16_LONG taps per group, whose sums are set aside now and then (bf16x3.h).
template <typename T, int BM, int BN, int KS, bool LONG>
__global__ __launch_bounds__(256 * KS, LONG && KS == 1 ? 4 : 1) void direct_gemm_kernel(const T *__restrict__ D, const T *__restrict__ G, T *__restrict__ Y,
                                                             DgGeo g, unsigned g_bytes, size_t d_elems)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int NP = F32 ? 3 : 1;                            // parts
    constexpr int WM = BM / 32, WN = 4 / WM, TN = BN / 32 / WN; // wavefronts along filters and pixels, pixel tiles of one
    constexpr int BQ = BN * 4 / 256;                           // quads of pixels a thread fetches (of filters: one, or none)
    static_assert(WM == 1 || WM == 2, "32 or 64 filters");
    constexpr int GROUP_WORDS = 2 * 2 * NP * (BM + BN);        // LDS of a group: two slabs of both operands
    constexpr int SUM_WORDS = (KS - 1) * BM * BN / 4;          // or the sums of all groups but one
    extern __shared__ uintx4_b dg_taps[];                      // of a period: offset in D, u | v << 16
    __shared__ uintx4_b lds[KS * GROUP_WORDS > SUM_WORDS ? KS * GROUP_WORDS : SUM_WORDS];
    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    uintx4_b *const As = lds + ks * GROUP_WORDS, *const Bs = As + 2 * 2 * NP * BM;
    const int bid = blockIdx.x;
    const int k0 = bid % g.tiles_m * BM, p0 = bid / g.tiles_m * BN;
    const int plane = g.Ho * g.Wo, image = g.C * g.H * g.W;
    const int n0 = p0 / plane;

    // D from the block's first image on, and (pad rows and columns) in front of it, so that offsets are not negative;
    // only taps inside an image are fetched
    const int lead = g.pad * g.W + g.pad;
    const size_t left = (d_elems - (size_t)n0 * image + lead) * sizeof(T);
    const __amdgpu_buffer_rsrc_t rsrc_d = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(D + (size_t)n0 * image - lead), 0, (unsigned)(left < 0x7fffffffu ? left : 0x7fffffffu), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_g = __builtin_amdgcn_make_buffer_rsrc((void *)G, 0, g_bytes, 0x00020000);
    constexpr unsigned OOB = 0x80000000u;

    // quad j of this thread: taps 4 qb[j] .. + 3 of a step, pixel (filter) column; the quad is the wavefront's
    unsigned vo[BQ];
    ushortx2_dc first_tap[BQ], last_tap[BQ];                   // (u, v) of the window's part inside the image; last from first on
#pragma unroll
    for (int j = 0; j < BQ; ++j) {
        const int col = (tid + j * 256) % BN;
        const int p = min(p0 + col, g.P - 1);                  // (pixels past the last are never stored)
        const int n = p / plane, r = p - n * plane;
        const int ox = r / g.Wo, oy = r - ox * g.Wo;
        const int x = ox * g.stride - g.pad, y = oy * g.stride - g.pad;
        const int u0 = max(-x, 0), u1 = min(g.H - x, g.R), v0 = max(-y, 0), v1 = min(g.W - y, g.S);
        const bool some = u0 < u1 && v0 < v1;                  // (none: tap 0x8000, which no window has)
        first_tap[j] = some ? ushortx2_dc{(unsigned short)u0, (unsigned short)v0} : ushortx2_dc{0x8000, 0x8000};
        last_tap[j] = some ? ushortx2_dc{(unsigned short)(u1 - u0 - 1), (unsigned short)(v1 - v0 - 1)} : ushortx2_dc{0, 0};
        vo[j] = (unsigned)((n - n0) * image + ox * g.stride * g.W + oy * g.stride) * (unsigned)sizeof(T);
    }
    for (int t = threadIdx.x; t < g.period; t += 256 * KS) {
        const int c = t / (g.R * g.S), r = t - c * (g.R * g.S), u = r / g.S, v = r - u * g.S;
        const unsigned at = (((unsigned)c * g.H + u) * g.W + v) * (unsigned)sizeof(T);
        reinterpret_cast<uintx2_d *>(dg_taps)[t] = uintx2_d{at, (unsigned)u | (unsigned)v << 16};
    }
    // filters: four threads fetch the 16 taps of a step of one filter, which lie side by side
    const int arow = tid >> 2, a_quad = tid & 3;
    const bool a_role = BM == 64 || arow < BM;
    const unsigned ao = a_role ? ((unsigned)min(k0 + arow, g.K - 1) * (unsigned)g.J + 4u * a_quad) * (unsigned)sizeof(T) : OOB;
    // (a 16-byte request needs four-byte alignment, an 8-byte one of fp16 taps too)
    const bool a_wide = F32 || g.J % 2 == 0;

    T rb[2][BQ][4], ra[2][4];
    // a group's run of steps; runs differ by one step at most, as the error grows with the longest (of ten steps 2, 3, 2 and 3:
    // 3, 3, 3 and 1 were 1.10 times as far from float64 with 3 -> 34 channels, 7 x 7)
    const int all_steps = (g.J + DG_STEP - 1) / DG_STEP;
    const int j_end = min(all_steps * (ks + 1) / KS * DG_STEP, g.J);       // its taps end here
    int j_next = all_steps * ks / KS * DG_STEP;                // first tap of the step requested next
    int entry = j_next % g.period;                             // its place in the period
    unsigned base = (unsigned)(j_next / g.period) * g.ahead;   // the period's offset in D
    auto request = [&](int slot) {
        const unsigned so = base & (unsigned)((j_next - j_end) >> 31);       // (masks from signs: choices between scalars become branches)
#pragma unroll
        for (int j = 0; j < BQ; ++j) {
            const int q = (wave * 64 + j * 256) / BN;
            const uintx4_b e[2] = {dg_taps[(entry + 4 * q) / 2], dg_taps[(entry + 4 * q) / 2 + 1]};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned past = (unsigned)((j_end - 1 - j_next - 4 * q - i) >> 31);   // all ones behind the last tap
                const ushortx2_dc uv = __builtin_bit_cast(ushortx2_dc, e[i / 2][2 * (i % 2) + 1] | past) - first_tap[j];
                const bool ok = __builtin_bit_cast(unsigned, __builtin_elementwise_min(uv, last_tap[j])) == __builtin_bit_cast(unsigned, uv);
                const unsigned o = ok ? vo[j] + e[i / 2][2 * (i % 2)] : OOB;
                if constexpr (F32)
                    rb[slot][j][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_d, o, so, 0));
                else
                    rb[slot][j][i] = __builtin_bit_cast(__half, __builtin_amdgcn_raw_buffer_load_b16(rsrc_d, o, so, 0));
            }
        }
        entry += DG_STEP;
        const unsigned wrap = ~(unsigned)((entry - g.period) >> 31);       // all ones where the next period begins
        entry -= g.period & (int)wrap, base += g.ahead & wrap;
        const unsigned o = ao + (unsigned)j_next * (unsigned)sizeof(T);
        if (a_wide && j_next + DG_STEP <= j_end) {
            if constexpr (F32) {
                const floatx4_dc w = __builtin_bit_cast(floatx4_dc, __builtin_amdgcn_raw_buffer_load_b128(rsrc_g, o, 0, 0));
#pragma unroll
                for (int i = 0; i < 4; ++i) ra[slot][i] = w[i];
            } else {
                typedef _Float16 halfx4_dc __attribute__((ext_vector_type(4)));
                const halfx4_dc w = __builtin_bit_cast(halfx4_dc, __builtin_amdgcn_raw_buffer_load_b64(rsrc_g, o, 0, 0));
#pragma unroll
                for (int i = 0; i < 4; ++i) ra[slot][i] = __builtin_bit_cast(__half, (_Float16)w[i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned oi = a_role && j_next + 4 * a_quad + i < j_end ? o + i * (unsigned)sizeof(T) : OOB;
                if constexpr (F32)
                    ra[slot][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_g, oi, 0, 0));
                else
                    ra[slot][i] = __builtin_bit_cast(__half, __builtin_amdgcn_raw_buffer_load_b16(rsrc_g, oi, 0, 0));
            }
        }
        j_next += DG_STEP;
    };
    // quad q of column col: half q % 2 of words [q / 2][part][col]
    auto put = [&](uintx4_b *dst, int cols, int col, int q, const T (&x)[4]) {
        uintx2_d *w = reinterpret_cast<uintx2_d *>(dst + (q / 2) * NP * cols + col) + q % 2;
        if constexpr (F32) {
            unsigned h0, m0, l0, h1, m1, l1;
            bf16_split2(BF16_SCALE * x[0], BF16_SCALE * x[1], h0, m0, l0);
            bf16_split2(BF16_SCALE * x[2], BF16_SCALE * x[3], h1, m1, l1);
            w[0] = uintx2_d{h0, h1}, w[2 * cols] = uintx2_d{m0, m1}, w[4 * cols] = uintx2_d{l0, l1};
        } else {
            const unsigned short *h = reinterpret_cast<const unsigned short *>(x);
            w[0] = uintx2_d{h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16};
        }
    };
    auto store = [&](int slot, int buf) {
#pragma unroll
        for (int j = 0; j < BQ; ++j) put(Bs + buf * (2 * NP * BN), BN, (tid + j * 256) % BN, (wave * 64 + j * 256) / BN, rb[slot][j]);
        if (a_role) put(As + buf * (2 * NP * BM), BM, arow, a_quad, ra[slot]);
    };

    const int wm = wave % WM, wn = wave / WM, li = lane & 31, lh = lane >> 5;
    floatx16_dc acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
    auto multiply = [&](int buf) {
        uintx4_b a[NP], b[NP][TN];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            a[q] = As[(buf * 2 * NP + lh * NP + q) * BM + wm * 32 + li];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[q][j] = Bs[(buf * 2 * NP + lh * NP + q) * BN + (wn * TN + j) * 32 + li];
        }
        if constexpr (F32) {
#pragma unroll
            for (int n = 0; n < BF16_PRODUCTS; ++n)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[bf16_part_a(n)]),
                                                                     __builtin_bit_cast(bf16x8, b[bf16_part_b(n)][j]), acc[j], 0, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8_dc, a[0]),
                                                                __builtin_bit_cast(halfx8_dc, b[0][j]), acc[j], 0, 0, 0);
        }
    };
    const int steps = (all_steps + KS - 1) / KS;                     // (the same for every group: a step past the last tap is zeros)
    // (requests past the last step fetch nothing; the number of loads in flight does not depend on the path taken)
    __syncthreads();
    request(0);
    request(1);
    store(0, 0);
    __syncthreads();
    int t = 0;
    auto step = [&](int odd) {
        request(odd);
        multiply(odd);
        store(odd ^ 1, odd ^ 1);
        dg_lds_barrier();
    };
    // accumulator register r of lane (li, lh) is filter row 8 (r / 4) + 4 lh + r % 4, pixel li of its tile
    auto each = [&](auto f) {
        int first = p0 + wn * TN * 32;
        asm volatile("" : "+s"(first));           // (opaque: no address is formed ahead of where it is used)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int p = first + j * 32 + li;
            if (p < g.P) {
                const int n = p / plane;
                T *dst = Y + ((size_t)n * g.K + k0 + wm * 32 + 4 * lh) * plane + (p - n * plane);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kk = 8 * (r / 4) + r % 4;
                    if (k0 + wm * 32 + 4 * lh + kk < g.K) acc[j][r] = f(acc[j][r], dst + (size_t)kk * plane);
                }
            }
        }
    };
    // set aside in registers, or, where there is one group only, where the result will be (64 x 128 blocks lose half of
    // their workgroups per CU to the registers: 512 -> 512 channels at 28 x 28, stride 2, N = 64, with taps counted up in
    // scalars: 665 us with sums of one run, 874 set aside in registers, 700 so)
    constexpr bool IN_Y = LONG && KS == 1;
    floatx16_dc aside[LONG && !IN_Y ? TN : 1] = {};
    for (; t + 1 < steps; t += 2) {
        step(0);
        step(1);
        if (IN_Y && (t + 2) % (BF16_RUN / DG_STEP) == 0) {
            const bool first = t + 2 == BF16_RUN / DG_STEP;
            each([first](float sum, T *y) { st_d<T>(y, first ? sum : ld_d<T>(y) + sum); return 0.0f; });
        }
        if (LONG && !IN_Y && (t + 2) % (BF16_RUN / DG_STEP) == 0) {
#pragma unroll
            for (int j = 0; j < TN; ++j) aside[j] += acc[j], acc[j] = floatx16_dc{};
        }
    }
    if (t < steps) multiply(0);
    if constexpr (IN_Y) each([](float sum, T *y) { return ld_d<T>(y) + sum; });
    if constexpr (LONG && !IN_Y) {
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] += aside[j];
    }
    if constexpr (KS > 1) {
        // the groups' sums, added in order by the first: [group - 1][register][thread]
        float *sums = reinterpret_cast<float *>(lds);
        __syncthreads();
        if (ks > 0) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sums[(((ks - 1) * TN + j) * 16 + r) * 256 + tid] = acc[j][r];
        }
        __syncthreads();
        if (ks > 0) return;
#pragma unroll
        for (int z = 0; z < KS - 1; ++z)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][r] += sums[((z * TN + j) * 16 + r) * 256 + tid];
    }

    if constexpr (F32) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float t = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                acc[j][r] *= BF16_UNSCALE, acc[j][r + 1] *= BF16_UNSCALE;
                t = bf16_look(acc[j][r], acc[j][r + 1], t);
            }
            if (!__any(!bf16_finite(t))) continue;
            // the sums that are not finite, with fp32 instructions (bf16x3.h): lane (li, lh) brings tap 2 i + lh of filter and
            // pixel li
            const int p = min(p0 + (wn * TN + j) * 32 + li, g.P - 1);
            const int n = p / plane, ox = (p - n * plane) / g.Wo, oy = p - n * plane - ox * g.Wo;
            const T *window = D + (size_t)n * image, *filter = G + (size_t)min(k0 + wm * 32 + li, g.K - 1) * g.J;
            floatx16_dc exact;
#pragma unroll
            for (int r = 0; r < 16; ++r) exact[r] = 0.0f;
#pragma unroll 4
            for (int i = 0; i < (g.J + 1) / 2; ++i) {
                const int tap = 2 * i + lh, c = tap / (g.R * g.S), uv = tap - c * (g.R * g.S);
                const int x = ox * g.stride - g.pad + uv / g.S, y = oy * g.stride - g.pad + uv % g.S;
                const bool ok = tap < g.J && x >= 0 && x < g.H && y >= 0 && y < g.W;
                exact = __builtin_amdgcn_mfma_f32_32x32x2f32(tap < g.J ? filter[tap] : 0.0f,
                                                             ok ? window[((size_t)c * g.H + x) * g.W + y] : 0.0f, exact, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!bf16_finite(acc[j][r])) acc[j][r] = exact[r];
        }
    }

    each([](float sum, T *y) { st_d<T>(y, sum); return sum; });
}

// What the product form takes: the images one block of pixels touches within 31-bit byte offsets, filters likewise,
// pixels and blocks within 32 bits.  Everything else goes to the general form above.
static bool direct_gemm_ok(int N, int C, int H, int W, int K, int R, int S, int pad, int Ho, int Wo, int size)
{
    const unsigned long long plane = (unsigned long long)Ho * Wo, P = plane * N;
    const unsigned long long span = (128 + plane - 2) / plane + 1;
    const unsigned long long image = (unsigned long long)C * H * W + (unsigned long long)pad * W + pad;
    const unsigned long long limit = 1ull << 31;
    return P < limit - 256 && (unsigned long long)C * R * S < limit / 8 && span * image * size < limit - 65536 &&
           (unsigned long long)K * C * R * S * size < limit && (P / 64 + 1) * ((K + 31) / 32) < limit;
}

// entries of the table: 16 channels, or every tap the groups request
static int dg_table(const DgGeo &g, int KS)
{
    const int period = DG_STEP * g.R * g.S, all = (g.J + DG_STEP * KS - 1) / (DG_STEP * KS) * (DG_STEP * KS);
    return period < all ? period : all;
}

template <typename T, int BM, int BN, int KS>
static hipError_t launch_direct_gemm(DgGeo g, int N, const void *D, const void *G, void *Y, hipStream_t s)
{
    g.tiles_m = (g.K + BM - 1) / BM;
    g.period = dg_table(g, KS);
    g.ahead = (unsigned)DG_STEP * g.H * g.W * (unsigned)sizeof(T);
    const size_t table = (size_t)g.period * 8;
    const long long blocks = (long long)g.tiles_m * ((g.P + BN - 1) / BN);
    const unsigned g_bytes = (unsigned)((size_t)g.K * g.J * sizeof(T));
    const size_t d_elems = (size_t)N * g.C * g.H * g.W;
    const dim3 grid((unsigned)blocks), block(256 * KS);
    if constexpr (sizeof(T) == 4) {
        // (several groups: half as long again is still less than what a chain over all taps rounds off, 6100 taps of
        // operands between 1 and 1 + 2^-7, two groups: see below; and two groups with sums set aside are 7 % slower)
        if (g.J > (KS == 1 ? BF16_LONG : BF16_LONG * 3 / 2 * KS)) {
            direct_gemm_kernel<T, BM, BN, KS, true><<<grid, block, table, s>>>((const T *)D, (const T *)G, (T *)Y, g, g_bytes, d_elems);
            return hipGetLastError();
        }
    }
    direct_gemm_kernel<T, BM, BN, KS, false><<<grid, block, table, s>>>((const T *)D, (const T *)G, (T *)Y, g, g_bytes, d_elems);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_direct_gemm(const DgGeo &g, int N, const void *D, const void *G, void *Y, hipStream_t s)
{
    const int steps = (g.J + DG_STEP - 1) / DG_STEP;
    // (a table of 40 KB fits beside 32 x 128 blocks of four groups: filters of up to 320 taps per channel.  Beside all others
    // 64 KB do, what the 512 taps take that a filter may have.)
    auto groups = [&](long long blocks, int entries) {
        return blocks <= 256 && steps >= 8 && dg_table(g, 4) <= entries ? 4 : blocks <= 512 && steps >= 4 ? 2 : 1;
    };
    if (g.K <= 32) {
        const long long blocks = (g.P + 127) / 128;
        const int KS = groups(blocks, 5120);
        if (KS == 4) return launch_direct_gemm<T, 32, 128, 4>(g, N, D, G, Y, s);
        if (KS == 2) return launch_direct_gemm<T, 32, 128, 2>(g, N, D, G, Y, s);
        return launch_direct_gemm<T, 32, 128, 1>(g, N, D, G, Y, s);
    }
    if ((long long)((g.K + 63) / 64) * ((g.P + 127) / 128) >= 512) return launch_direct_gemm<T, 64, 128, 1>(g, N, D, G, Y, s);
    const long long blocks = (long long)((g.K + 63) / 64) * ((g.P + 63) / 64);
    const int KS = groups(blocks, 8192);
    if (KS == 4) return launch_direct_gemm<T, 64, 64, 4>(g, N, D, G, Y, s);
    if (KS == 2) return launch_direct_gemm<T, 64, 64, 2>(g, N, D, G, Y, s);
    return launch_direct_gemm<T, 64, 64, 1>(g, N, D, G, Y, s);
}

hipError_t launch_direct_conv(int N, int C, int H, int W, int K, int R, int S, int pad, int stride, int dt,
                              const void *D, const void *G, void *Y, hipStream_t s)
{
    const int Ho = (H + 2 * pad - R) / stride + 1, Wo = (W + 2 * pad - S) / stride + 1;
    int CC = DC_LDS_FLOATS / (DC_KB * R * S);
    if (CC < 1) return hipErrorInvalidValue;
    if (CC > C) CC = C;
    dim3 grid((Ho * Wo + 255) / 256, (K + DC_KB - 1) / DC_KB, N), block(256);
    if (grid.y > 65535 || grid.z > 65535) return hipErrorInvalidValue;
    // (D is read in 16-byte units)
    if (direct_mfma_ok(C, H, W, K, R, S, pad, stride, Ho, Wo, N) && (size_t)D % 16 == 0) {
        const bool f32 = dt == WINO_F32;
        switch (C) {
        case 1: return f32 ? launch_direct_mfma<float, 1>(N, H, W, K, pad, Ho, Wo, D, G, Y, s)
                           : launch_direct_mfma<__half, 1>(N, H, W, K, pad, Ho, Wo, D, G, Y, s);
        case 2: return f32 ? launch_direct_mfma<float, 2>(N, H, W, K, pad, Ho, Wo, D, G, Y, s)
                           : launch_direct_mfma<__half, 2>(N, H, W, K, pad, Ho, Wo, D, G, Y, s);
        case 3: return f32 ? launch_direct_mfma<float, 3>(N, H, W, K, pad, Ho, Wo, D, G, Y, s)
                           : launch_direct_mfma<__half, 3>(N, H, W, K, pad, Ho, Wo, D, G, Y, s);
        default: return f32 ? launch_direct_mfma<float, 4>(N, H, W, K, pad, Ho, Wo, D, G, Y, s)
                            : launch_direct_mfma<__half, 4>(N, H, W, K, pad, Ho, Wo, D, G, Y, s);
        }
    }
    // (up to four taps the layer is bound by writing Y, in 256-pixel runs by the general form: 1 x 1, 3 -> 300 channels, stride
    // 2 at 32 x 32, N = 64: 9.0 us against 10.0)
    if (C * R * S > 4 && direct_gemm_ok(N, C, H, W, K, R, S, pad, Ho, Wo, dt == WINO_F32 ? 4 : 2)) {
        DgGeo g;
        g.C = C, g.H = H, g.W = W, g.K = K, g.R = R, g.S = S, g.pad = pad, g.stride = stride, g.Ho = Ho, g.Wo = Wo;
        g.J = C * R * S, g.P = N * Ho * Wo, g.tiles_m = 0;
        g.period = 0, g.ahead = 0;
        return dt == WINO_F32 ? launch_direct_gemm<float>(g, N, D, G, Y, s) : launch_direct_gemm<__half>(g, N, D, G, Y, s);
    }
    if (dt == WINO_F32)
        direct_conv_kernel<float><<<grid, block, 0, s>>>((const float *)D, (const float *)G, (float *)Y, N, C, H, W, K,
                                                         R, S, pad, stride, Ho, Wo, CC);
    else
        direct_conv_kernel<__half><<<grid, block, 0, s>>>((const __half *)D, (const __half *)G, (__half *)Y, N, C, H,
                                                          W, K, R, S, pad, stride, Ho, Wo, CC);
    return hipGetLastError();
}

}  // namespace wino
