// Non-negative factorisation of the magnitude matrix, tile by tile (Algorithm 1's first step, Sec. 2.1):
// M = |W| (optionally manipulated, Sec. 3.2) ~ M_p M_z with M_p (r x k), M_z (k x c) >= 0, minimising the
// Frobenius distance.  The paper uses an off-the-shelf library and names no algorithm; this is Lee and Seung's
// multiplicative update for that objective, from the caller's starting point, M_z first and then M_p:
//     M_z <- M_z * (M_p^T M) / (M_p^T M_p M_z + eps)
//     M_p <- M_p * (M M_z^T) / (M_p M_z M_z^T + eps)
// Per half update two kernels, all tiles per launch: the k x k Gram matrix of the factor that stays fixed
// (M_p^T M_p or M_z M_z^T), then the update itself.  Every sum is a contraction, so all of them run on the matrix
// cores in fp32 (v_mfma_f32_32x32x2, or 16x16x4 up to rank 16): the products are exact fp32 fused multiply-adds, as on
// the vector ALUs, and the operands come straight from global memory in the instruction's own lane layout, because
// the order of the reduction index is free and a lane may take neighbouring elements:
//   * M_z update: a workgroup of four wavefronts owns 64 columns of a tile (a row of them is one 128-byte line in 16
//     bits) and each wavefront takes a quarter of the rows.  A lane holds 2 (4) neighbouring columns of its row of W and
//     one value of M_p per step; no LDS in the loop.
//   * M_p update: a workgroup owns 64 rows, a wavefront a quarter of the columns.  A lane takes 8 neighbouring
//     columns of its row of W and of its row of M_z per two (one) steps, out of chunks that the wavefront copies into LDS.
// The denominators (Gram matrix times the old factor) are split over the wavefronts in the same way, and both partial
// results are added through LDS in wavefront order.  New factors go to a second buffer (the other half update still
// needs the old values), the two buffers swap every iteration.  fp32 throughout, every sum in a fixed order.  Up to 64
// ranks share one pass over W; any k up to 256 (the paper's largest) is served.
// What bounds it: the fp32 matrix rate, 2 m n k flops per half update (4096 x 9216 at rank 32: 16 us at 154 TFLOP/s), and
// beside it W from the memory-side cache (75 MB).  Measured there, f16 in 512 x 576 tiles:
// M_z 37 us, M_p 42 us, Gram matrices 7 us each (one lane per column and vector fused multiply-adds: 215, 183, 31 and
// 42 us); error against 64 bits after 20 iterations 6.2e-7 (7.5e-7).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "lrbi_internal.hpp"

namespace lrbi {

static constexpr int kNmfThreads = 256;
static constexpr int kNmfWaves = kNmfThreads / 64;
static constexpr int kNmfMaxK = 256;
static constexpr int kNmfOwn = 64; // columns (rows) of a tile per workgroup
// wavefronts per SIMD that the updates' registers have to leave room for (four hide the loads of the loops; the forms with
// more results or single-element loads do not fit 128 registers)
template <typename T, int R, int RB, int VW>
static constexpr int kNmfWavesPerSimd = (VW == 1 || RB > 1) ? 2 : (R == 32 && VW == 8 ? 4 : 3);
static constexpr int kNmfChunk = 32; // columns of W and M_z that a wavefront of the M_p update copies into LDS at a time
static constexpr int kGramThreads = 512;
static constexpr int kGramWaves = kGramThreads / 64;

// Element e of the packed words of a lane, as |w| in fp32, with the manipulation of Sec. 3.2: 1 none, 2 squared, 3
// amplified where magnitude pruning keeps the weight.
template <typename T> __device__ __forceinline__ float nmf_elem(const uint32_t *w, int e);
template <> __device__ __forceinline__ float nmf_elem<float>(const uint32_t *w, int e) { return __builtin_bit_cast(float, w[e]); }
template <> __device__ __forceinline__ float nmf_elem<__half>(const uint32_t *w, int e)
{
    const uint16_t h = (uint16_t)((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu));
    return (float)__builtin_bit_cast(_Float16, h);
}
template <> __device__ __forceinline__ float nmf_elem<__hip_bfloat16>(const uint32_t *w, int e)
{
    return __builtin_bit_cast(float, (e & 1) ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16));
}
struct NmfManip {
    int method;
    float w_threshold, amplify;
};
template <typename T, bool PLAIN> __device__ __forceinline__ float nmf_mag(const uint32_t *w, int e, const NmfManip &m)
{
    const float a = fabsf(nmf_elem<T>(w, e));
    if (PLAIN) return a;
    const float squared = a * a;
    const float amplified = (a >= m.w_threshold) ? a * m.amplify : a;
    return (m.method == 2) ? squared : ((m.method == 3) ? amplified : a);
}

__device__ __forceinline__ int64_t nmf_tiles(const Geom &g) { return (int64_t)g.tile_rows * g.tile_cols; }
__device__ __forceinline__ void nmf_tile_extent(const Geom &g, int64_t t, int &ti, int &tj, int &rt, int &ct)
{
    ti = (int)(t / g.tile_cols);
    tj = (int)(t - (int64_t)ti * g.tile_cols);
    rt = (int)((g.m - (int64_t)ti * g.r < g.r) ? g.m - (int64_t)ti * g.r : g.r);
    ct = (int)((g.n - (int64_t)tj * g.c < g.c) ? g.n - (int64_t)tj * g.c : g.c);
}

// fp32 matrix instruction with a square R x R result: lane = (index li of the operand's row / column, reduction index lk)
template <int R> struct NmfMat;
template <> struct NmfMat<32> {
    static constexpr int KS = 2, NR = 16; // reduction steps per instruction, result registers
    typedef __attribute__((ext_vector_type(16))) float acc_t;
    __device__ static acc_t mma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
};
template <> struct NmfMat<16> {
    static constexpr int KS = 4, NR = 4;
    typedef __attribute__((ext_vector_type(4))) float acc_t;
    __device__ static acc_t mma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int v, int lane) { return 4 * (lane >> 4) + v; }
};
template <int R> __device__ __forceinline__ typename NmfMat<R>::acc_t nmf_zero()
{
    typename NmfMat<R>::acc_t z;
#pragma unroll
    for (int v = 0; v < NmfMat<R>::NR; ++v) z[v] = 0.f;
    return z;
}

// consecutive workgroups go round the eight XCDs: the workgroups of one tile, which share its factors, get one L2
__device__ __forceinline__ int64_t nmf_block_id()
{
    if (gridDim.y > 1) return wide_block(); // millions of tiles
    const unsigned q = gridDim.x / 8, rest = gridDim.x % 8, x = blockIdx.x % 8;
    return (int64_t)x * q + (x < rest ? x : rest) + blockIdx.x / 8;
}

// COUNT consecutive elements from p + at, VW per load (VW = 1: any alignment), packed into 32-bit words.  A piece that
// starts at or past `limit` reads the one at p instead: the callers replace what it holds by zero or never store its result.
template <typename T, int COUNT> struct NmfPack {
    static constexpr int WORDS = COUNT * (int)sizeof(T) / 4;
    uint32_t w[WORDS];
};
template <int VW, typename T, int COUNT>
__device__ __forceinline__ void nmf_load(NmfPack<T, COUNT> &out, const T *__restrict__ p, int at, int limit)
{
    constexpr int V = VW < COUNT ? VW : COUNT;
    constexpr int WORDS = V * (int)sizeof(T) / 4; // per piece
    if constexpr (V == 1 && sizeof(T) == 2) {
        uint32_t h[COUNT];
#pragma unroll
        for (int q = 0; q < COUNT; ++q) h[q] = *reinterpret_cast<const uint16_t *>(p + (at + q < limit ? at + q : 0));
#pragma unroll
        for (int q = 0; q < COUNT; q += 2) out.w[q / 2] = h[q] | (h[q + 1] << 16);
    } else {
#pragma unroll
        for (int q = 0; q < COUNT; q += V) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(p + (at + q < limit ? at + q : 0));
            uint32_t *dst = out.w + q * (int)sizeof(T) / 4;
            if constexpr (WORDS == 1) {
                dst[0] = src[0];
            } else if constexpr (WORDS == 2) {
                const uint2 v = *reinterpret_cast<const uint2 *>(src);
                dst[0] = v.x, dst[1] = v.y;
            } else {
#pragma unroll
                for (int e = 0; e < WORDS; e += 4) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(src + e);
                    dst[e] = v.x, dst[e + 1] = v.y, dst[e + 2] = v.z, dst[e + 3] = v.w;
                }
            }
        }
    }
}

// one piece of BYTES as it goes from global memory to LDS
template <int BYTES> struct NmfRaw;
template <> struct NmfRaw<2> {
    typedef uint16_t type;
    __device__ static type zero() { return 0; }
};
template <> struct NmfRaw<4> {
    typedef uint32_t type;
    __device__ static type zero() { return 0u; }
};
template <> struct NmfRaw<8> {
    typedef __attribute__((ext_vector_type(2))) uint32_t type;
    __device__ static type zero() { return type{0u, 0u}; }
};
template <> struct NmfRaw<16> {
    typedef __attribute__((ext_vector_type(4))) uint32_t type;
    __device__ static type zero() { return type{0u, 0u, 0u, 0u}; }
};
template <int WORDS> __device__ __forceinline__ void nmf_lds_read(uint32_t (&out)[WORDS], const unsigned char *p)
{
#pragma unroll
    for (int e = 0; e < WORDS; e += 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(p + 4 * e);
        out[e] = v.x, out[e + 1] = v.y, out[e + 2] = v.z, out[e + 3] = v.w;
    }
}

// Keeps a request where it is written: without it the compiler merges the request in front of a loop and the one at the
// loop's end into one load right before its use, and nothing is in flight any more.
__device__ __forceinline__ void nmf_requested() { asm volatile("" ::: "memory"); }

// First of the `steps` steps that belong to wavefront `wave` of `waves` (to the next wavefront's first).  In 64 bits: a tile
// may have 2^31 rows or columns.
__host__ __device__ constexpr int nmf_share(int steps, int wave, int waves) { return (int)((int64_t)steps * wave / waves); }
static_assert(nmf_share(1 << 30, kNmfWaves, kNmfWaves) == 1 << 30 && nmf_share(1 << 30, 7, kGramWaves) == 7 << 27, "shares of 2^30 steps");

// Gram matrix of a tile's fixed factor: G[a][b] = sum_i Mp[i][a] Mp[i][b] (ZSIDE = false) or sum_j Mz[a][j] Mz[b][j]
// (ZSIDE = true).  Workgroup = (tile, pair of rank blocks a <= b); its eight wavefronts split the sum.
template <int R, int VW, bool ZSIDE>
__global__ __launch_bounds__(kGramThreads) void nmf_gram_kernel(Geom g, const float *__restrict__ F, float *__restrict__ G,
                                                               int kblocks, int pairs)
{
    using M = NmfMat<R>;
    static __shared__ float stage[kGramWaves * M::NR * 64];
    const int64_t id = nmf_block_id(), t = id / pairs;
    if (t >= nmf_tiles(g)) return;
    int pair = (int)(id - t * pairs), ab = 0;
    while (pair >= kblocks - ab) pair -= kblocks - ab++;
    const int bb = ab + pair;
    int ti, tj, rt, ct;
    nmf_tile_extent(g, t, ti, tj, rt, ct);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane % R, lk = lane / R, k = g.k;
    const int ra = (ab * R + li < k) ? ab * R + li : k - 1, rb = (bb * R + li < k) ? bb * R + li : k - 1;
    typename M::acc_t acc = nmf_zero<R>();
    if (ZSIDE) {
        const float *f = F + t * (int64_t)k * g.c;
        const float *fa = f + (int64_t)ra * g.c, *fb = f + (int64_t)rb * g.c;
        const int steps = (ct + 8 * M::KS - 1) / (8 * M::KS);
        for (int s = nmf_share(steps, wave, kGramWaves); s < nmf_share(steps, wave + 1, kGramWaves); ++s) {
            const int j = s * 8 * M::KS + 8 * lk;
            NmfPack<float, 8> va, vb;
            nmf_load<VW>(va, fa, j, ct);
            if (ab != bb) nmf_load<VW>(vb, fb, j, ct);
            else vb = va;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                acc = M::mma(j + u < ct ? nmf_elem<float>(va.w, u) : 0.f, j + u < ct ? nmf_elem<float>(vb.w, u) : 0.f, acc);
        }
    } else {
        const float *f = F + t * (int64_t)g.r * k;
        const int steps = (rt + M::KS - 1) / M::KS;
        const int send = nmf_share(steps, wave + 1, kGramWaves);
        for (int s0 = nmf_share(steps, wave, kGramWaves); s0 < send; s0 += 8) {
            float va[8], vb[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = (s0 + u) * M::KS + lk, ic = i < rt ? i : rt - 1;
                va[u] = f[(int64_t)ic * k + ra];
                vb[u] = f[(int64_t)ic * k + rb];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool in = s0 + u < send && (s0 + u) * M::KS + lk < rt;
                acc = M::mma(in ? va[u] : 0.f, in ? vb[u] : 0.f, acc);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < M::NR; ++v) stage[(wave * M::NR + v) * 64 + lane] = acc[v];
    __syncthreads();
    for (int v = wave; v < M::NR; v += kGramWaves) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kGramWaves; ++w) sum += stage[(w * M::NR + v) * 64 + lane];
        const int a = ab * R + M::row(v, lane), b = bb * R + li;
        if (a < k && b < k) {
            float *gt = G + t * (int64_t)k * k;
            gt[(int64_t)a * k + b] = sum;
            if (ab != bb) gt[(int64_t)b * k + a] = sum;
        }
    }
}

// Adds the four wavefronts' partial results of one rank block, in wavefront order; lane and register keep their meaning.
// A wavefront gets the registers v of [wave * NR / 4, (wave + 1) * NR / 4) of each of the NB result blocks.
template <int R, int NB, int ITEMS>
__device__ __forceinline__ void nmf_reduce(float *stage, const typename NmfMat<R>::acc_t (&acc)[NB], float (&out)[ITEMS],
                                           int wave, int lane)
{
    constexpr int NR = NmfMat<R>::NR;
    __syncthreads(); // what the staging area held has been consumed
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < NR; ++v) stage[((wave * NB + b) * NR + v) * 64 + lane] = acc[b][v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < ITEMS; ++e) {
        const int b = e % NB, v = wave * (NR / kNmfWaves) + e / NB;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kNmfWaves; ++w) sum += stage[((w * NB + b) * NR + v) * 64 + lane];
        out[e] = sum;
    }
}

// M_z update.  Workgroup = (tile, 64 columns); lane li holds columns NB * li .. + NB - 1, block b of the result the
// columns NB * li + b.
template <typename T, int R, int RB, int VW, bool PLAIN>
__global__ __launch_bounds__(kNmfThreads, (kNmfWavesPerSimd<T, R, RB, VW>)) void nmf_update_z_kernel(Geom g, const T *__restrict__ W, int64_t ldw, NmfManip manip,
                                                                  const float *__restrict__ Mp,
                                                                  const float *__restrict__ MzCur,
                                                                  float *__restrict__ MzNew, const float *__restrict__ G,
                                                                  float eps, int cblocks)
{
    using M = NmfMat<R>;
    using acc_t = typename M::acc_t;
    constexpr int NB = kNmfOwn / R, ITEMS = NB * M::NR / kNmfWaves;
    constexpr int U = 8;
    static __shared__ float stage[kNmfWaves * NB * M::NR * 64];
    const int64_t id = nmf_block_id(), t = id / cblocks;
    if (t >= nmf_tiles(g)) return;
    const int cb = (int)(id - t * cblocks);
    int ti, tj, rt, ct;
    nmf_tile_extent(g, t, ti, tj, rt, ct);
    if (cb * kNmfOwn >= ct) return; // a cut-off tile (uniform over the workgroup)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane % R, lk = lane / R, k = g.k;
    const int j = cb * kNmfOwn + NB * li;
    const float *mp = Mp + t * (int64_t)g.r * k;
    const float *mzc = MzCur + t * (int64_t)k * g.c;
    float *mzn = MzNew + t * (int64_t)k * g.c;
    const float *gt = G + t * (int64_t)k * k;
    const T *wtile = W + (int64_t)ti * g.r * ldw + (int64_t)tj * g.c;
    const int steps = (rt + M::KS - 1) / M::KS;
    const int ibeg = nmf_share(steps, wave, kNmfWaves) * M::KS;
    const int iend = wave + 1 < kNmfWaves ? nmf_share(steps, wave + 1, kNmfWaves) * M::KS : rt;

    for (int l0 = 0; l0 < k; l0 += RB * R) {
        int rank[RB]; // ranks beyond k repeat the last one; their sums are never stored
#pragma unroll
        for (int q = 0; q < RB; ++q) rank[q] = (l0 + q * R + li < k) ? l0 + q * R + li : k - 1;
        acc_t acc[RB][NB];
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[q][b] = nmf_zero<R>();

        // U steps are in flight: as soon as a step's operands have gone to the matrix cores, the same registers are
        // asked for the step U further on.  Whole batches of steps need no clamps (lane pointers plus offsets that all lanes
        // share); what is left at the end of the wavefront's rows goes in half batches with clamps and zeros.  (Clamps, multiplications
        // and selects for every element kept the vector ALUs busier than the matrix cores: 52 us against 40 for the M_z
        // update of the size above.)
        NmfPack<T, NB> wraw[U];
        float praw[U][RB];
        const int batches = (iend - ibeg) / (U * M::KS);
        const T *wl = wtile + (int64_t)(ibeg + lk) * ldw + (j < ct ? j : 0);
        const float *pl[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) pl[q] = mp + (int64_t)(ibeg + lk) * k + rank[q];
        auto request = [&](int u) __attribute__((always_inline)) {
            nmf_load<VW>(wraw[u], wl + u * M::KS * ldw, 0, ct - j);
#pragma unroll
            for (int q = 0; q < RB; ++q) praw[u][q] = pl[q][(int64_t)(u * M::KS) * k];
            nmf_requested();
        };
        {
            if (batches > 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) request(u);
                for (int bt = 1; bt <= batches; ++bt) {
                    if (bt < batches) { // else the last batch is asked for again and not looked at
                        wl += U * M::KS * ldw;
#pragma unroll
                        for (int q = 0; q < RB; ++q) pl[q] += (int64_t)(U * M::KS) * k;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        float mv[NB];
#pragma unroll
                        for (int b = 0; b < NB; ++b) mv[b] = nmf_mag<T, PLAIN>(wraw[u].w, b, manip);
#pragma unroll
                        for (int q = 0; q < RB; ++q)
#pragma unroll
                            for (int b = 0; b < NB; ++b) acc[q][b] = M::mma(praw[u][q], mv[b], acc[q][b]);
                        request(u);
                    }
                }
            }
#pragma clang loop unroll(disable)
            for (int i0 = ibeg + batches * U * M::KS; i0 < iend; i0 += U / 2 * M::KS) {
#pragma unroll
                for (int u = 0; u < U / 2; ++u) {
                    const int i = i0 + u * M::KS + lk, ic = i < rt ? i : rt - 1;
                    nmf_load<VW>(wraw[u], wtile + (int64_t)ic * ldw + (j < ct ? j : 0), 0, ct - j);
#pragma unroll
                    for (int q = 0; q < RB; ++q) praw[u][q] = mp[(int64_t)ic * k + rank[q]];
                }
#pragma unroll
                for (int u = 0; u < U / 2; ++u) {
                    const bool in = i0 + u * M::KS + lk < iend;
#pragma unroll
                    for (int q = 0; q < RB; ++q)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[q][b] = M::mma(in ? praw[u][q] : 0.f, in ? nmf_mag<T, PLAIN>(wraw[u].w, b, manip) : 0.f, acc[q][b]);
                }
            }
        }

        float num[RB][ITEMS];
#pragma unroll
        for (int q = 0; q < RB; ++q) nmf_reduce<R, NB, ITEMS>(stage, acc[q], num[q], wave, lane);

        // denominators: rows of the Gram matrix times the old M_z
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[q][b] = nmf_zero<R>();
        const int gsteps = (k + M::KS - 1) / M::KS;
        const int gend = gsteps * (wave + 1) / kNmfWaves;
#pragma clang loop unroll(disable)
        for (int s0 = gsteps * wave / kNmfWaves; s0 < gend; s0 += 4) { // four steps' loads together
            NmfPack<float, NB> z[4];
            float ga[4][RB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = (s0 + u) * M::KS + lk, lc = l < k ? l : k - 1;
                nmf_load<VW>(z[u], mzc + (int64_t)lc * g.c, j, ct);
#pragma unroll
                for (int q = 0; q < RB; ++q) ga[u][q] = gt[(int64_t)lc * k + rank[q]]; // symmetric
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = s0 + u < gend && (s0 + u) * M::KS + lk < k;
#pragma unroll
                for (int q = 0; q < RB; ++q)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[q][b] = M::mma(in ? ga[u][q] : 0.f, in ? nmf_elem<float>(z[u].w, b) : 0.f, acc[q][b]);
            }
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            float den[ITEMS];
            nmf_reduce<R, NB, ITEMS>(stage, acc[q], den, wave, lane);
#pragma unroll
            for (int e = 0; e < ITEMS; ++e) {
                const int l = l0 + q * R + M::row(wave * (M::NR / kNmfWaves) + e / NB, lane), jj = j + e % NB;
                if (l < k && jj < ct) {
                    const int64_t at = (int64_t)l * g.c + jj;
                    mzn[at] = mzc[at] * num[q][e] / (den[e] + eps);
                }
            }
        }
    }
}

// M_p update.  Workgroup = (tile, 64 rows); block b of the result holds rows b * R + (its row index), lane li = rank.
template <typename T, int R, int RB, int VW, bool PLAIN>
__global__ __launch_bounds__(kNmfThreads, (VW == 1 || RB > 1 || sizeof(T) == 4) ? 2 : 3) void nmf_update_p_kernel(Geom g, const T *__restrict__ W, int64_t ldw, NmfManip manip,
                                                                  const float *__restrict__ MpCur,
                                                                  const float *__restrict__ Mz,
                                                                  float *__restrict__ MpNew, const float *__restrict__ G,
                                                                  float eps, int rblocks)
{
    using M = NmfMat<R>;
    using acc_t = typename M::acc_t;
    constexpr int NB = kNmfOwn / R, ITEMS = NB * M::NR / kNmfWaves;
    constexpr int ES = (int)sizeof(T), ZV = VW > 1 ? 4 : 1;      // elements per piece: VW of W, ZV of M_z
    constexpr int WPITCH = kNmfChunk * ES + 16, ZPITCH = kNmfChunk * 4 + 16; // bytes; eight rows' 16-byte reads miss each other
    constexpr int WBYTES = kNmfOwn * WPITCH, WAVE_BYTES = WBYTES + RB * R * ZPITCH;
    constexpr int STAGE_BYTES = kNmfWaves * NB * M::NR * 64 * 4;
    constexpr int LDS_BYTES = kNmfWaves * WAVE_BYTES > STAGE_BYTES ? kNmfWaves * WAVE_BYTES : STAGE_BYTES;
    __align__(16) static __shared__ unsigned char lds[LDS_BYTES];
    float *stage = reinterpret_cast<float *>(lds);
    const int64_t id = nmf_block_id(), t = id / rblocks;
    if (t >= nmf_tiles(g)) return;
    const int rblk = (int)(id - t * rblocks);
    int ti, tj, rt, ct;
    nmf_tile_extent(g, t, ti, tj, rt, ct);
    if (rblk * kNmfOwn >= rt) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane % R, lk = lane / R, k = g.k;
    const float *mz = Mz + t * (int64_t)k * g.c;
    const float *mpc = MpCur + t * (int64_t)g.r * k;
    float *mpn = MpNew + t * (int64_t)g.r * k;
    const float *gt = G + t * (int64_t)k * k;
    const T *wtile = W + (int64_t)ti * g.r * ldw + (int64_t)tj * g.c;
    int row[NB]; // rows beyond the tile repeat its last one; their sums are never stored
#pragma unroll
    for (int b = 0; b < NB; ++b) row[b] = (rblk * kNmfOwn + b * R + li < rt) ? rblk * kNmfOwn + b * R + li : rt - 1;
    const int chunks = (ct + kNmfChunk - 1) / kNmfChunk;
    const int sbeg = nmf_share(chunks, wave, kNmfWaves), send = nmf_share(chunks, wave + 1, kNmfWaves);
    unsigned char *wlds = lds + wave * WAVE_BYTES, *zlds = wlds + WBYTES;

    for (int l0 = 0; l0 < k; l0 += RB * R) {
        if (l0 > 0) __syncthreads(); // the chunks overlay the staging area, whose last sums a slower wavefront may still be reading
        int rank[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) rank[q] = (l0 + q * R + li < k) ? l0 + q * R + li : k - 1;
        acc_t acc[RB][NB];
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[q][b] = nmf_zero<R>();

        // Rows of the result across the lanes and 8 columns per lane would be 64 separate cache lines per load (measured:
        // 44 us against 42 for the M_p update of the size
        // above, 11 against 9 on 192 x 512 tiles), so the wavefront copies chunks of 32 columns into LDS
        // row by row, its own part of it (no barrier), the next chunk's loads in flight meanwhile.  Columns past the tile
        // are stored as zero.
        using WPiece = NmfRaw<VW * ES>;
        using ZPiece = NmfRaw<ZV * 4>;
        constexpr int WPPR = kNmfChunk / VW, WSTEP = 64 / WPPR, WL = kNmfOwn / WSTEP;     // pieces per row, rows and loads
        constexpr int ZPPR = kNmfChunk / ZV, ZSTEP = 64 / ZPPR, ZL = RB * R / ZSTEP;
        const int wr = lane / WPPR, wc = lane % WPPR * VW, zr = lane / ZPPR, zc = lane % ZPPR * ZV;
        typename WPiece::type wraw[WL];
        typename ZPiece::type zraw[ZL];
        auto request = [&](int s) __attribute__((always_inline)) {
            const int j = s * kNmfChunk, jw = j + wc < ct ? j + wc : 0, jz = j + zc < ct ? j + zc : 0;
            int r0 = rblk * kNmfOwn + wr, z0 = l0 + zr;
            // the addresses are formed anew for every chunk: kept from chunk to chunk they would take 32 registers
            asm volatile("" : "+v"(r0), "+v"(z0));
#pragma unroll
            for (int i = 0; i < WL; ++i) {
                const int r = r0 + i * WSTEP;
                wraw[i] = *reinterpret_cast<const typename WPiece::type *>(wtile + (int64_t)(r < rt ? r : rt - 1) * ldw + jw);
            }
#pragma unroll
            for (int i = 0; i < ZL; ++i) {
                const int l = z0 + i * ZSTEP;
                zraw[i] = *reinterpret_cast<const typename ZPiece::type *>(mz + (int64_t)(l < k ? l : k - 1) * g.c + jz);
            }
            nmf_requested();
        };
        if (sbeg < send) request(sbeg);
#pragma clang loop unroll(disable)
        for (int s = sbeg; s < send; ++s) {
            const int j = s * kNmfChunk;
#pragma unroll
            for (int i = 0; i < WL; ++i)
                *reinterpret_cast<typename WPiece::type *>(wlds + (wr + i * WSTEP) * WPITCH + wc * ES) =
                    j + wc < ct ? wraw[i] : WPiece::zero();
#pragma unroll
            for (int i = 0; i < ZL; ++i)
                *reinterpret_cast<typename ZPiece::type *>(zlds + (zr + i * ZSTEP) * ZPITCH + zc * 4) =
                    j + zc < ct ? zraw[i] : ZPiece::zero();
            if (s + 1 < send) request(s + 1);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int h = 0; h < kNmfChunk / (8 * M::KS); ++h) {
                const int at = h * 8 * M::KS + 8 * lk;
                NmfPack<T, 8> w[NB];
                NmfPack<float, 8> z[RB];
#pragma unroll
                for (int b = 0; b < NB; ++b) nmf_lds_read(w[b].w, wlds + (b * R + li) * WPITCH + at * ES);
#pragma unroll
                for (int q = 0; q < RB; ++q) nmf_lds_read(z[q].w, zlds + (q * R + li) * ZPITCH + at * 4);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float mv = nmf_mag<T, PLAIN>(w[b].w, u, manip);
#pragma unroll
                        for (int q = 0; q < RB; ++q) acc[q][b] = M::mma(mv, nmf_elem<float>(z[q].w, u), acc[q][b]);
                    }
            }
            __builtin_amdgcn_wave_barrier(); // the chunk has been read before the next one is stored
        }

        float num[RB][ITEMS];
#pragma unroll
        for (int q = 0; q < RB; ++q) nmf_reduce<R, NB, ITEMS>(stage, acc[q], num[q], wave, lane);

        // denominators: the old M_p times columns of the Gram matrix
#pragma unroll
        for (int q = 0; q < RB; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[q][b] = nmf_zero<R>();
        const int gsteps = (k + M::KS - 1) / M::KS;
        const int gend = gsteps * (wave + 1) / kNmfWaves;
#pragma clang loop unroll(disable)
        for (int s0 = gsteps * wave / kNmfWaves; s0 < gend; s0 += 4) { // four steps' loads together
            float p[4][NB], gb[4][RB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int l = (s0 + u) * M::KS + lk, lc = l < k ? l : k - 1;
#pragma unroll
                for (int b = 0; b < NB; ++b) p[u][b] = mpc[(int64_t)row[b] * k + lc];
#pragma unroll
                for (int q = 0; q < RB; ++q) gb[u][q] = gt[(int64_t)lc * k + rank[q]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = s0 + u < gend && (s0 + u) * M::KS + lk < k;
#pragma unroll
                for (int q = 0; q < RB; ++q)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[q][b] = M::mma(in ? p[u][b] : 0.f, in ? gb[u][q] : 0.f, acc[q][b]);
            }
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            float den[ITEMS];
            nmf_reduce<R, NB, ITEMS>(stage, acc[q], den, wave, lane);
#pragma unroll
            for (int e = 0; e < ITEMS; ++e) {
                const int i = rblk * kNmfOwn + (e % NB) * R + M::row(wave * (M::NR / kNmfWaves) + e / NB, lane);
                const int l = l0 + q * R + li;
                if (i < rt && l < k) {
                    const int64_t at = (int64_t)i * k + l;
                    mpn[at] = mpc[at] * num[q][e] / (den[e] + eps);
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void nmf_copy_kernel(const float *__restrict__ src, float *__restrict__ dst, int64_t count)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256) dst[e] = src[e];
}

static int nmf_copy(const float *src, float *dst, int64_t count, hipStream_t stream)
{
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    LRBI_LAUNCH(nmf_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, src, dst, count);
    return LRBI_OK;
}

template <typename T, int R, int RB, int VW, bool PLAIN>
static int nmf_iterate(const Geom &g, const void *dW, int64_t ldw, int method, float w_threshold, float amplify, float *dMp,
                       float *dMz, int iters, float eps, float *wsMp, float *wsMz, float *wsG, hipStream_t stream)
{
    const int64_t tiles = (int64_t)g.tile_rows * g.tile_cols;
    const int cblocks = (g.c + kNmfOwn - 1) / kNmfOwn, rblocks = (g.r + kNmfOwn - 1) / kNmfOwn;
    const int kblocks = (g.k + R - 1) / R, pairs = kblocks * (kblocks + 1) / 2;
    if (tiles * cblocks > 0x7FFFFFFF || tiles * rblocks > 0x7FFFFFFF || tiles * pairs > 0x7FFFFFFF) return LRBI_ERR_SHAPE;
    const NmfManip manip{method, w_threshold, amplify};
    float *mp_cur = dMp, *mp_new = wsMp, *mz_cur = dMz, *mz_new = wsMz;
    for (int it = 0; it < iters; ++it) {
        LRBI_LAUNCH((nmf_gram_kernel<R, VW, false>), wide_grid(tiles * pairs, kGramThreads), dim3(kGramThreads), 0, stream, g, mp_cur,
                    wsG, kblocks, pairs);
        LRBI_LAUNCH((nmf_update_z_kernel<T, R, RB, VW, PLAIN>), wide_grid(tiles * cblocks, kNmfThreads), dim3(kNmfThreads), 0, stream, g,
                    (const T *)dW, ldw, manip, mp_cur, mz_cur, mz_new, wsG, eps, cblocks);
        LRBI_LAUNCH((nmf_gram_kernel<R, VW, true>), wide_grid(tiles * pairs, kGramThreads), dim3(kGramThreads), 0, stream, g, mz_new,
                    wsG, kblocks, pairs);
        LRBI_LAUNCH((nmf_update_p_kernel<T, R, RB, VW, PLAIN>), wide_grid(tiles * rblocks, kNmfThreads), dim3(kNmfThreads), 0, stream, g,
                    (const T *)dW, ldw, manip, mp_cur, mz_new, mp_new, wsG, eps, rblocks);
        float *tmp = mp_cur;
        mp_cur = mp_new;
        mp_new = tmp;
        tmp = mz_cur;
        mz_cur = mz_new;
        mz_new = tmp;
    }
    if (mp_cur != dMp) { // an odd number of iterations ends in the workspace
        int rc = nmf_copy(mp_cur, dMp, tiles * g.r * g.k, stream);
        if (rc != LRBI_OK) return rc;
        rc = nmf_copy(mz_cur, dMz, tiles * (int64_t)g.k * g.c, stream);
        if (rc != LRBI_OK) return rc;
    }
    return LRBI_OK;
}

template <typename T>
static int nmf_dtype(const Geom &g, const void *dW, int64_t ldw, int method, float w_threshold, float amplify, float *dMp,
                     float *dMz, int iters, float eps, float *wsMp, float *wsMz, float *wsG, hipStream_t stream)
{
    // elements per load: 8, 4 or 1.  A piece lies inside a tile and inside a row as a whole (c and n are multiples of
    // it) and is aligned to its size or to 16 bytes; the factors are read in 16-byte pieces from 4 elements up.
    const auto fits = [&](int vw) {
        const int64_t bytes = (int64_t)vw * (int64_t)sizeof(T) < 16 ? (int64_t)vw * (int64_t)sizeof(T) : 16;
        return g.c % vw == 0 && g.n % vw == 0 && (ldw * (int64_t)sizeof(T)) % bytes == 0 && ((uintptr_t)dW % bytes) == 0 &&
               (((uintptr_t)dMz | (uintptr_t)wsMz) & 15) == 0;
    };
#define LRBI_NMF_ARGS g, dW, ldw, method, w_threshold, amplify, dMp, dMz, iters, eps, wsMp, wsMz, wsG, stream
#define LRBI_NMF_RANKS(VW, PLAIN)                                                                           \
    return g.k <= 16   ? nmf_iterate<T, 16, 1, VW, PLAIN>(LRBI_NMF_ARGS)                                    \
           : g.k <= 32 ? nmf_iterate<T, 32, 1, VW, PLAIN>(LRBI_NMF_ARGS)                                    \
                       : nmf_iterate<T, 32, 2, VW, PLAIN>(LRBI_NMF_ARGS)
#define LRBI_NMF_METHOD(VW)                                                                                 \
    if (method == 1) { LRBI_NMF_RANKS(VW, true); }                                                          \
    LRBI_NMF_RANKS(VW, false)
    if constexpr (sizeof(T) == 2) {
        if (fits(8)) { LRBI_NMF_METHOD(8); }
    }
    if (fits(4)) { LRBI_NMF_METHOD(4); }
    LRBI_NMF_METHOD(1);
#undef LRBI_NMF_METHOD
#undef LRBI_NMF_RANKS
#undef LRBI_NMF_ARGS
}

uint64_t nmf_workspace_bytes(const Geom &g)
{
    const uint64_t tiles = (uint64_t)g.tile_rows * g.tile_cols;
    const uint64_t mp = (tiles * g.r * g.k * 4 + 255) / 256 * 256;
    const uint64_t mz = (tiles * g.k * g.c * 4 + 255) / 256 * 256;
    const uint64_t gram = (tiles * g.k * g.k * 4 + 255) / 256 * 256;
    return mp + mz + gram;
}

int launch_nmf(const Geom &g, lrbi_dtype dt, const void *dW, int64_t ldw, int method, float w_threshold, float amplify,
               float *dMp, float *dMz, int iters, float eps, void *dWorkspace, hipStream_t stream)
{
    if (g.k > kNmfMaxK) return LRBI_ERR_RANK;
    const uint64_t tiles = (uint64_t)g.tile_rows * g.tile_cols;
    float *wsMp = (float *)dWorkspace;
    float *wsMz = (float *)((char *)dWorkspace + (tiles * g.r * g.k * 4 + 255) / 256 * 256);
    float *wsG = (float *)((char *)wsMz + (tiles * g.k * g.c * 4 + 255) / 256 * 256);
    // the second buffers start as copies, so that what a cut-off tile does not use is the same in both
    int rc = nmf_copy(dMp, wsMp, (int64_t)(tiles * g.r * g.k), stream);
    if (rc != LRBI_OK) return rc;
    rc = nmf_copy(dMz, wsMz, (int64_t)(tiles * g.k * g.c), stream);
    if (rc != LRBI_OK) return rc;
    switch (dt) {
    case LRBI_F32: return nmf_dtype<float>(g, dW, ldw, method, w_threshold, amplify, dMp, dMz, iters, eps, wsMp, wsMz, wsG, stream);
    case LRBI_F16: return nmf_dtype<__half>(g, dW, ldw, method, w_threshold, amplify, dMp, dMz, iters, eps, wsMp, wsMz, wsG, stream);
    case LRBI_BF16:
        return nmf_dtype<__hip_bfloat16>(g, dW, ldw, method, w_threshold, amplify, dMp, dMz, iters, eps, wsMp, wsMz, wsG, stream);
    default: return LRBI_ERR_DTYPE;
    }
}

} // namespace lrbi
