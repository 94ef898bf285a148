// Masked products in fp32 on the matrix cores (v_mfma_f32_32x32x2): the forward product and the weight gradient of
// fp32 layers, and the transposed product of every type where the 16-bit matrix-core kernels do not apply (fp32, and
// 16-bit rows that are not whole aligned 16-byte pieces).  The products are exact fp32 fused multiply-adds, the sums
// fp32 in a fixed order.
//
// Operands go from global memory (the caches) to registers in the instruction's lane layout: lane l holds row (column)
// l & 31 of the left (right) operand at reduction index l >> 5.  One step of the instruction takes 64 cycles, a step's
// operand loads a few, so tiles through LDS would buy nothing.  A workgroup owns one block of outputs and its
// wavefronts take chunks of the reduction in turn (the layers are small: the blocks of outputs alone would leave most
// of the chip idle); their sums are added through LDS in wavefront order.  Kernel times at 500 x 800 in 100 x 100 tiles,
// 64 columns, against one wavefront per 64 columns (a row) on the vector ALUs: product 131 -> 12.9 us, transposed 522 -> 10.1,
// gradient 12.9 -> 8.1 (the three calls of a training step 660 -> 31 us), most of it the launch and the two chains of
// factor loads behind a mask word; 4096 x 4096 in 512 x 512 tiles at 64 columns 55, 62 and 55 us (2.1 GFLOP: 14 us at
// the instruction's rate, the reads of W 13 us), transposed at 8 columns 4019 -> 63 us.  Relative error against 64 bits
// at 500 x 800, 64 columns: 7.2e-8 -> 6.3e-8, 1.4e-7 -> 7.1e-8 and 1.4e-7 -> 1.1e-7.
//
// A zeroed weight still meets its other operand inside the instruction, and 0 * inf is NaN.  The products therefore
// watch their unmasked operand: batch columns that hold an infinity or a NaN are formed again, stepping over the
// pruned weights; the others do not meet them.
#include <float.h>
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "lrbi_internal.hpp"

namespace lrbi {

static constexpr int kF32Waves = 8; // wavefronts of a product's workgroup, but for a reduction of one chunk
static constexpr int64_t kMaxColumnsT = 4 * 65535; // the transposed product's limit on N, part of the interface (lrbi.h)
static constexpr int kF32Chunk = 64; // reduction steps of one wavefront between two mask decodes

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

__device__ __forceinline__ f32x16_t mfma_32x32x2(float a, float b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
// row of accumulator element v (its column is lane & 31)
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

__device__ __forceinline__ float as_f32(float v) { return v; }
__device__ __forceinline__ float as_f32(__half v) { return __half2float(v); }
__device__ __forceinline__ float as_f32(__hip_bfloat16 v) { return __bfloat162float(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ __half from_f32<__half>(float v) { return __float2half_rn(v); }
template <> __device__ __forceinline__ __hip_bfloat16 from_f32<__hip_bfloat16>(float v) { return __float2bfloat16(v); }

__device__ __forceinline__ int64_t at_most(int64_t i, int64_t last) { return i < last ? i : last; }

// The batch columns (bits) of a workgroup's block that hold a value that is not finite; bad[b]: the wavefront's lanes that have met
// one in their columns (lane & 31) + 32 b.  One value for the whole workgroup; columns from N on, which repeat the last one, are left out.
template <int NQ, int WAVES>
__device__ __forceinline__ unsigned long long bad_columns(const unsigned long long (&bad)[NQ], int64_t cols)
{
    static __shared__ uint32_t met[WAVES * NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b)
        if ((threadIdx.x & 63) == 0) met[(threadIdx.x >> 6) * NQ + b] = (uint32_t)bad[b] | (uint32_t)(bad[b] >> 32);
    __syncthreads();
    unsigned long long all = 0ull;
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
#pragma unroll
        for (int b = 0; b < NQ; ++b) all |= (unsigned long long)met[w * NQ + b] << (32 * b);
    return cols < 64 ? all & ((1ull << cols) - 1ull) : all;
}

// How a wavefront forms a row (or column) of results in those columns again: lane = (part of the reduction, column).  The
// parts' sums are in double and a lane stops at a NaN, which nothing that follows changes.
struct BadLanes {
    int parts, part, qlanes;
    int64_t q;     // column of the block
    bool last_one; // no column of its own: repeats the last
    __device__ BadLanes(unsigned long long columns)
    {
        const int lane = threadIdx.x & 63, count = __builtin_popcountll(columns);
        qlanes = 1;
        while (qlanes < count) qlanes *= 2;
        parts = 64 / qlanes;
        part = lane / qlanes;
        const int ql = lane % qlanes;
        last_one = ql >= count;
        for (int skip = last_one ? count - 1 : ql; skip > 0; --skip) columns &= columns - 1ull;
        q = __builtin_ctzll(columns);
    }
    __device__ double total(double s) const
    {
        for (int d = qlanes; d < 64; d *= 2) s += __shfl_xor(s, d, 64);
        return s;
    }
    __device__ bool stores() const { return part == 0 && !last_one; }
};

// s += sum of w[at] x[at], at = base + the set bits, four at a time in flight
template <typename T>
__device__ __forceinline__ void add_kept(double &s, unsigned long long bits, int64_t base, const T *w, int64_t wstride, const T *x,
                                         int64_t xstride)
{
    while (bits && s == s) {
        int64_t at[4];
        bool live[4];
        T wv[4], xv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            live[e] = bits != 0ull;
            at[e] = live[e] ? base + __builtin_ctzll(bits) : at[0];
            bits &= bits - 1ull;
            wv[e] = w[at[e] * wstride];
            xv[e] = x[at[e] * xstride];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (live[e]) s = __fma_rn((double)as_f32(wv[e]), (double)as_f32(xv[e]), s);
    }
}

// mask word of row `row`, word column w
template <bool AHEAD = false>
__device__ __forceinline__ uint32_t row_word(const Geom &g, const uint32_t *Ip, const uint32_t *Iz, int64_t row, int w)
{
    const int ti = (int)(row / g.r), il = (int)(row - (int64_t)ti * g.r);
    return decode_word<AHEAD>(g, Ip, Iz, ti, il, w);
}

// adds the wavefronts' sums of a 32 x (32 NQ) block in wavefront order and stores it, without the batch columns in `skip`
template <typename T, int NQ, int WAVES>
__device__ __forceinline__ void reduce_store(float (*red)[1024], const f32x16_t (&acc)[NQ], int64_t row0, int64_t rows,
                                             int64_t q0, int64_t N, unsigned long long skip, T *__restrict__ out, int64_t ldo)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
        if (b) __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][acc_row(v, lane) * 32 + (lane & 31)] = acc[b][v];
        __syncthreads();
        for (int e = tid; e < 1024; e += 64 * WAVES) {
            double s = (double)red[0][e]; // rounded once
#pragma unroll
            for (int w = 1; w < WAVES; ++w) s += (double)red[w][e];
            const int64_t i = row0 + (e >> 5), q = q0 + 32 * b + (e & 31);
            if (i < rows && q < N && !((skip >> (32 * b + (e & 31))) & 1ull)) out[i * ldo + q] = from_f32<T>((float)s);
        }
    }
}

// dX = (W o I_a)^T dY.  Workgroup = 32 columns of W (rows of dX) x 32 NQ batch columns; a wavefront's chunk is 64
// rows of W, whose 64 mask words (one per row: the block's columns are one word) its lanes decode together.
template <typename T, int NQ, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void f32_gemm_t_kernel(Geom g, const T *__restrict__ W, int64_t ldw,
                                                                 const uint32_t *__restrict__ Ip,
                                                                 const uint32_t *__restrict__ Iz,
                                                                 const T *__restrict__ DY, int64_t lddy, int64_t N,
                                                                 T *__restrict__ DX, int64_t lddx, int jblocks)
{
    static __shared__ float red[WAVES][1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
    const unsigned block = (unsigned)wide_block();
    const int jb = (int)(block % (unsigned)jblocks);
    const int64_t j0 = 32 * (int64_t)jb, q0 = 32 * NQ * (int64_t)(block / (unsigned)jblocks);
    if (q0 >= N) return; // past the last workgroup of the grid's second dimension
    const T *wcol = W + at_most(j0 + li, g.n - 1); // clamped: what lies beyond has no mask bit, or is not stored
    const T *ycol[NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b) ycol[b] = DY + at_most(q0 + 32 * b + li, N - 1);

    constexpr int U = 8; // steps of the instruction whose operands are requested together
    f32x16_t acc[NQ] = {};
    unsigned long long bad[NQ] = {}; // lanes; in scalar registers
    for (int64_t i0 = (int64_t)kF32Chunk * wave; i0 < g.m; i0 += kF32Chunk * WAVES) {
        T w[2][U], y[2][U][NQ];
        const auto load = [&](int s0, T (&wv)[U], T (&yv)[U][NQ]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = at_most(i0 + 2 * (s0 + u) + half, g.m - 1);
                wv[u] = wcol[i * ldw];
#pragma unroll
                for (int b = 0; b < NQ; ++b) yv[u][b] = ycol[b][i * lddy];
            }
        };
        load(0, w[0], y[0]);
        // (not with four I_z rows in flight where there are two batch blocks: they took the kernel from 128 to 129 registers and
        // from two workgroups a compute unit to one, 300 x 8000, 1024 columns 112 -> 172 us)
        const uint32_t words = (i0 + lane < g.m) ? row_word<NQ == 1 || WAVES == 1>(g, Ip, Iz, i0 + lane, jb) : 0u;
#pragma unroll
        for (int s = 0; s < kF32Chunk / 2 / U; ++s) {
            if (s + 1 < kF32Chunk / 2 / U) load((s + 1) * U, w[(s + 1) & 1], y[(s + 1) & 1]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t word = __shfl(words, 2 * (s * U + u) + half, 64);
                const float a = ((word >> li) & 1u) ? as_f32(w[s & 1][u]) : 0.f;
#pragma unroll
                for (int b = 0; b < NQ; ++b) {
                    const float x = as_f32(y[s & 1][u][b]);
                    bad[b] |= __ballot(!(fabsf(x) <= FLT_MAX));
                    acc[b] = mfma_32x32x2(a, x, acc[b]);
                }
            }
        }
    }
    const unsigned long long again = bad_columns<NQ, WAVES>(bad, N - q0);
    reduce_store<T, NQ, WAVES>(red, acc, j0, g.n, q0, N, again, DX, lddx);
    if (!again) return;
    // a wavefront forms four columns of W; the mask words of 64 rows at a time are decoded once for them
    const BadLanes lanes(again);
    unsigned long long mine = 0ull; // the lane's rows of 64
    for (int i = lanes.part; i < 64; i += lanes.parts) mine |= 1ull << i;
    constexpr int JW = 4;
#pragma clang loop unroll(disable)
    for (int turn = 0; turn < 32 / (JW * WAVES); ++turn) {
        const int jl = JW * (turn * WAVES + wave);
        double s[JW] = {};
        for (int64_t i0 = 0; i0 < g.m; i0 += 64) {
            const uint32_t words = (i0 + lane < g.m) ? row_word(g, Ip, Iz, i0 + lane, jb) : 0u;
            bool open = false;
#pragma unroll
            for (int u = 0; u < JW; ++u) { // (no bit is set in rows from m on and in columns from n on)
                const unsigned long long rows = __ballot((words >> (jl + u)) & 1u) & mine;
                add_kept<T>(s[u], rows, i0, W + at_most(j0 + jl + u, g.n - 1), ldw, DY + q0 + lanes.q, lddy);
                open |= s[u] == s[u];
            }
            if (!__any(open)) break;
        }
#pragma unroll
        for (int u = 0; u < JW; ++u) {
            const double sum = lanes.total(s[u]);
            const int64_t j = j0 + jl + u;
            if (lanes.stores() && j < g.n) DX[j * lddx + q0 + lanes.q] = from_f32<T>((float)sum);
        }
    }
}

// Y = (W o I_a) X, fp32.  Workgroup = 32 rows of W x 32 NQ batch columns; a wavefront's chunk is 64 columns of W, two
// mask words per row.  A lane reads four consecutive weights of its row: the instruction's two reduction indices of
// step e are columns e and 4 + e of a group of eight, so the lane halves hold adjacent 16-byte pieces.
template <int NQ, bool VEC, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void f32_gemm_kernel(Geom g, const float *__restrict__ W, int64_t ldw,
                                                               const uint32_t *__restrict__ Ip,
                                                               const uint32_t *__restrict__ Iz,
                                                               const float *__restrict__ X, int64_t ldx, int64_t N,
                                                               float *__restrict__ Y, int64_t ldy, int iblocks)
{
    static __shared__ float red[WAVES][1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
    const unsigned block = (unsigned)wide_block();
    const int64_t i0 = 32 * (int64_t)(block % (unsigned)iblocks);
    const int64_t q0 = 32 * NQ * (int64_t)(block / (unsigned)iblocks);
    if (q0 >= N) return; // past the last workgroup of the grid's second dimension
    const int64_t row = at_most(i0 + li, g.m - 1);
    const float *wrow = W + row * ldw;
    const float *xcol[NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b) xcol[b] = X + at_most(q0 + 32 * b + li, N - 1);

    constexpr int G = kF32Chunk / 8; // groups of eight columns per chunk
    // the sums of 32 columns go into doubles: one fp32 chain over a wavefront's whole share of the row would round more
    // often than a sum spread over 64 lanes (relative error 1.5e-7 at 300 x 4000, where this gives 6.2e-8)
    double sum[NQ][16] = {};
    unsigned long long bad[NQ] = {}; // lanes; in scalar registers
    for (int64_t j0 = (int64_t)kF32Chunk * wave; j0 < g.n; j0 += kF32Chunk * WAVES) {
        float w[2][4], x[2][4][NQ];
        const auto load = [&](int gq, float (&wv)[4], float (&xv)[4][NQ]) {
            const int64_t j = j0 + 8 * gq + 4 * half;
            if (VEC) {
                const float4 p = *reinterpret_cast<const float4 *>(wrow + at_most(j, g.n - 4));
                wv[0] = p.x; wv[1] = p.y; wv[2] = p.z; wv[3] = p.w;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t je = at_most(j + e, g.n - 1);
                if (!VEC) wv[e] = wrow[je];
#pragma unroll
                for (int b = 0; b < NQ; ++b) xv[e][b] = xcol[b][je * ldx];
            }
        };
        load(0, w[0], x[0]);
        const uint32_t words = row_word(g, Ip, Iz, row, (int)(j0 >> 5) + half); // no bits at or beyond column n
        f32x16_t acc[NQ];
        const uint32_t word01[2] = {(uint32_t)__shfl(words, li, 64), (uint32_t)__shfl(words, li + 32, 64)};
#pragma unroll
        for (int gq = 0; gq < G; ++gq) {
            if (gq % 4 == 0) {
#pragma unroll
                for (int b = 0; b < NQ; ++b) acc[b] = f32x16_t{};
            }
            if (gq + 1 < G) load(gq + 1, w[(gq + 1) & 1], x[(gq + 1) & 1]);
            const uint32_t bits = word01[gq >> 2] >> (8 * (gq & 3) + 4 * half);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = ((bits >> e) & 1u) ? w[gq & 1][e] : 0.f;
#pragma unroll
                for (int b = 0; b < NQ; ++b) {
                    const float v = x[gq & 1][e][b];
                    bad[b] |= __ballot(!(fabsf(v) <= FLT_MAX));
                    acc[b] = mfma_32x32x2(a, v, acc[b]);
                }
            }
            if (gq % 4 == 3) {
#pragma unroll
                for (int b = 0; b < NQ; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum[b][v] += (double)acc[b][v];
            }
        }
    }
    const unsigned long long again = bad_columns<NQ, WAVES>(bad, N - q0);
    f32x16_t acc[NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = (float)sum[b][v];
    reduce_store<float, NQ, WAVES>(red, acc, i0, g.m, q0, N, again, Y, ldy);
    if (!again) return;
    // a wavefront forms four rows; 64 mask words of a row are decoded at a time, and a lane takes every parts-th
    const BadLanes lanes(again);
    const int words_per_row = (int)((g.n + 31) / 32);
    for (int64_t i = i0 + wave; i < i0 + 32 && i < g.m; i += WAVES) {
        double s = 0.0;
        for (int w0 = 0; w0 < words_per_row && __any(s == s); w0 += 64) {
            const uint32_t words = row_word(g, Ip, Iz, i, w0 + lane); // none past the row
            for (int step = 0; step < 64; step += lanes.parts) {
                const int at = step + lanes.part;
                add_kept<float>(s, __shfl(words, at, 64), 32 * ((int64_t)w0 + at), W + i * ldw, 1, X + q0 + lanes.q, ldx);
            }
        }
        s = lanes.total(s);
        if (lanes.stores()) Y[i * ldy + q0 + lanes.q] = (float)s;
    }
}

// dW = (dY X^T) o I_a, fp32.  One wavefront per 32 x (32 NJ) block of dW (no reduction is split: the blocks are many
// and the batch is short).  Both operands are read four batch columns at a time, in the order described above.
// AHEAD: the mask words formed with four I_z rows in flight.
template <int NJ, bool VEC, bool AHEAD>
__global__ __launch_bounds__(256) void f32_grad_kernel(Geom g, const float *__restrict__ DY, int64_t lddy,
                                                       const float *__restrict__ X, int64_t ldx, int64_t N,
                                                       const uint32_t *__restrict__ Ip, const uint32_t *__restrict__ Iz,
                                                       float *__restrict__ DW, int64_t lddw, int64_t jblocks, int64_t blocks)
{
    const int lane = threadIdx.x & 63, li = lane & 31, half = lane >> 5;
    const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blk >= blocks) return; // whole wavefront; no barrier below
    const int64_t ib = blk / jblocks, i0 = 32 * ib, j0 = 32 * NJ * (blk - ib * jblocks);
    const float *yrow = DY + at_most(i0 + li, g.m - 1) * lddy;
    const float *xrow[NJ];
#pragma unroll
    for (int b = 0; b < NJ; ++b) xrow[b] = X + at_most(j0 + 32 * b + li, g.n - 1) * ldx;
    const auto load4 = [&](const float *p, int64_t q, float (&v)[4]) {
        if (VEC) {
            if (q < N) {
                const float4 f = *reinterpret_cast<const float4 *>(p + q);
                v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (q + e < N) ? p[q + e] : 0.f;
        }
    };
    // groups of eight batch columns go to two sums in turn: half the roundings of one chain, and two independent ones
    f32x16_t acc[2][NJ] = {};
    float y[2][4], x[2][NJ][4];
    const auto load = [&](int64_t q, float (&yv)[4], float (&xv)[NJ][4]) { // past the last batch column: zeros, nothing is read
        load4(yrow, q + 4 * half, yv);
#pragma unroll
        for (int b = 0; b < NJ; ++b) load4(xrow[b], q + 4 * half, xv[b]);
    };
    const auto mma = [&](float (&yv)[4], float (&xv)[NJ][4], f32x16_t (&c)[NJ]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < NJ; ++b) c[b] = mfma_32x32x2(yv[e], xv[b][e], c[b]);
    };
    load(0, y[0], x[0]);
    // the block's mask words: lane l < 32 holds row i0 + l of the first word column, the other half the second's
    const uint32_t words = row_word<AHEAD>(g, Ip, Iz, at_most(i0 + li, g.m - 1), (int)(j0 >> 5) + (NJ == 2 ? half : 0));
    for (int64_t q = 0; q < N; q += 16) {
        load(q + 8, y[1], x[1]);
        mma(y[0], x[0], acc[0]);
        if (q + 8 >= N) break;
        load(q + 16, y[0], x[0]);
        mma(y[1], x[1], acc[1]);
    }
#pragma unroll
    for (int b = 0; b < NJ; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][b][v] += acc[1][b][v];
#pragma unroll
    for (int b = 0; b < NJ; ++b) {
        const int64_t j = j0 + 32 * b + li;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rr = acc_row(v, lane);
            const uint32_t word = __shfl(words, rr + 32 * b, 64);
            if (i0 + rr < g.m && j < g.n) DW[(i0 + rr) * lddw + j] = ((word >> li) & 1u) ? acc[0][b][v] : 0.f; // pruned: exactly zero
        }
    }
}

// Two 32-column batch blocks per workgroup halve the reads of W and the mask decodes; one keeps twice the workgroups
// busy.  The line is where two per workgroup still give every compute unit one.
static int batch_blocks(int64_t others, int64_t N) { return (N > 32 && others * ((N + 63) / 64) >= 256) ? 2 : 1; }

template <typename T>
static int launch_t(const Geom &g, const void *dW, int64_t ldw, const uint32_t *dIp, const uint32_t *dIz, const void *dDY,
                    int64_t lddy, int64_t N, void *dDX, int64_t lddx, hipStream_t stream)
{
    const int64_t jblocks = (g.n + 31) / 32;
    const int nq = batch_blocks(jblocks, N);
    const int64_t blocks = jblocks * ((N + 32 * nq - 1) / (32 * nq));
    if (blocks > 0x7FFFFFFF || N > kMaxColumnsT) return LRBI_ERR_SHAPE;
#define LRBI_LAUNCH_F32(NQ, WAVES)                                                                                       \
    LRBI_LAUNCH((f32_gemm_t_kernel<T, NQ, WAVES>), wide_grid(blocks, 64 * WAVES), dim3(64 * WAVES), 0, stream, g, (const T *)dW, \
                ldw, dIp, dIz, (const T *)dDY, lddy, N, (T *)dDX, lddx, (int)jblocks)
    // one chunk of rows: the other wavefronts would only have their zeros added (16 x 65536, N = 1: 24.6 us against 10.0)
    if (g.m <= kF32Chunk) {
        if (nq == 2) LRBI_LAUNCH_F32(2, 1);
        else LRBI_LAUNCH_F32(1, 1);
    } else {
        if (nq == 2) LRBI_LAUNCH_F32(2, kF32Waves);
        else LRBI_LAUNCH_F32(1, kF32Waves);
    }
#undef LRBI_LAUNCH_F32
    return LRBI_OK;
}

int launch_f32_gemm_t(const Geom &g, lrbi_dtype dt, const void *dW, int64_t ldw, const uint32_t *dIp, const uint32_t *dIz,
                      const void *dDY, int64_t lddy, int64_t N, void *dDX, int64_t lddx, hipStream_t stream)
{
    switch (dt) {
    case LRBI_F32: return launch_t<float>(g, dW, ldw, dIp, dIz, dDY, lddy, N, dDX, lddx, stream);
    case LRBI_F16: return launch_t<__half>(g, dW, ldw, dIp, dIz, dDY, lddy, N, dDX, lddx, stream);
    case LRBI_BF16: return launch_t<__hip_bfloat16>(g, dW, ldw, dIp, dIz, dDY, lddy, N, dDX, lddx, stream);
    default: return LRBI_ERR_DTYPE;
    }
}

int launch_f32_gemm(const Geom &g, const float *dW, int64_t ldw, const uint32_t *dIp, const uint32_t *dIz, const float *dX,
                    int64_t ldx, int64_t N, float *dY, int64_t ldy, hipStream_t stream)
{
    const int64_t iblocks = (g.m + 31) / 32;
    const int nq = batch_blocks(iblocks, N);
    const int64_t blocks = iblocks * ((N + 32 * nq - 1) / (32 * nq));
    if (blocks > 0x7FFFFFFF) return LRBI_ERR_SHAPE;
    const bool vec = ((uintptr_t)dW & 15) == 0 && ldw % 4 == 0 && g.n % 4 == 0;
#define LRBI_LAUNCH_F32(NQ, V, WAVES)                                                                                       \
    LRBI_LAUNCH((f32_gemm_kernel<NQ, V, WAVES>), wide_grid(blocks, 64 * (WAVES)), dim3(64 * (WAVES)), 0, stream, g, dW, ldw, dIp, \
                dIz, dX, ldx, N, dY, ldy, (int)iblocks)
    if (nq == 2) {
        if (vec) LRBI_LAUNCH_F32(2, true, kF32Waves);
        else LRBI_LAUNCH_F32(2, false, kF32Waves);
    } else if (blocks <= 128 && g.n > kF32Chunk * kF32Waves) {
        // half the chip idle and wavefronts with several chunks each: twice the wavefronts (8 columns, 200 x 50000 570 -> 480 us,
        // 300 x 4000 45.5 -> 40.5, 1000 x 1000 17.5 -> 14.7; with 250 workgroups, 777 x 1333 at 300 columns, 27.3 against 29.9)
        if (vec) LRBI_LAUNCH_F32(1, true, 2 * kF32Waves);
        else LRBI_LAUNCH_F32(1, false, 2 * kF32Waves);
    } else {
        if (vec) LRBI_LAUNCH_F32(1, true, kF32Waves);
        else LRBI_LAUNCH_F32(1, false, kF32Waves);
    }
#undef LRBI_LAUNCH_F32
    return LRBI_OK;
}

int launch_f32_grad(const Geom &g, const float *dDY, int64_t lddy, const float *dX, int64_t ldx, int64_t N,
                    const uint32_t *dIp, const uint32_t *dIz, float *dDW, int64_t lddw, hipStream_t stream)
{
    const int64_t iblocks = (g.m + 31) / 32;
    // two column blocks per wavefront share its reads of dY; one, while that leaves fewer than two wavefronts per SIMD
    const int nj = iblocks * ((g.n + 63) / 64) >= 2048 ? 2 : 1;
    const int64_t jblocks = (g.n + 32 * nj - 1) / (32 * nj), blocks = iblocks * jblocks;
    if ((blocks + 3) / 4 > 0x7FFFFFFF) return LRBI_ERR_SHAPE;
    const dim3 grid((unsigned)((blocks + 3) / 4));
    const bool vec = (((uintptr_t)dDY | (uintptr_t)dX) & 15) == 0 && lddy % 4 == 0 && ldx % 4 == 0 && N % 4 == 0;
    // I_z rows ahead unless a word has several tiles, with few rows set in each (us, without and with: 2000 x 2000 in 5 x 5 tiles, rank
    // 2, 8 columns 13.0 / 16.5, 1000 x 4000 in 100 x 31, rank 40 11.4 / 12.5; a kernel of its own: a test in it took 5 % of the other shapes)
    const bool ahead = g.c >= 32;
#define LRBI_LAUNCH_F32(NJ, V)                                                                                     \
    do {                                                                                                           \
        auto kern = ahead ? f32_grad_kernel<NJ, V, true> : f32_grad_kernel<NJ, V, false>;                          \
        LRBI_LAUNCH(kern, grid, dim3(256), 0, stream, g, dDY, lddy, dX, ldx, N, dIp, dIz, dDW, lddw, jblocks, blocks); \
    } while (0)
    if (nj == 2) {
        if (vec) LRBI_LAUNCH_F32(2, true);
        else LRBI_LAUNCH_F32(2, false);
    } else {
        if (vec) LRBI_LAUNCH_F32(1, true);
        else LRBI_LAUNCH_F32(1, false);
    }
#undef LRBI_LAUNCH_F32
    return LRBI_OK;
}

} // namespace lrbi
