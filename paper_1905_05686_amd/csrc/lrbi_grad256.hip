// Weight gradient dW = (dY X^T) o I_a on the matrix cores in 256 x 256 output tiles (f16 / bf16, fp32 accumulate): the form
// for batches long enough that the products, not the output, take the time.
//
// The 128 x 128 kernel stages its operands through registers and reads 16 bytes of LDS per lane for every two matrix
// instructions; four workgroups share a compute unit, which is what a short batch wants (the output is most of its work).
// On a long one it is bound by the operand bytes per flop (4096 x 4096 bf16, batch 1024: 52 us, 0.66 PFLOP/s).  Here a
// workgroup of eight wavefronts owns 256 x 256 of dW, wavefront (wm, wn) 64 rows x 128 columns; dY rows and X rows both lie
// along the batch, so both operands are the same image: slabs of 32 batch columns, 16 KB each, from global memory straight
// into a ring of four LDS stages, read with plain 16-byte LDS reads.  One barrier per slab, counted waits.
// The mask touches only the output: its bits under the tile are formed once (Eq. 3), in the first iteration, from factor
// slices in LDS (tiles line up with 64 columns and 128 rows), and select on the way out.
// 4096 x 4096 bf16, 512 x 512 tiles: batch 1024 51 -> 39 us, 512 33 -> 27, 256 24 -> 21.
#include "lrbi_internal.hpp"
#include "lrbi_lds_dma.hpp"
#include "lrbi_mfma_common.hpp"

namespace lrbi {

static constexpr int G256_THREADS = 512;
static constexpr int G256_B = 256;           // rows and columns of the output tile
static constexpr int G256_BK = 32;           // batch columns per slab
static constexpr int G256_NS = 4;            // stages
static constexpr int G256_STAGE = 32768;     // dY: 256 rows x 64 bytes, then X: 256 rows x 64 bytes
static constexpr int G256_STAGE_X = 16384;
static constexpr int G256_MT_ROW = 36;       // bytes of mask per row: 32 + 4
static constexpr int G256_HU = G256_B / 64;
static constexpr int G256_FZ_ROW = G256_HU * 8;
static constexpr int G256_FZ_SET = FAST_MAX_K * G256_FZ_ROW;

struct SmemG256 {
    static constexpr size_t mt_off = (size_t)G256_NS * G256_STAGE;
    static constexpr size_t fz_off = mt_off + G256_B * G256_MT_ROW;
    static constexpr size_t fip_off = fz_off + 2 * G256_FZ_SET;
    static constexpr size_t bytes = fip_off + G256_B * G256_HU * 2 * 4;
};
static_assert(SmemG256::bytes <= 160 * 1024, "LDS of a compute unit");

template <typename Tag>
__global__ __launch_bounds__(G256_THREADS) LRBI_WAVES_PER_SIMD(2) void mfma_grad256_kernel(
    Geom g, const uint16_t *__restrict__ DY, int64_t lddy, const uint16_t *__restrict__ X, int64_t ldx, int N,
    const uint32_t *__restrict__ Ip, const uint32_t *__restrict__ Iz, uint16_t *__restrict__ DW, int64_t lddw, int iblocks,
    int jblocks, int xcd_remap, int w_vec_ok)
{
    constexpr int NS = G256_NS;
    using S = SmemG256;
    extern __shared__ uint4 lrbi_dyn_smem[];
    unsigned char *smem = (unsigned char *)lrbi_dyn_smem;
    unsigned char *Mt = smem + S::mt_off;            // [256][MT_ROW]     mask bytes of the tile
    unsigned char *Fz = smem + S::fz_off;            // [2][64][8 words]  I_z rows under the tile, per 128-row half
    uint32_t *Fip = (uint32_t *)(smem + S::fip_off); // [256][4][2]       I_p words per row and 64-column half unit

    int64_t bid = blockIdx.x;
    if (xcd_remap) {
        const int64_t per = gridDim.x / 8;
        bid = (bid % 8) * per + bid / 8;
    }
    int ii, ji;
    grouped_tile<4>(bid, iblocks, jblocks, &ii, &ji);
    const int64_t i0 = (int64_t)ii * G256_B;
    const int j0 = ji * G256_B;
    const int n = (int)g.n;
    const int nslabs = N / G256_BK;
    const int last = nslabs - 1;
    const int a_last = (int)((g.m - 1 - i0 < G256_B - 1) ? g.m - 1 - i0 : G256_B - 1); // last row of the tile inside the matrix
    const int b_last = (n - 1 - j0 < G256_B - 1) ? n - 1 - j0 : G256_B - 1;             // last column

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lg = lane >> 5;

    // ---- global -> LDS: both images have 64-byte rows, piece p of row q at slot p ^ ((q >> 2) & 3); a load instruction fills
    // 16 rows; wavefront w issues the chunks w and w + 8 of each.  Rows past the matrix repeat the last one and are not stored.
    uint32_t avo[2], bvo[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave + 8 * i) * 16 + (lane >> 2);
        const int p = (lane & 3) ^ ((row >> 2) & 3);
        avo[i] = (uint32_t)(((row < a_last ? row : a_last) * lddy + p * 8) * 2);
        bvo[i] = (uint32_t)(((row < b_last ? row : b_last) * ldx + p * 8) * 2);
    }
    const uint16_t *aptr = DY + i0 * lddy, *bptr = X + (int64_t)j0 * ldx;
    int asl = 0, bsl = 0; // the slabs that are asked for next; past the last one it is fetched again
    const uint32_t lds0 = lds_address(smem);
    const uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    auto issue_piece = [&](int stage, auto i_c) { // 0, 1: chunks of dY, 2, 3: of X; the second one moves on
        constexpr int i = decltype(i_c)::value;
        const uint32_t sb = lds_w + (uint32_t)stage * G256_STAGE;
        if constexpr (i < 2) load_to_lds16(sb + i * 8192u, aptr, avo[i]);
        else load_to_lds16(sb + G256_STAGE_X + (i - 2) * 8192u, bptr, bvo[i - 2]);
        if constexpr (i == 1) {
            if (asl < last) aptr += G256_BK;
            ++asl;
        }
        if constexpr (i == 3) {
            if (bsl < last) bptr += G256_BK;
            ++bsl;
        }
    };

    // ---- operand reads: row 32 (block) + lane % 32, piece 2 j + lane / 32 of step j; addresses of stage 0 and of stage 2
    uint32_t afa[2][2], bfa[2][2];
    {
        const int c3 = (l32 >> 2) & 3;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t p = (uint32_t)(((2 * j + lg) ^ c3) * 16);
            afa[0][j] = (uint32_t)((wm * 64 + l32) * 64) + p;
            bfa[0][j] = (uint32_t)(G256_STAGE_X + (wn * 128 + l32) * 64) + p;
            afa[1][j] = afa[0][j] + 2 * G256_STAGE;
            bfa[1][j] = bfa[0][j] + 2 * G256_STAGE;
        }
    }
    u32x4 af[2][2], bf[2][4]; // [step][block]
    auto read_a = [&](auto st_c, auto j_c, auto b_c) {
        constexpr int st = decltype(st_c)::value, j = decltype(j_c)::value, b = decltype(b_c)::value;
        af[j][b] = *reinterpret_cast<const u32x4 *>(smem + afa[st >> 1][j] + (st & 1) * G256_STAGE + b * 2048);
    };
    auto read_b = [&](auto st_c, auto j_c, auto a_c) {
        constexpr int st = decltype(st_c)::value, j = decltype(j_c)::value, a = decltype(a_c)::value;
        bf[j][a] = *reinterpret_cast<const u32x4 *>(smem + bfa[st >> 1][j] + (st & 1) * G256_STAGE + a * 2048);
    };
    f32x16 acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    auto mma = [&](auto j_c, auto a_c, auto b_c) {
        constexpr int j = decltype(j_c)::value, a = decltype(a_c)::value, b = decltype(b_c)::value;
        acc[a][b] = mfma_32x32x16(Tag{}, bf[j][a], af[j][b], acc[a][b]);
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
#define LRBI_SB() __builtin_amdgcn_sched_barrier(0)
// workgroup barrier that drains nothing: what it hands over is the stage of slab s - 1, whose operands have been multiplied
#define LRBI_BARRIER()                                             \
    do {                                                           \
        LRBI_SB();                                                 \
        asm volatile("" ::: "memory");                             \
        __builtin_amdgcn_s_barrier();                              \
        asm volatile("" ::: "memory");                             \
        LRBI_SB();                                                 \
    } while (0)

    // ---- prologue: factor slices, slabs 0 .. NS - 2 (the last one's X half follows in the first iteration), the mask
    {
        const int64_t ih = (i0 + 128 < g.m) ? i0 + 128 : i0; // (a half past the matrix: stand-ins)
        const int hu = (lane >> 1) & 3;
        const int col = j0 + 64 * hu < n ? j0 + 64 * hu : j0;
        const int tj = col / g.c, zw = (col - tj * g.c) >> 5;
#pragma unroll
        for (int i = 0; i < 2; ++i) { // I_z: ranks 8 qq .. + 7 of a half, lane = (rank, half unit, word)
            const int q = wave * 2 + i, half = q >> 3, qq = q & 7;
            const int rank = qq * 8 + (lane >> 3);
            const int64_t t = ((half ? ih : i0) / g.r) * g.tile_cols + tj;
            load_to_lds4(lds0 + (uint32_t)(S::fz_off + half * G256_FZ_SET + qq * 256), Iz,
                         (uint32_t)(((t * g.k + (rank < g.k ? rank : 0)) * g.izw + zw + (lane & 1)) * 4));
        }
        const int iw = (lane & 1) < g.ipw ? (lane & 1) : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) { // I_p: rows 8 q .. + 7, lane = (row, half unit, word)
            const int q = wave * 4 + i, half = q >> 4;
            const int64_t ib = half ? ih : i0;
            const int64_t t = (ib / g.r) * g.tile_cols + tj;
            const int il = (int)(ib % g.r) + (q & 15) * 8 + (lane >> 3);
            load_to_lds4(lds0 + (uint32_t)(S::fip_off + q * 256), Ip, (uint32_t)(((t * g.r + il) * g.ipw + iw) * 4));
        }
    }
    constexpr int kProloguePieces = (NS - 2) * 4 + 2;
    static_for<NS - 1>([&](auto sc) {
        constexpr int st = decltype(sc)::value;
        issue_piece(st, I0{});
        issue_piece(st, I1{});
        if constexpr (st != NS - 2) {
            issue_piece(st, I2{});
            issue_piece(st, I3{});
        }
    });
    wait_loads<kProloguePieces - 4>(); // slab 0
    __syncthreads();
    static_for<2>([&](auto b) { read_a(I0{}, I0{}, b); });
    static_for<4>([&](auto a) { read_b(I0{}, I0{}, a); });

    // Eq. 3: a lane forms the four mask words of one row under 128 columns
    auto form_mask = [&]() {
        const int row = tid >> 1, u = tid & 1;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        const uint32_t *fp = Fip + (row * G256_HU + 2 * u) * 2;
        const unsigned char *fz = Fz + (row >> 7) * G256_FZ_SET + u * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            for (int iw = 0; iw < g.ipw; ++iw) {
                uint32_t sel = fp[2 * h + iw];
                while (sel) {
                    const int l = __builtin_ctz(sel) + 32 * iw;
                    sel &= sel - 1u;
                    const u32x2 z = *reinterpret_cast<const u32x2 *>(fz + l * G256_FZ_ROW + h * 8);
                    w[2 * h] |= z.x;
                    w[2 * h + 1] |= z.y;
                }
            }
        uint32_t *out = reinterpret_cast<uint32_t *>(Mt + row * G256_MT_ROW + u * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = w[e];
    };

    // ---- main loop, unrolled by NS.  Iteration s multiplies slab s out of stage s % NS in two steps; between them every
    // wavefront waits until its own pieces of slab s + 1 have landed, the barrier makes the slab visible and frees the stage
    // of slab s - 1.  Each step reads the next one's operands; LRBI_SB() keeps the other instructions between the matrix ones.
    for (int s0 = 0; s0 < nslabs; s0 += NS) {
        static_for<NS>([&](auto sc) {
            constexpr int st = decltype(sc)::value;
            using St = std::integral_constant<int, st>;
            using St1 = std::integral_constant<int, (st + 1) % NS>;
            constexpr int stn = (st + NS - 1) % NS; // stage of slab s + NS - 1
            constexpr int stp = (st + NS - 2) % NS; // stage of slab s + NS - 2
            if (s0 + st < nslabs) {
                read_a(St{}, I1{}, I0{}); read_a(St{}, I1{}, I1{});
                LRBI_SB();
                mma(I0{}, I0{}, I0{}); read_b(St{}, I1{}, I0{});
                LRBI_SB();
                mma(I0{}, I0{}, I1{}); read_b(St{}, I1{}, I1{}); issue_piece(stp, I2{});
                LRBI_SB();
                mma(I0{}, I1{}, I0{}); read_b(St{}, I1{}, I2{}); issue_piece(stp, I3{});
                LRBI_SB();
                mma(I0{}, I1{}, I1{}); read_b(St{}, I1{}, I3{});
                LRBI_SB();
                mma(I0{}, I2{}, I0{}); mma(I0{}, I2{}, I1{}); mma(I0{}, I3{}, I0{}); mma(I0{}, I3{}, I1{});
                wait_loads<(NS - 3) * 4>();
                LRBI_BARRIER();
                read_a(St1{}, I0{}, I0{}); read_a(St1{}, I0{}, I1{});
                LRBI_SB();
                mma(I1{}, I0{}, I0{}); read_b(St1{}, I0{}, I0{});
                LRBI_SB();
                mma(I1{}, I0{}, I1{}); read_b(St1{}, I0{}, I1{}); issue_piece(stn, I0{});
                LRBI_SB();
                mma(I1{}, I1{}, I0{}); read_b(St1{}, I0{}, I2{}); issue_piece(stn, I1{});
                LRBI_SB();
                mma(I1{}, I1{}, I1{}); read_b(St1{}, I0{}, I3{});
                LRBI_SB();
                mma(I1{}, I2{}, I0{}); mma(I1{}, I2{}, I1{}); mma(I1{}, I3{}, I0{}); mma(I1{}, I3{}, I1{});
                // the factor slices are older than slab 1, which every wavefront has waited for
                if (st == 0 && s0 == 0) form_mask();
            }
        });
    }
#undef LRBI_SB
#undef LRBI_BARRIER
    wait_loads<0>(); // nothing may still be landing in LDS
    __syncthreads();

    // ---- epilogue: lane holds, per 32-column block a, columns 8 (v / 4) + 4 lg + (v % 4) of row l32 of block b.  Each 32 x 128
    // block goes through the wavefront's own strip of LDS and leaves, masked, as 16-byte pieces of whole rows.
    constexpr int RS = 128 * 2 + 8;
    unsigned char *strip = smem + wave * (32 * RS);
    const int l16 = lane & 15, rq = lane >> 4;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                uint16_t o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = cvt_store(Tag{}, acc[a][b][4 * v4 + e]);
                *reinterpret_cast<uint2 *>(strip + l32 * RS + (a * 32 + 8 * v4 + 4 * lg) * 2) = *reinterpret_cast<uint2 *>(o);
            }
        // (the strip is private to the wavefront: its own LDS operations complete in order)
#pragma unroll
        for (int i = 0; i < 8; ++i) { // 4 rows per instruction: 16 lanes x 16 bytes per row
            const int rr = 4 * i + rq, row = wm * 64 + b * 32 + rr, pc = wn * 16 + l16;
            const uint2 lo = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16);
            const uint2 hi = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16 + 8);
            const uint4 v = apply_mask8(make_uint4(lo.x, lo.y, hi.x, hi.y), (uint32_t)Mt[row * G256_MT_ROW + pc]);
            const int jj = j0 + pc * 8;
            if (row > a_last || jj >= n) continue;
            uint16_t *wp = DW + (i0 + row) * lddw + jj;
            if (w_vec_ok && jj + 8 <= n) {
                *reinterpret_cast<uint4 *>(wp) = v;
            } else {
                const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (jj + e < n) wp[e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

// operands in 16-byte pieces and whole slabs, 32-bit byte offsets, tiles that line up with the factor slices
bool grad256_ok(const Geom &g, const void *dDY, int64_t lddy, const void *dX, int64_t ldx, int64_t N)
{
    if ((g.c % 64) != 0 || (g.r % 128) != 0 || g.k > FAST_MAX_K || g.ragged || N % G256_BK != 0) return false;
    if ((((uintptr_t)dDY | (uintptr_t)dX) & 15) != 0 || lddy % 8 != 0 || ldx % 8 != 0) return false;
    if (lddy >= ((int64_t)1 << 22) || ldx >= ((int64_t)1 << 22)) return false;
    const int64_t tiles = (int64_t)g.tile_rows * g.tile_cols;
    return tiles * g.k * g.izw * 4 < (int64_t)1 << 31 && tiles * g.r * g.ipw * 4 < (int64_t)1 << 31;
}
// One workgroup per compute unit does its round alone, so the rounds have to be nearly full, or a single one on a long
// batch, and longer ones the more of them there are: the 128 x 128 form, four workgroups a unit, runs a tile's output under another
// one's products.  Us, 256 against 128, 256 x 256 tiles of rank 16, f16 and bf16:
//   * One round: 4096 x 4096, 256 tiles: batch 128 17.3 / 18.6, 1024 39 / 49; 2304 x 4096, 144 tiles, batch 1024 27 / 32, 512 18.3 /
//     19.9; but 2048 x 4096, 128 tiles, batch 1024 31.2 / 29.0.
//   * Two: 8192 x 4096, batch 512 50 / 56, 256 37.9 / 37.2, 128 30 / 29; 6912 x 4096, 432 tiles, batch 384 34 / 37.
//   * More: 8192 x 8192, four, batch 512 97 / 103, 256 71 / 65, 128 57 / 50; 9216 x 9216, 1296 tiles in six (84 % of them full), batch
//     512 137 / 128, 768 152 / 168, 256 102 / 81; 4096 x 9216, 576 tiles in three (75 %), batch 512 67 / 60.
//   * Tile widths of 64 (2 j + 1) with more than 32 ranks, whose mask the 128 x 128 form takes longer over: 8192 x 4096 in 128 x 64, rank
//     40, batch 128 31 / 36, 256 38 / 43; 8192 x 8192, rank 64, batch 128 59 / 68, 256 74 / 82; 12288 x 4096, rank 40, batch 384 67 / 76.
bool grad256_wins(const Geom &g, int64_t N)
{
    constexpr int64_t cus = 256;
    const int64_t t256 = ((g.m + 255) / 256) * ((g.n + 255) / 256), rounds = (t256 + cus - 1) / cus;
    const bool full = rounds * cus * 5 <= t256 * 6;
    if (rounds == 1) return (N >= 128 && full) || (N >= 512 && t256 >= 144);
    if (rounds <= 4 && g.c % 128 != 0 && g.k > 32) return full && N >= 128;
    if (rounds == 2) return full && N > 256;
    return full && (N >= 768 || (N >= 512 && rounds * cus * 9 <= t256 * 10));
}

int launch_grad256(const Geom &g, lrbi_dtype dt, const void *dDY, int64_t lddy, const void *dX, int64_t ldx, int64_t N,
                   const uint32_t *dIp, const uint32_t *dIz, void *dDW, int64_t lddw, hipStream_t stream)
{
    const int64_t iblocks = (g.m + G256_B - 1) / G256_B, jblocks = (g.n + G256_B - 1) / G256_B;
    const int64_t blocks = iblocks * jblocks;
    if (blocks > 0x7FFFFFFF / G256_THREADS) return LRBI_ERR_SHAPE;
    const int w_vec_ok = (((uintptr_t)dDW & 15) == 0) && (lddw % 8 == 0);
    auto kern = dt == LRBI_F16 ? mfma_grad256_kernel<F16Tag> : mfma_grad256_kernel<BF16Tag>;
    LRBI_SET_MAX_LDS(kern, SmemG256::bytes);
    LRBI_LAUNCH(kern, dim3((unsigned)blocks), dim3(G256_THREADS), SmemG256::bytes, stream, g, (const uint16_t *)dDY, lddy,
                (const uint16_t *)dX, ldx, (int)N, dIp, dIz, (uint16_t *)dDW, lddw, (int)iblocks, (int)jblocks,
                (blocks % 8 == 0) ? 1 : 0, w_vec_ok);
    return LRBI_OK;
}

} // namespace lrbi
