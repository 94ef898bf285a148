// Fused masked product on the matrix cores in 256 x 256 output tiles (f16 / bf16, fp32 accumulate): the pipelined tile
// kernel for products whose result alone fills the chip with such tiles.
//
// What bounds the 128 x 128 form on large products is not the matrix pipe but the operand bytes that come through the
// compute unit's load path and the mask work, both per flop: 32 KB and two masked operand pieces for 512 clocks of matrix
// work a SIMD (16384 x 16384 bf16, N = 4096: 2454 us; without the loads 1930, without loads, mask and factor work 1443,
// matrix instructions alone 1178).  A 256 x 256 tile halves both: 1644 us there, at 1304 clocks a slab (1024 of them matrix
// work, 75 the panels) and 1.7 GHz, where matrix instructions alone run at 2.3.
//
// One workgroup of eight wavefronts (two per SIMD); wavefront (wm, wn) owns 64 rows x 128 columns of the tile: 128
// accumulator registers, and per 16-column step two W operands and four X operands for eight matrix instructions.
//   * Slabs of 32 columns of W: 16 KB of W and 16 KB of X, from global memory straight into a ring of four LDS stages
//     (128 KB), three slabs ahead, counted waits, one barrier per slab, as in the 128 x 128 kernel.
//   * Mask panels of 256 columns (eight slabs), rebuilt one panel ahead from factor slices gathered per 64-column half
//     unit, so any tile width that is a multiple of 64 fits; the two 128-row halves of the tile may lie in different tile
//     rows (r % 128 == 0) and have I_z slices of their own.
//   * A step's operands are read while the step before it is multiplied; the W operands are masked there as well (select
//     on the bit pattern).
#include "lrbi_internal.hpp"
#include "lrbi_lds_dma.hpp"
#include "lrbi_mfma_common.hpp"

namespace lrbi {

static constexpr int P256_THREADS = 512;
static constexpr int P256_B = 256;             // rows and columns of the output tile
static constexpr int P256_BK = 32;             // columns of W per slab
static constexpr int P256_NS = 4;              // stages
static constexpr int P256_STAGE = 32768;       // W: 256 rows x 64 bytes, then X: 32 rows x 512 bytes
static constexpr int P256_STAGE_X = 16384;
static constexpr int P256_PW = 256;            // panel width
static constexpr int P256_PSLABS = P256_PW / P256_BK;
static constexpr int P256_HU = P256_PW / 64;   // half units of a panel
static constexpr int P256_MT_ROW = 36;         // bytes per row of a mask panel: 32 + 4 (rows of a read on distinct banks)
static constexpr int P256_MT = P256_B * P256_MT_ROW;
static constexpr int P256_FZ_ROW = P256_HU * 8; // bytes of a rank's I_z words under a panel
static constexpr int P256_FZ_SET = (FAST_MAX_K + 1) * P256_FZ_ROW; // (row 32 stays zero)
static constexpr int P256_FACTOR_LOADS = 6;    // load instructions of a wavefront per panel

struct SmemP256 {
    static constexpr size_t mt_off = (size_t)P256_NS * P256_STAGE;
    static constexpr size_t fz_off = mt_off + 2 * P256_MT;
    static constexpr size_t fip_off = fz_off + 2 * P256_FZ_SET;
    static constexpr size_t bytes = fip_off + P256_B * P256_HU * 2 * 4;
};
static_assert(SmemP256::bytes <= 160 * 1024, "LDS of a compute unit");
static_assert(SmemP256::fz_off % 16 == 0 && SmemP256::fip_off % 16 == 0, "16-byte pieces");

// KW: I_p words per row (ranks up to 32, up to 64).  HALF: tile widths that are an odd multiple of 64.
template <typename Tag, int KW, bool HALF>
__global__ __launch_bounds__(P256_THREADS) LRBI_WAVES_PER_SIMD(2) void mfma_gemm_pipe256_kernel(
    Geom g, const uint16_t *__restrict__ W, int64_t ldw, const uint32_t *__restrict__ Ip,
    const uint32_t *__restrict__ Iz, const uint16_t *__restrict__ X, int64_t ldx, int N, uint16_t *__restrict__ Y,
    int64_t ldy, int mblocks, int nblocks, int xcd_remap, int y_vec_ok)
{
    constexpr int NS = P256_NS;
    using S = SmemP256;
    extern __shared__ uint4 lrbi_dyn_smem[];
    unsigned char *smem = (unsigned char *)lrbi_dyn_smem;
    unsigned char *Mt = smem + S::mt_off;          // [2][256][MT_ROW]     mask bytes of two panels
    unsigned char *Fz = smem + S::fz_off;          // [2][65][8 words]     I_z rows under the panel, per 128-row half
    uint32_t *Fip = (uint32_t *)(smem + S::fip_off); // [256][4][2]        I_p words per row and half unit

    int64_t bid = blockIdx.x;
    if (xcd_remap) {
        const int64_t per = gridDim.x / 8;
        bid = (bid % 8) * per + bid / 8;
    }
    int mi, ni;
    grouped_tile<4>(bid, mblocks, nblocks, &mi, &ni);
    const int64_t m0 = (int64_t)mi * P256_B;
    const int n0 = ni * P256_B;
    const int nslabs = (int)(g.n / P256_BK);
    const int last = nslabs - 1;
    // the upper 128 rows of the last tile row of an odd number of 128-row blocks repeat the lower ones and are not stored
    const int64_t mh = (m0 + 128 < g.m) ? m0 + 128 : m0;
    const int ti0 = (int)(m0 / g.r), ti1 = (int)(mh / g.r);
    const int il0 = (int)(m0 - (int64_t)ti0 * g.r), il1 = (int)(mh - (int64_t)ti1 * g.r);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lg = lane >> 5;

    // ---- global -> LDS: a load instruction fills 1 KiB; wavefront w issues the chunks w and w + 8 of both images.
    // W image: 64-byte rows, piece p of row q at slot p ^ ((q >> 2) & 3); X image: 512-byte rows, piece p of row q at slot
    // p ^ (4 (q & 3)) (the operand reads below then meet every LDS bank once).
    uint32_t wvo[2], xvo[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int chunk = wave + 8 * i;
        const int wr = chunk * 16 + (lane >> 2);
        const int wp = (lane & 3) ^ ((wr >> 2) & 3);
        const int64_t row = (wr < 128) ? wr : (mh - m0) + wr - 128;
        wvo[i] = (uint32_t)((row * ldw + wp * 8) * 2);
        const int xr = chunk * 2 + (lane >> 5);
        int nn = ((lane & 31) ^ (4 * (xr & 3))) * 8;
        if (n0 + nn + 8 > N) nn = N - 8 - n0; // piece beyond N: a valid piece instead, its columns are dropped
        xvo[i] = (uint32_t)((xr * ldx + nn) * 2);
    }
    const uint16_t *wptr = W + m0 * ldw, *xptr = X + n0;
    const int64_t xstep = (int64_t)P256_BK * ldx;
    int wsl = 0, xsl = 0; // the slabs that are asked for next; past the last one it is fetched again
    const uint32_t lds0 = lds_address(smem);
    const uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    // piece i (0, 1: W chunks, 2, 3: X chunks) of the next slab into a stage; the second piece moves on
    auto issue_piece = [&](int stage, auto i_c) {
        constexpr int i = decltype(i_c)::value;
        const uint32_t sb = lds_w + (uint32_t)stage * P256_STAGE;
        if constexpr (i < 2) load_to_lds16(sb + i * 8192u, wptr, wvo[i]);
        else load_to_lds16(sb + P256_STAGE_X + (i - 2) * 8192u, xptr, xvo[i - 2]);
        if constexpr (i == 1) {
            if (wsl < last) wptr += P256_BK;
            ++wsl;
        }
        if constexpr (i == 3) {
            if (xsl < last) xptr += xstep;
            ++xsl;
        }
    };

    // ---- operand reads: addresses of stage 0 and of stage 2 (a read instruction's offset spans two stages)
    // W operand of step j, block b: row 64 wm + 32 b + lane % 32, piece 2 j + lane / 32
    uint32_t wfa[2][2], xfa[2][4];
    {
        const int q = wm * 64 + l32;
        const int c3 = (q >> 2) & 3; // the same for both blocks
#pragma unroll
        for (int j = 0; j < 2; ++j) wfa[0][j] = (uint32_t)(q * 64 + (((2 * j + lg) ^ c3) * 16));
    }
    // X operand (transposing read): 16-lane group G = lane / 16 serves columns 16 (G % 2) .. + 15 of a 32-column block and
    // k group G / 2; lane d of the group addresses row d / 4, columns 4 (d % 4); block a sits at 64 (a ^ (row & 3))
    {
        const int d16 = lane & 15, G16 = lane >> 4;
        const int q = 8 * (G16 >> 1) + (d16 >> 2); // row inside the step (+ 4 for the upper half)
        const uint32_t base = (uint32_t)(P256_STAGE_X + q * 512 + wn * 256 + (2 * (G16 & 1) + ((d16 & 3) >> 1)) * 16 + 8 * (d16 & 1));
#pragma unroll
        for (int a = 0; a < 4; ++a) xfa[0][a] = base + 64u * (uint32_t)(a ^ (q & 3));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) wfa[1][j] = wfa[0][j] + 2 * P256_STAGE;
#pragma unroll
    for (int a = 0; a < 4; ++a) xfa[1][a] = xfa[0][a] + 2 * P256_STAGE;
    // mask bytes: four per row and slab, of which step j uses byte 2 j + lane / 32
    const uint32_t mta = (uint32_t)((wm * 64 + l32) * P256_MT_ROW);

    u32x4 wf[2][2], xf[2][4]; // [step][block]
    auto read_w = [&](auto st_c, auto j_c, auto b_c) {
        constexpr int st = decltype(st_c)::value, j = decltype(j_c)::value, b = decltype(b_c)::value;
        wf[j][b] = *reinterpret_cast<const u32x4 *>(smem + wfa[st >> 1][j] + (st & 1) * P256_STAGE + b * 2048);
    };
    auto read_x = [&](auto st_c, auto j_c, auto a_c) {
        constexpr int st = decltype(st_c)::value, j = decltype(j_c)::value, a = decltype(a_c)::value;
        const unsigned char *p = smem + xfa[st >> 1][a] + (st & 1) * P256_STAGE + j * 8192;
        const u32x2 lo = lds_read_tr16_v((const uint16_t *)p);
        const u32x2 hi = lds_read_tr16_v((const uint16_t *)(p + 2048));
        xf[j][a] = u32x4{lo.x, lo.y, hi.x, hi.y};
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
        acc[a][b] = mfma_32x32x16(Tag{}, xf[j][a], wf[j][b], acc[a][b]);
    };
    // mask of a W operand in two halves (between two matrix instructions each); m: the row's mask word, shifted by 8 (lane / 32)
    auto mask_lo = [&](auto j_c, auto b_c, uint32_t m) -> uint32_t {
        constexpr int j = decltype(j_c)::value, b = decltype(b_c)::value;
        const uint32_t y = ((m >> (16 * j)) & 0xFFu) * 0x8001u;
        wf[j][b].x = select2(wf[j][b].x, y & 0x00010001u);
        wf[j][b].y = select2(wf[j][b].y, (y >> 2) & 0x00010001u);
        return y;
    };
    auto mask_hi = [&](auto j_c, auto b_c, uint32_t y) {
        constexpr int j = decltype(j_c)::value, b = decltype(b_c)::value;
        wf[j][b].z = select2(wf[j][b].z, (y >> 4) & 0x00010001u);
        wf[j][b].w = select2(wf[j][b].w, (y >> 6) & 0x00010001u);
    };
    // mask word of this lane's row of block b under slab `ps` of the panel whose bytes start at `panel`
    auto fetch_mask = [&](uint32_t panel, int ps, int b) -> uint32_t {
        return *reinterpret_cast<const uint32_t *>(Mt + panel + mta + ps * 4 + b * (32 * P256_MT_ROW));
    };

    // ---- factor slices of one panel: global -> LDS, word by word, per 64-column half unit (two words of an I_z row).
    // A lane fetches for one of the panel's half units; (ftj, foff, fcol): that half unit's tile column, offset in it and
    // first column, carried from panel to panel.  Ranks at or beyond k fetch rank 0 (no I_p bit selects them); half units
    // past the last column fetch the tile row's first tile (their mask bytes are never read).
    const uint32_t izs = (uint32_t)(g.k * g.izw * 4), ips = (uint32_t)(g.r * g.ipw * 4); // bytes of a tile's factors
    const uint32_t z0 = (uint32_t)ti0 * (uint32_t)g.tile_cols * izs, z1 = (uint32_t)ti1 * (uint32_t)g.tile_cols * izs;
    const uint32_t p0 = (uint32_t)ti0 * (uint32_t)g.tile_cols * ips + (uint32_t)(il0 * g.ipw * 4);
    const uint32_t p1 = (uint32_t)ti1 * (uint32_t)g.tile_cols * ips + (uint32_t)(il1 * g.ipw * 4);
    int fcol = 64 * ((lane >> 1) & 3);
    int ftj = fcol / g.c, foff = fcol - ftj * g.c;
    const int n_cols = (int)g.n;
    auto load_factors = [&]() {
        const bool ok = fcol < n_cols;
        const uint32_t zsel = ok ? (uint32_t)ftj * izs + (uint32_t)(foff >> 5) * 4u : 0u;
        const uint32_t psel = ok ? (uint32_t)ftj * ips : 0u;
        fcol += P256_PW;
        foff += P256_PW;
        while (foff >= g.c) {
            foff -= g.c;
            ++ftj;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = wave * 2 + i, half = q >> 3, qq = q & 7; // ranks 8 qq .. + 7, lane = (rank, half unit, word)
            const int rank = qq * 8 + (lane >> 3);
            load_to_lds4(lds0 + (uint32_t)(S::fz_off + half * P256_FZ_SET + qq * 256 + (qq >= 4 ? P256_FZ_ROW : 0)), Iz,
                         (half ? z1 : z0) + zsel + (uint32_t)((((rank < g.k) ? rank : 0) * g.izw + (lane & 1)) * 4));
        }
        const int iw = (lane & 1) < g.ipw ? (lane & 1) : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = wave * 4 + i, half = q >> 4; // rows 8 q .. + 7, lane = (row, half unit, word)
            const int row = (q & 15) * 8 + (lane >> 3);
            load_to_lds4(lds0 + (uint32_t)(S::fip_off + q * 256), Ip, (half ? p1 : p0) + psel + (uint32_t)((row * g.ipw + iw) * 4));
        }
    };
    // Eq. 3 for the panel: a lane forms the four mask words of one row under one 128-column unit (HALF: under its two half
    // units, each from the factors of its own tile).  The set ranks are taken two at a time, over three slabs of the loop, so
    // that the reads have come back when they are added; rows with more ranks than that (few: the factors are sparse) loop
    // over the rest.  Ranks are found per 32-bit word of I_p; a word without one left reads the zero row, 32 (which is what
    // counting its trailing zeros gives), rank l >= 32 sits in row l + 1.
    constexpr int NH = HALF ? 2 : 1, PER = KW == 1 ? 2 : 1;
    using zvec = std::conditional_t<HALF, u32x2, u32x4>;
    const int drow = tid >> 1, du = tid & 1;
    const unsigned char *dfz = Fz + (drow >> 7) * P256_FZ_SET + du * 16;
    uint32_t sel[NH][KW];
    zvec dz[NH][KW * PER], dh[NH];
    auto decode_words = [&]() {
        const uint32_t *fp = Fip + (drow * P256_HU + 2 * du) * 2;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int w = 0; w < KW; ++w) sel[h][w] = fp[2 * h + w];
            dh[h] = zvec(0u);
        }
    };
    auto decode_ask = [&]() {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int w = 0; w < KW; ++w)
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const uint32_t v = sel[h][w];
                    const uint32_t l = v ? (uint32_t)__builtin_ctz(v) : 32u;
                    sel[h][w] = v & (v - 1u);
                    // (the second word's ranks are 33 rows on; its zero row is the first word's)
                    const uint32_t row = w == 0 ? l : (v ? l + 33u : 32u);
                    dz[h][w * PER + e] = *reinterpret_cast<const zvec *>(dfz + row * P256_FZ_ROW + h * 8);
                }
    };
    auto decode_add = [&]() {
#pragma unroll
        for (int h = 0; h < NH; ++h) dh[h] |= dz[h][0] | dz[h][1];
    };
    auto decode_store = [&](uint32_t panel) {
        auto left = [&]() {
            uint32_t any = 0u;
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int w = 0; w < KW; ++w) any |= sel[h][w];
            return any;
        };
        while (left()) {
            decode_ask();
            decode_add();
        }
        uint32_t *out = reinterpret_cast<uint32_t *>(Mt + panel + drow * P256_MT_ROW + du * 16);
        if constexpr (HALF) {
            out[0] = dh[0].x;
            out[1] = dh[0].y;
            out[2] = dh[1].x;
            out[3] = dh[1].y;
        } else {
            out[0] = dh[0].x;
            out[1] = dh[0].y;
            out[2] = dh[0].z;
            out[3] = dh[0].w;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // landed before the next barrier
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
#define LRBI_SB() __builtin_amdgcn_sched_barrier(0)
// workgroup barrier that drains nothing: operand reads of slab s may be under way across it, what is handed over is the
// stage of slab s - 1, whose operands have all been multiplied
#define LRBI_BARRIER()                                             \
    do {                                                           \
        LRBI_SB();                                                 \
        asm volatile("" ::: "memory");                             \
        __builtin_amdgcn_s_barrier();                              \
        asm volatile("" ::: "memory");                             \
        LRBI_SB();                                                 \
    } while (0)

    // ---- prologue: factor slices of panel 0, slabs 0 .. NS - 2 (the last one's X half follows in the first iteration)
    if (tid < 2 * P256_HU * 2) *reinterpret_cast<uint32_t *>(Fz + (tid / (P256_HU * 2)) * P256_FZ_SET + 32 * P256_FZ_ROW + (tid % (P256_HU * 2)) * 4) = 0u;
    load_factors();
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
    wait_loads<kProloguePieces>();
    __syncthreads();
    decode_words();
    decode_store(0);
    wait_loads<kProloguePieces - 4>(); // slab 0
    __syncthreads();
    uint32_t mcur[2], mnext[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) mcur[b] = fetch_mask(0, 0, b) >> (8 * lg);
    static_for<2>([&](auto b) { read_w(I0{}, I0{}, b); });
    static_for<4>([&](auto a) { read_x(I0{}, I0{}, a); });
    static_for<2>([&](auto b) { mask_hi(I0{}, b, mask_lo(I0{}, b, mcur[decltype(b)::value])); });

    // ---- main loop, unrolled by a panel (two rounds of the ring), so that the stage of a slab and its place in the panel are
    // compile-time constants.  Iteration s multiplies slab s out of stage s % NS in two steps.  Between them every wavefront
    // waits until its own pieces of slab s + 1 have landed; the barrier makes the whole slab visible and tells that nobody
    // reads slab s - 1 any more.  What stands between two LRBI_SB() is issued there: the other instructions of a step, spread
    // over its eight matrix instructions.
    // (Behind the last panel one more is formed, from stand-ins, and not used: without tests the waits for operand reads stay
    // exact.)
    uint32_t mt_cur = 0, mt_next = P256_MT; // mask bytes of this panel and of the next one
    for (int s0 = 0; s0 < nslabs; s0 += P256_PSLABS) {
        static_for<P256_PSLABS>([&](auto sc) {
            constexpr int ps = decltype(sc)::value;
            constexpr int st = ps % NS;
            using St = std::integral_constant<int, st>;
            using St1 = std::integral_constant<int, (st + 1) % NS>;
            constexpr int stn = (st + NS - 1) % NS; // stage of slab s + NS - 1
            constexpr int stp = (st + NS - 2) % NS; // stage of slab s + NS - 2
            if (s0 + ps < nslabs) {
                uint32_t y;
                // first step; the second step's operands
                if constexpr (ps >= 3 && ps <= 5) decode_ask();
                read_w(St{}, I1{}, I0{}); read_w(St{}, I1{}, I1{}); read_x(St{}, I1{}, I0{});
                LRBI_SB();
                mma(I0{}, I0{}, I0{}); read_x(St{}, I1{}, I1{});
                LRBI_SB();
                mma(I0{}, I0{}, I1{}); read_x(St{}, I1{}, I2{}); issue_piece(stp, I2{});
                LRBI_SB();
                mma(I0{}, I1{}, I0{}); read_x(St{}, I1{}, I3{}); issue_piece(stp, I3{});
                LRBI_SB();
                mma(I0{}, I1{}, I1{});
                mnext[0] = fetch_mask(ps == P256_PSLABS - 1 ? mt_next : mt_cur, (ps + 1) % P256_PSLABS, 0);
                mnext[1] = fetch_mask(ps == P256_PSLABS - 1 ? mt_next : mt_cur, (ps + 1) % P256_PSLABS, 1);
                LRBI_SB();
                mma(I0{}, I2{}, I0{}); y = mask_lo(I1{}, I0{}, mcur[0]);
                LRBI_SB();
                mma(I0{}, I2{}, I1{}); mask_hi(I1{}, I0{}, y);
                LRBI_SB();
                mma(I0{}, I3{}, I0{}); y = mask_lo(I1{}, I1{}, mcur[1]);
                LRBI_SB();
                mma(I0{}, I3{}, I1{}); mask_hi(I1{}, I1{}, y);
                if constexpr (ps >= 3 && ps <= 5) decode_add();
                LRBI_SB();
                // factor slices of the next panel, asked for at the panel's first slab: landed, for every wavefront,
                // behind the next iteration's wait and barrier
                if constexpr (ps == 0) {
                    load_factors();
                    wait_loads<(NS - 3) * 4 + P256_FACTOR_LOADS>(); // slab s + 1: everything older than these
                } else
                    wait_loads<(NS - 3) * 4>();
                LRBI_BARRIER();
                // second step; the next slab's first operands
                read_w(St1{}, I0{}, I0{}); read_w(St1{}, I0{}, I1{}); read_x(St1{}, I0{}, I0{});
                LRBI_SB();
                mma(I1{}, I0{}, I0{}); read_x(St1{}, I0{}, I1{});
                LRBI_SB();
                mma(I1{}, I0{}, I1{}); read_x(St1{}, I0{}, I2{}); issue_piece(stn, I0{});
                LRBI_SB();
                mma(I1{}, I1{}, I0{}); read_x(St1{}, I0{}, I3{}); issue_piece(stn, I1{});
                LRBI_SB();
                mma(I1{}, I1{}, I1{});
                mcur[0] = mnext[0] >> (8 * lg);
                mcur[1] = mnext[1] >> (8 * lg);
                LRBI_SB();
                mma(I1{}, I2{}, I0{}); y = mask_lo(I0{}, I0{}, mcur[0]);
                LRBI_SB();
                mma(I1{}, I2{}, I1{}); mask_hi(I0{}, I0{}, y);
                LRBI_SB();
                mma(I1{}, I3{}, I0{}); y = mask_lo(I0{}, I1{}, mcur[1]);
                LRBI_SB();
                mma(I1{}, I3{}, I1{}); mask_hi(I0{}, I1{}, y);
                LRBI_SB();
                // mask of the next panel: written in front of slab 6's barrier, first read at slab 7
                if constexpr (ps == 2) decode_words();
                if constexpr (ps == 5) decode_store(mt_next);
            }
        });
        const uint32_t t = mt_cur;
        mt_cur = mt_next;
        mt_next = t;
    }
#undef LRBI_SB
#undef LRBI_BARRIER
    wait_loads<0>(); // nothing may still be landing in LDS
    __syncthreads();

    // ---- epilogue: lane holds, per 32-column block a, columns 8 (v / 4) + 4 lg + (v % 4) of output row l32 of block b.  Each
    // 32 x 128 block goes through the wavefront's own strip of LDS and leaves as 16-byte pieces of whole rows.
    constexpr int RS = 128 * 2 + 8;
    unsigned char *strip = smem + wave * (32 * RS);
    const int l16 = lane & 15, rq = lane >> 4;
    const bool y16 = y_vec_ok && (((uintptr_t)Y & 15) == 0) && (ldy % 8 == 0);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t row0 = m0 + wm * 64 + b * 32;
        if (row0 >= g.m) break; // uniform: whole 128-row halves
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
            const int rr = 4 * i + rq, col = n0 + wn * 128 + 8 * l16;
            const uint2 lo = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16);
            const uint2 hi = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16 + 8);
            uint16_t *yp = Y + (row0 + rr) * ldy + col;
            if (y16 && col + 7 < N) {
                *reinterpret_cast<uint4 *>(yp) = make_uint4(lo.x, lo.y, hi.x, hi.y);
            } else {
                const uint32_t w4[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (col + e < N) yp[e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

// Shapes that this kernel is chosen for, of those that pipe_shape_ok() admits: a round of 256 x 256 tiles takes 2.2 to 2.5
// times a round of 128 x 128 ones (bf16, rank 32, 512 x 512 tiles, us, 256 against 128: 4096 x 4096, N = 4096, 256 tiles:
// 114 / 183; N = 3072, 192 tiles: 95 / 136; 6144 x 4096, N = 1536, 144 tiles: 89 / 121; 5120 x 4096, N = 4096, 320 tiles, two
// rounds against five: 190 / 216; 4096 x 512, N = 4096: 26 / 43; 16384 x 16384, N = 1024: 440 / 642).  Below half a round of
// them the smaller tiles have two rounds at most.
bool pipe256_wins(const Geom &g, int64_t N)
{
    if (!pipe_shape_ok(g) || g.ragged) return false;
    constexpr int64_t cus = 256;
    const int64_t t256 = ((g.m + 255) / 256) * ((N + 255) / 256), t128 = (g.m / 128) * ((N + 127) / 128);
    const int64_t r256 = (t256 + cus - 1) / cus, r128 = (t128 + cus - 1) / cus;
    return r256 * 5 <= r128 * 2;
}

int launch_pipe256_gemm(const Geom &g, lrbi_dtype dt, const void *dW, int64_t ldw, const uint32_t *dIp,
                        const uint32_t *dIz, const void *dX, int64_t ldx, int64_t N, void *dY, int64_t ldy,
                        hipStream_t stream)
{
    const int64_t mblocks = (g.m + P256_B - 1) / P256_B, nblocks = (N + P256_B - 1) / P256_B;
    const int64_t blocks = mblocks * nblocks;
    if (blocks > 0x7FFFFFFF / P256_THREADS) return LRBI_ERR_SHAPE;
    const int y_vec_ok = (((uintptr_t)dY & 7) == 0) && (ldy % 4 == 0);
    const bool half = (g.c % 128) != 0;
    auto kern = dt == LRBI_F16
                    ? (g.ipw == 1 ? (half ? mfma_gemm_pipe256_kernel<F16Tag, 1, true> : mfma_gemm_pipe256_kernel<F16Tag, 1, false>)
                                  : (half ? mfma_gemm_pipe256_kernel<F16Tag, 2, true> : mfma_gemm_pipe256_kernel<F16Tag, 2, false>))
                    : (g.ipw == 1 ? (half ? mfma_gemm_pipe256_kernel<BF16Tag, 1, true> : mfma_gemm_pipe256_kernel<BF16Tag, 1, false>)
                                  : (half ? mfma_gemm_pipe256_kernel<BF16Tag, 2, true> : mfma_gemm_pipe256_kernel<BF16Tag, 2, false>));
    LRBI_SET_MAX_LDS(kern, SmemP256::bytes);
    LRBI_LAUNCH(kern, dim3((unsigned)blocks), dim3(P256_THREADS), SmemP256::bytes, stream, g, (const uint16_t *)dW, ldw, dIp,
                dIz, (const uint16_t *)dX, ldx, (int)N, (uint16_t *)dY, ldy, (int)mblocks, (int)nblocks,
                (blocks % 8 == 0) ? 1 : 0, y_vec_ok);
    return LRBI_OK;
}

} // namespace lrbi
