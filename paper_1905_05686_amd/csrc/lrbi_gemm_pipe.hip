// Fused masked product on the matrix cores, tile kernel with both operands loaded straight into LDS
// (f16 / bf16, fp32 accumulate): Y = (W o I_a) X.  Its forms, and what the host asks of each (all: n and N multiples of 8, X in
// 16-byte pieces, ldw and ldx up to 2^22 elements, for the lanes' 32-bit byte offsets):
//   * base: the mask of Eq. 3 rebuilt inside the kernel, for tile shapes that line up with its blocking (c % 128 == 0, r % 128 ==
//     0, k <= 64, whole tiles; I_z in 16-byte pieces, packed factors below 2^31 bytes each); with CONV on a padded activation below
//     2^32 bytes, with EMIT the mask stored on the way;
//   * HALF: c an odd multiple of 64;
//   * RAG: matrices that end inside a tile, or rows that end inside a 128-column unit;
//   * PRE: any tile shape and rank, on a mask decoded before, its rows up to 2^25 bytes apart.
//
// One workgroup of eight wavefronts (two per SIMD) owns a 128 x 128 tile of Y and walks the reduction range in
// slabs of 64 columns of W.  Wavefront (kg, wq) owns rows 32 wq .. + 31 of the tile for the 16-column steps
// 2 kg and 2 kg + 1 of every slab; the two halves' sums are added through LDS at the end (fixed order).
//   * Both operands of a slab go from global memory straight into LDS (the load-to-LDS form of the global
//     load: no registers, no LDS store instructions, no vector-ALU work), three slabs ahead of the arithmetic,
//     into a ring of four stages.  A lane may fetch any 16-byte piece, but lands it at (stage base + 16 lane):
//     the pieces are fetched in a permuted order, so that the linear image in LDS is the swizzled layout in
//     which the operand reads below hit every bank once (no padding).
//   * The mask is applied where a W operand leaves LDS: the 16 bytes a lane holds for one MFMA are 8
//     consecutive weights of one row, their 8 mask bits one byte of that row's mask.  Pruned weights are zeroed by a
//     packed 16-bit integer multiply by 0 / 1 (a select on the bit pattern: nothing stored under a 0 bit, NaN
//     and Inf included, reaches the product).
//   * The mask itself is rebuilt one panel (512 columns) at a time, one panel ahead, from the panel's slices of
//     the factors (also loaded straight into LDS): mask row = OR of the I_z rows that the row's I_p word selects
//     (Eq. 3); PRE copies the panel.
//   * X stays in its natural [k][n] order in LDS and is read with the transposing LDS read of gfx950.
//   * One workgroup barrier per slab, without a drain of the loads in flight: what must have landed is waited
//     for by count.  Two wavefronts per SIMD: measured, one wavefront per SIMD cannot keep enough 8-byte LDS
//     reads in flight (68 against 160 bytes per clock and compute unit).
//   * The output tile leaves through LDS as 16-byte pieces of whole rows.
#include "lrbi_internal.hpp"
#include "lrbi_lds_dma.hpp"
#include "lrbi_mfma_common.hpp"

namespace lrbi {

static constexpr int PIPE_THREADS = 512;
static constexpr int PIPE_BM = 128, PIPE_BN = 128;
static constexpr int STAGE_BYTES = 32768; // W: 128 rows x 128 bytes, then X: 64 rows x 256 bytes
static constexpr int STAGE_X = 16384;
static constexpr int MT_ROW = 72;                    // bytes per row of a mask panel: 64 + 8 (conflict-free 8-byte reads)
static constexpr int MT_BYTES = PIPE_BM * MT_ROW;    // one mask panel
static constexpr int FZ_ROWS = FAST_MAX_K + 2;       // I_z rows under a panel: 0 .. 31, a zero row, 32 .. 63, a zero row
static constexpr int FZ_ROW_BYTES = PANEL_WORDS * 4; // 64

template <int NS, bool HALF = false> struct SmemDma {
    static constexpr size_t mt_off = (size_t)NS * STAGE_BYTES;
    static constexpr size_t fz_off = mt_off + 2 * MT_BYTES;
    static constexpr size_t fip_off = fz_off + FZ_ROWS * FZ_ROW_BYTES;
    static constexpr size_t bytes = fip_off + PIPE_BM * PANEL_UNITS * (HALF ? 2 : 1) * 2 * 4;
};
static_assert(SmemDma<4, true>::bytes <= 160 * 1024, "LDS of a compute unit");

// order of a launch's tiles: consecutive ones on one XCD; tile row after tile row instead of groups of four rows
static constexpr int kOrderXcd = 1, kOrderRows = 2;


// CONV: X is not a matrix in memory but a zero-padded activation [B][H + 2][Wd + 2][C] (channels fastest), and column
// (b, oh, ow) of the product's X holds, at reduction index (kh * 3 + kw) * C + ci, the value act[b][oh + kh][ow + kw][ci]
// (a 3 x 3 convolution with padding 1 written as a product, the unfolded matrix never materialised).  A slab of 64
// reduction indices is then 64 consecutive channels of one tap: 128 contiguous bytes per column, which go into the
// stage in the same swizzled row-major image as W's rows and come out with the same 16-byte operand reads.
// EMIT: the mask bytes that the kernel rebuilds anyway also go to global memory, in the layout of the stand-alone
// decode (one bit per weight, rows of `mask_pitch16` 16-byte pieces): every (row, 128-column unit) of the mask is
// formed by exactly one workgroup of the first column block, so the decode costs one 16-byte store per lane and
// panel instead of a kernel of its own.
// HALF: tile widths that are an odd multiple of 64 (the paper's 576-column tiles, Table 2): a 128-column unit may
// then lie across two tile columns, so the factor slices are gathered, and Eq. 3 is evaluated, per 64-column half
// unit, each with the I_p word and the I_z words of its own tile.  Everything behind the mask bytes is the same.
// RAG: matrices that end inside a tile, or whose rows end inside a 128-column unit.  Rows past the last one are fetched as the
// last one and not stored; in the last slab, pieces of W past the last column are fetched as the last ones and meet zero mask
// bits (the mask words are cut at the last column), rows of X past the last one too: a short last slab is multiplied behind the
// loop, where the operands of such rows are cleared (an infinity in the last row would come back as a NaN from the zeroed weights;
// a test for that slab inside the loop cost up to 7 % of it).
// PRE: tile shapes that line up with nothing, and any rank.  The mask has been decoded to global memory before (mask_out, rows
// of mask_pitch16 pieces): a panel of it is copied into LDS as it lies there, 64 bytes a row, piece p of row q at slot p ^
// ((q >> 2) & 3), and nothing is formed here.
template <typename Tag, int NS, bool SPREAD, bool SPLIT, bool CONV, bool EMIT = false, bool HALF = false, bool RAG = false, bool PRE = false>
__global__ __launch_bounds__(PIPE_THREADS) void mfma_gemm_pipe_kernel(
    Geom g, const uint16_t *__restrict__ W, int64_t ldw, const uint32_t *__restrict__ Ip,
    const uint32_t *__restrict__ Iz, const uint16_t *__restrict__ X, int64_t ldx, int N,
    uint16_t *__restrict__ Y, int64_t ldy, float *__restrict__ P, int64_t ldp, int mblocks, int nblocks,
    int64_t kper, int order, int y_vec_ok, ConvGeom cg, uint4 *__restrict__ mask_out, int64_t mask_pitch16)
{
    static_assert(NS == 4, "LDS stages (an even number: the W operand registers alternate with the slab's parity)");
    static_assert(!SPREAD || NS == 4, "loads spread over the iteration land one iteration later: four stages");
    constexpr int FN = PIPE_BN / 32; // 32-column blocks of the wave tile
    static_assert(!PRE || (RAG && !EMIT && !HALF), "a decoded mask: the cut-off form, nothing stored");
    static_assert(!(HALF && CONV) && !(RAG && CONV), "half units, cut-off tiles: the plain product only");
    using S = SmemDma<NS, HALF>;

    extern __shared__ uint4 lrbi_dyn_smem[];
    unsigned char *smem = (unsigned char *)lrbi_dyn_smem;
    unsigned char *Mt = smem + S::mt_off;                // [2][128][MT_ROW]  mask bytes of two panels
    uint32_t *Fz = (uint32_t *)(smem + S::fz_off);       // [66][16]          I_z rows under the panel being decoded
    uint32_t *Fip = (uint32_t *)(smem + S::fip_off);     // [128][4][2]       I_p words per row and 128-column unit
                                                         // (HALF: [128][8][2], per 64-column half unit)

    int64_t bid = blockIdx.x;
    if (order & kOrderXcd) {
        const int64_t per = gridDim.x / 8;
        bid = (bid % 8) * per + bid / 8;
    }
    const int slice = (int)(bid / ((int64_t)nblocks * mblocks));
    const int64_t in = bid - (int64_t)slice * nblocks * mblocks;
    int mi, ni;
    if (order & kOrderRows) {
        mi = (int)(in / nblocks);
        ni = (int)(in - (int64_t)mi * nblocks);
    } else
        grouped_tile<4>(in, mblocks, nblocks, &mi, &ni);
    const int64_t m0 = (int64_t)mi * PIPE_BM;
    const int n0 = ni * PIPE_BN;
    const int kbeg = (int)(slice * kper);
    const int kend = (int)((kbeg + kper < g.n) ? kbeg + kper : g.n);
    // whole slabs only: n % 128 == 0 (RAG: n % 8 == 0, the last slab may be short), kper % 128 == 0
    const int nslabs = RAG ? (kend - kbeg + BK - 1) / BK : (kend - kbeg) / BK;
    const int last = nslabs - 1;
    const int ti = (int)(m0 / g.r); // the workgroup's rows lie inside one tile row (r % 128 == 0)
    const int il0 = (int)(m0 - (int64_t)ti * g.r);
    const int64_t trow = (int64_t)ti * g.tile_cols;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // 0 .. 7
    const int kg = wave >> 2;                                  // which half of every slab's 16-column steps
    const int wq = wave & 3;                                   // which 32 rows of the tile
    const int l32 = lane & 31, lg = lane >> 5;

    // ---- global -> LDS: per-lane byte offsets of the pieces this lane fetches (they never change)
    // W stage image: row-major 128-byte rows, piece p of row q stored at slot p ^ ((q >> 1) & 7).  A load
    // instruction fills 1 KiB = 8 rows; wavefront w issues the chunks w and w + 8.
    // X stage image: row-major 256-byte rows, piece p of row q stored at slot p ^ (4 (q & 3)); a load instruction
    // fills 4 rows; same chunk assignment.  (Half a wavefront of a transposing read takes 64 bytes of each of four
    // rows; LDS serves 256 bytes a clock from 64 banks, so the four have to lie 64 bytes apart: measured 256 bytes a
    // clock and compute unit with this swizzle, 128 with rows 32 bytes apart.)
    uint32_t wvo[2], xvo[2], wvl[2], xvl[2]; // (.vl, RAG: in the last slab)
    const int m_last = RAG && g.m - m0 < PIPE_BM ? (int)(g.m - m0) - 1 : PIPE_BM - 1;
    const int k_left = kend - kbeg - last * BK; // columns of the last slab
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int chunk = wave + 8 * i;
        const int wr = chunk * 8 + (lane >> 3);
        const int wp = (lane & 7) ^ ((wr >> 1) & 7);
        const int wrow = RAG && wr > m_last ? m_last : wr;
        wvo[i] = (uint32_t)((wrow * ldw + wp * 8) * 2);
        if constexpr (RAG) wvl[i] = (uint32_t)((wrow * ldw + (wp * 8 < k_left ? wp * 8 : k_left - 8)) * 2);
        if constexpr (CONV) {
            // same image as W: 8 columns of X (128 bytes of channels each) per instruction
            const int xr = chunk * 8 + (lane >> 3);
            const int xp = (lane & 7) ^ ((xr >> 1) & 7);
            int col = n0 + xr;
            if (col >= N) col = N - 1; // column beyond N: a valid column instead, it is dropped at the end
            const int hw = cg.H * cg.Wd;
            const int b = col / hw, rem = col - b * hw;
            const int oh = rem / cg.Wd, ow = rem - oh * cg.Wd;
            const int64_t pix = ((int64_t)b * (cg.H + 2) + oh) * (cg.Wd + 2) + ow; // tap (0, 0) of the column
            xvo[i] = (uint32_t)((pix * cg.cin + xp * 8) * 2);
        } else {
            const int xr = chunk * 4 + (lane >> 4);
            const int xp = (lane & 15) ^ (4 * (xr & 3));
            int nn = xp * 8;
            if (n0 + nn + 8 > N) nn = N - 8 - n0; // piece beyond N: fetch a valid piece instead, its columns are dropped
            xvo[i] = (uint32_t)((xr * ldx + nn) * 2);
            if constexpr (RAG) xvl[i] = (uint32_t)(((xr < k_left ? xr : k_left - 1) * ldx + nn) * 2);
        }
    }
    const uint16_t *wbase = W + m0 * ldw + kbeg;
    const uint16_t *xbase = CONV ? X : X + (int64_t)kbeg * ldx + n0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // The slabs are asked for in order: (wsl, wp), (xsl, xp) are the next slab of W and of X and where it begins; past the
    // last slab the last one is fetched again.  (Pointers that advance: two scalar adds per slab.  The same addresses formed
    // from the slab's number, a division by the channels among them for a convolution, were a third of the loop's scalar
    // instructions, and the loop is bound by the instructions its wavefronts issue.)
    const uint16_t *wp = wbase, *xp = xbase;
    int wsl = 0, xsl = 0;
    int ci = 0, kw = 0; // CONV: channels ci .. ci + 63 of tap (., kw)
    if constexpr (CONV) {
        const int tap = kbeg / cg.cin, kh = tap / 3;
        ci = kbeg - tap * cg.cin;
        kw = tap - 3 * kh;
        xp += (kh * (cg.Wd + 2) + kw) * cg.cin + ci;
    }
    const int64_t xstep = (int64_t)BK * ldx;
    auto next_w = [&]() {
        if (wsl < last) wp += BK;
        ++wsl;
    };
    auto next_x = [&]() {
        if (xsl < last) {
            if constexpr (CONV) {
                xp += BK; // the next channels, or the first ones of the next tap: the pixel to the right
                ci += BK;
                if (ci == cg.cin) {
                    ci = 0;
                    if (++kw == 3) { // the first pixel of the tap row below
                        kw = 0;
                        xp += (cg.Wd + 2 - 3) * cg.cin;
                    }
                }
            } else
                xp += xstep;
        }
        ++xsl;
    };
    // piece i (0, 1: W chunks, 2, 3: X chunks) of the next slab into a stage; the second piece moves on
    const uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    auto issue_piece = [&](int stage, auto i_c) {
        constexpr int i = decltype(i_c)::value;
        const uint32_t sb = lds_w + (uint32_t)stage * STAGE_BYTES;
        if constexpr (i < 2) load_to_lds16(sb + i * 8192u, wp, RAG && wsl >= last ? wvl[i] : wvo[i]);
        else load_to_lds16(sb + STAGE_X + (i - 2) * 8192u, xp, RAG && xsl >= last ? xvl[i - 2] : xvo[i - 2]);
        if constexpr (i == 1) next_w();
        if constexpr (i == 3) next_x();
    };

    // ---- operand reads: byte addresses inside a stage.  This wavefront's steps are kk = 2 kg + j, j = 0, 1.
    // W operand of step kk: row q = 32 wq + (lane % 32), piece 2 kk + (lane / 32)
    uint32_t wfa[2];
    {
        const int q = wq * 32 + l32;
        const int c7 = (q >> 1) & 7;
#pragma unroll
        for (int j = 0; j < 2; ++j) wfa[j] = (uint32_t)(q * 128 + (((2 * (2 * kg + j) + lg) ^ c7) * 16));
    }
    // X operand (transposing read): 16-lane group G = lane / 16 serves columns 16 (G % 2) .. + 15 of a
    // 32-column block and k group G / 2; lane d of the group addresses row d / 4, columns 4 (d % 4).
    // Block a sits at 64 (a ^ (q & 3)), q the row.
    const int d16 = lane & 15, G16 = lane >> 4;
    uint32_t xfa[FN]; // step j = 0 (+4096 for j = 1)
    {
        const int q = 8 * (G16 >> 1) + (d16 >> 2); // row inside the step (+ 4 for the upper half)
        const uint32_t base = (uint32_t)(STAGE_X + kg * 8192 + q * 256 + (2 * (G16 & 1) + ((d16 & 3) >> 1)) * 16 + 8 * (d16 & 1));
#pragma unroll
        for (int a = 0; a < FN; ++a) xfa[a] = base + 64u * (uint32_t)(a ^ (q & 3));
    }
    // mask bytes of this lane's row: 8 bytes per slab, of which this wavefront's steps use bytes 4 kg + 2 j + lg
    const uint32_t mta = (uint32_t)((wq * 32 + l32) * (PRE ? 64 : MT_ROW) + 4 * kg);

    u32x4 wf[2][2], xf[2][FN]; // W operands [slab parity][j]; X operands [j][block]
    auto read_w = [&](int stage, auto par_c, auto j_c) {
        constexpr int par = decltype(par_c)::value, j = decltype(j_c)::value;
        wf[par][j] = *reinterpret_cast<const u32x4 *>(smem + stage * STAGE_BYTES + wfa[j]);
    };
    // CONV: X operand of step kk, block a: column q = 32 a + (lane % 32), piece 2 kk + (lane / 32), image as W's
    uint32_t xca[2];
    {
        const int c7 = (l32 >> 1) & 7; // (q >> 1) & 7 does not depend on the block
#pragma unroll
        for (int j = 0; j < 2; ++j) xca[j] = (uint32_t)(STAGE_X + l32 * 128 + (((2 * (2 * kg + j) + lg) ^ c7) * 16));
    }
    auto read_x = [&](int stage, auto j_c, auto a_c) {
        constexpr int j = decltype(j_c)::value, a = decltype(a_c)::value;
        if constexpr (CONV) {
            xf[j][a] = *reinterpret_cast<const u32x4 *>(smem + stage * STAGE_BYTES + xca[j] + a * 4096);
            return;
        }
        const unsigned char *p = smem + stage * STAGE_BYTES + xfa[a] + j * 4096;
        const u32x2 lo = lds_read_tr16_v((const uint16_t *)p);
        const u32x2 hi = lds_read_tr16_v((const uint16_t *)(p + 1024));
        xf[j][a] = u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    f32x16 acc[FN];
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][v] = 0.f;
    auto mma = [&](auto par_c, auto j_c, auto a_c) {
        constexpr int par = decltype(par_c)::value, j = decltype(j_c)::value, a = decltype(a_c)::value;
        acc[a] = mfma_32x32x16(Tag{}, xf[j][a], wf[par][j], acc[a]);
    };
    // mask of a W operand: m holds this wavefront's two mask bytes of the slab, step j's at bits 16 j
    auto mask_lo = [&](auto par_c, auto j_c, uint32_t m) -> uint32_t {
        constexpr int par = decltype(par_c)::value, j = decltype(j_c)::value;
        const uint32_t bits8 = (m >> (16 * j)) & 0xFFu;
        const uint32_t y = bits8 | (bits8 << 15);
        wf[par][j].x = select2(wf[par][j].x, y & 0x00010001u);
        wf[par][j].y = select2(wf[par][j].y, (y >> 2) & 0x00010001u);
        return y;
    };
    auto mask_hi = [&](auto par_c, auto j_c, uint32_t y) {
        constexpr int par = decltype(par_c)::value, j = decltype(j_c)::value;
        wf[par][j].z = select2(wf[par][j].z, (y >> 4) & 0x00010001u);
        wf[par][j].w = select2(wf[par][j].w, (y >> 6) & 0x00010001u);
    };
    auto fetch_mask = [&](int slab) -> uint32_t {
        const uint32_t us = (uint32_t)slab;
        if constexpr (PRE) {
            const uint32_t slot = ((us % PANEL_SLABS) >> 1) ^ (uint32_t)((l32 >> 2) & 3);
            return *reinterpret_cast<const uint32_t *>(Mt + ((us / PANEL_SLABS) & 1u) * 8192u + mta + slot * 16u + (us & 1u) * 8u);
        }
        const unsigned char *p = Mt + ((us / PANEL_SLABS) & 1u) * MT_BYTES + (us % PANEL_SLABS) * 8u + mta;
        return *reinterpret_cast<const uint32_t *>(p);
    };
    auto my_bytes = [&](uint32_t mk) -> uint32_t { return mk >> (8 * lg); };

    // ---- factor slices of one panel: global -> LDS (the same load-to-LDS form), then Eq. 3 for the panel.
    // A lane fetches for one of the panel's 128-column units (HALF: 64-column half units), each inside one tile: fz_u of I_z,
    // fp_u of I_p; (.tj, .off, .col): that unit's tile column, offset in it and first column, carried from panel to panel.
    // I_z: wavefronts 0 .. 3 fetch ranks 16 w .. + 15, lane = (rank, unit): the unit's four words of that
    // rank's row.  Ranks at or beyond k fetch rank 0 instead: no I_p bit selects them (pad bits are zero).
    // Units beyond the reduction range fetch the tile row's first tile instead: their mask bytes are never read.
    // I_p: one word per lane, 256 bytes per instruction, two instructions per wavefront, image [row][unit][2];
    // with one word per row the second word's slot receives the first word again and is ignored below.
    // (Per lane, not for all units with the lane's picked: a third of the instructions.)
    struct Unit {
        int col, tj, off;
    };
    auto unit_at = [&](int col) {
        const int tj = col / g.c;
        return Unit{col, tj, col - tj * g.c};
    };
    auto next_panel = [&](Unit &u) {
        u.col += PW;
        u.off += PW;
        while (u.off >= g.c) {
            u.off -= g.c;
            ++u.tj;
        }
    };
    Unit fz_u = unit_at(kbeg + (HALF ? 64 * ((lane >> 1) & 7) : 128 * (lane & 3)));
    Unit fp_u = unit_at(kbeg + (HALF ? 64 * ((lane >> 1) & 7) : 128 * ((lane >> 1) & 3)));
    const uint32_t izs = (uint32_t)(g.k * g.izw * 4), ips = (uint32_t)(g.r * g.ipw * 4); // bytes of a tile's factors
    const uint32_t z_row = (uint32_t)trow * izs, p_row = (uint32_t)trow * ips + (uint32_t)(il0 * g.ipw * 4);
    const int fz_l = wq * 16 + (lane >> 2);
    const uint32_t fz_lane = (uint32_t)(((fz_l < g.k) ? fz_l : 0) * g.izw * 4);
    int pre_piece = kbeg / 128 + ((lane & 3) ^ ((lane >> 4) & 3)), pre_buf = 0; // PRE: this lane's piece of the next panel
    const int pre_row = wave * 16 + (lane >> 2);
    const uint32_t pre_off = (uint32_t)((pre_row < m_last ? pre_row : m_last) * mask_pitch16 * 16);
    const int pre_last = (int)((g.n + 127) / 128) - 1;
    auto load_factors = [&]() {
        if constexpr (PRE) {
            load_to_lds16(lds0 + (uint32_t)S::mt_off + (uint32_t)(pre_buf * 8192 + wave * 1024), mask_out + m0 * mask_pitch16,
                          pre_off + (uint32_t)((pre_piece < pre_last ? pre_piece : pre_last) * 16));
            pre_piece += PANEL_UNITS;
            pre_buf ^= 1;
            return;
        }
        const uint32_t zsel = z_row + (fz_u.col < kend ? (uint32_t)fz_u.tj * izs + (uint32_t)(fz_u.off >> 5) * 4u : 0u);
        const uint32_t psel = p_row + (fp_u.col < kend ? (uint32_t)fp_u.tj * ips : 0u);
        next_panel(fz_u);
        next_panel(fp_u);
        if constexpr (HALF) {
            // per half unit (64 columns, two words of an I_z row): one word per lane.  I_z: instruction q of 16
            // (two per wavefront) fills ranks 4 q .. + 3, lane = (rank, half unit, word); I_p: image
            // [row][half unit][2], four instructions per wavefront.
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = wave * 2 + i;
                const int rank = q * 4 + (lane >> 4);
                load_to_lds4(lds0 + (uint32_t)S::fz_off + (uint32_t)(q * 256 + (q >= 8 ? FZ_ROW_BYTES : 0)), Iz,
                             zsel + (uint32_t)((((rank < g.k) ? rank : 0) * g.izw + (lane & 1)) * 4));
            }
            const int iw = (lane & 1) < g.ipw ? (lane & 1) : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = wave * 4 + i;
                const int row = q * 4 + (lane >> 4);
                load_to_lds4(lds0 + (uint32_t)S::fip_off + (uint32_t)q * 256u, Ip, psel + (uint32_t)((row * g.ipw + iw) * 4));
            }
            return;
        }
        if (kg == 0) load_to_lds16(lds0 + (uint32_t)S::fz_off + (uint32_t)(wq * 1024 + (wq >= 2 ? FZ_ROW_BYTES : 0)), Iz, zsel + fz_lane);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int idx = (wave * 2 + i) * 64 + lane;
            const int row = idx >> 3, iw = (idx & 1) < g.ipw ? (idx & 1) : 0;
            load_to_lds4(lds0 + (uint32_t)S::fip_off + (uint32_t)(wave * 2 + i) * 256u, Ip, psel + (uint32_t)((row * g.ipw + iw) * 4));
        }
    };
    // Eq. 3 for the panel.  A lane forms the 4 mask words of one row under one 128-column unit (HALF: under its two half
    // units, each from the factors of its own tile).  The set ranks are taken two at a time, over three slabs of the loop, so
    // that the reads have come back when they are added (all at once took a tenth of a product's time); rows with more
    // ranks than that (few: the factors are sparse) loop over the rest.  Ranks are found in one 32-bit word of I_p at a time,
    // the first one and, where there is one, the second; a word without one left reads the zero row behind the word's
    // rows, which is where counting its trailing zeros (32) leads.
    constexpr int NH = HALF ? 2 : 1;
    using zvec = std::conditional_t<HALF, u32x2, u32x4>;
    const int drow = tid >> 2, du = tid & 3;
    const unsigned char *dfz = (const unsigned char *)Fz + du * 16;
    uint32_t sel[NH], sel2[NH]; // the word in work and the one that waits
    uint32_t dbase = 0, dbase2 = 33 * FZ_ROW_BYTES;
    zvec dz[NH][2], dh[NH];
    auto decode_words = [&]() {
        const uint32_t *fp = Fip + (drow * PANEL_UNITS + du) * (HALF ? 4 : 2);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            sel[h] = fp[2 * h];
            sel2[h] = g.ipw > 1 ? fp[2 * h + 1] : 0u;
            dh[h] = zvec(0u);
        }
        dbase = 0;
        dbase2 = 33 * FZ_ROW_BYTES;
    };
    auto decode_other = [&](bool turn) { // the waiting word, if `turn`
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const uint32_t t = sel[h];
            sel[h] = turn ? sel2[h] : t;
            sel2[h] = turn ? t : sel2[h];
        }
        const uint32_t t = dbase;
        dbase = turn ? dbase2 : t;
        dbase2 = turn ? t : dbase2;
    };
    auto decode_ask = [&]() {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t l = sel[h] ? (uint32_t)__builtin_ctz(sel[h]) : 32u;
                sel[h] &= sel[h] - 1u;
                dz[h][e] = *reinterpret_cast<const zvec *>(dfz + dbase + l * FZ_ROW_BYTES + h * 8);
            }
    };
    auto decode_add = [&]() {
#pragma unroll
        for (int h = 0; h < NH; ++h) dh[h] |= dz[h][0] | dz[h][1];
    };
    auto decode_store = [&](int panel) {
        auto left = [&]() {
            uint32_t any = sel[0];
            if constexpr (HALF) any |= sel[1];
            return any;
        };
        while (left()) {
            decode_ask();
            decode_add();
        }
        if (g.ipw > 1) {
            decode_other(true);
            while (left()) {
                decode_ask();
                decode_add();
            }
        }
        uint4 a;
        if constexpr (HALF) a = make_uint4(dh[0].x, dh[0].y, dh[1].x, dh[1].y);
        else a = make_uint4(dh[0].x, dh[0].y, dh[0].z, dh[0].w);
        if constexpr (RAG) { // whatever the factors hold beyond the last column stays out
            const int left = kend - (kbeg + panel * PW + du * 128);
            a.x &= bit_range(0, left < 0 ? 0 : (left < 32 ? left : 32));
            a.y &= bit_range(0, left < 32 ? 0 : (left < 64 ? left - 32 : 32));
            a.z &= bit_range(0, left < 64 ? 0 : (left < 96 ? left - 64 : 32));
            a.w &= bit_range(0, left < 96 ? 0 : (left < 128 ? left - 96 : 32));
        }
        unsigned char *out = Mt + (panel & 1) * MT_BYTES + drow * MT_ROW + du * 16;
        *reinterpret_cast<uint2 *>(out) = make_uint2(a.x, a.y);
        *reinterpret_cast<uint2 *>(out + 8) = make_uint2(a.z, a.w);
        if constexpr (EMIT) {
            // units past the end of this workgroup's reduction range were formed from stand-in factors: not stored
            const int unit = kbeg / 128 + panel * PANEL_UNITS + du;
            if (ni == 0 && unit * 128 < kend && drow <= m_last) mask_out[(m0 + drow) * mask_pitch16 + unit] = a;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the mask bytes have landed before the next barrier
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
// nothing crosses this line when the compiler orders the instructions
#define LRBI_SB() __builtin_amdgcn_sched_barrier(0)
// workgroup barrier without the compiler's own "wait for every outstanding memory operation" in front of it (that
// wait would drain the slabs in flight); what has to be complete is waited for explicitly.  Operand reads of slab s may be
// under way across it: what is handed over is the stage of slab s - 1, whose operands have all been multiplied.
#define LRBI_BARRIER()                                             \
    do {                                                           \
        LRBI_SB();                                                 \
        asm volatile("" ::: "memory");                             \
        __builtin_amdgcn_s_barrier();                              \
        asm volatile("" ::: "memory");                             \
        LRBI_SB();                                                 \
    } while (0)

    // ---- prologue: the factor slices of panel 0 first, then slabs 0 .. NS - 2; the panel is decoded as soon as the
    // factor slices are in (the slabs issued behind them stay in flight), and slab 0 is waited for after that
    if (tid < 2 * PANEL_WORDS) Fz[(tid < PANEL_WORDS ? 32 : 64) * PANEL_WORDS + tid] = 0u; // rows 32 and 65
    load_factors();
    constexpr int kProloguePieces = SPREAD ? (NS - 2) * 4 + 2 : (NS - 1) * 4; // slab copies of this wavefront behind them
    static_for<NS - 1>([&](auto sc) {
        constexpr int st = decltype(sc)::value;
        issue_piece(st, I0{});
        issue_piece(st, I1{});
        if constexpr (!(SPREAD && st == NS - 2)) { // SPREAD: the last slab's other half follows in the first iteration
            issue_piece(st, I2{});
            issue_piece(st, I3{});
        }
    });
    if constexpr (!PRE) {
        wait_loads<kProloguePieces>();
        __syncthreads();
        decode_words();
        decode_store(0);
    }
    // slab 0 (EMIT: a mask store, where there is one, is younger: the wait is one piece longer than it has to be)
    wait_loads<kProloguePieces - 4>();
    __syncthreads();
    // entry state of the loop: X operands of this wavefront's first step, its W operand masked, the second read
    uint32_t mcur = my_bytes(fetch_mask(0));
    read_w(0, I0{}, I0{});
    read_w(0, I0{}, I1{});
    read_x(0, I0{}, I0{});
    read_x(0, I0{}, I1{});
    read_x(0, I0{}, I2{});
    read_x(0, I0{}, I3{});
    {
        const uint32_t y = mask_lo(I0{}, I0{}, mcur);
        mask_hi(I0{}, I0{}, y);
    }

    // ---- main loop, unrolled by a panel (two rounds of the ring), so that the stage of a slab and its place in the panel are
    // compile-time constants.
    // Iteration s multiplies slab s out of stage s % NS: each wavefront its two 16-column steps.  After the
    // first step every wavefront waits until its own pieces of slab s + 1 have landed; the barrier makes the
    // whole slab visible and tells that nobody reads slab s - 1 any more; the second step then runs next to the
    // loads of slab s + NS - 1 into the stage slab s - 1 occupied and to the reads of slab s + 1's operands.
    // The next panel's mask is formed in any case, behind the last one from that one's factors (and not used): tests there would
    // cost more than it does.  Its factors are asked for only where there is one: slab 1 waits for them, and slices of a panel or
    // two, which have nothing else to wait for, took up to a tenth longer (256 x 4608 convolution, two images of 28 x 28, slices of
    // one panel 16.8 us against 18.5; 40 images of 10 x 10 on 512 x 2304, slices of 18 slabs 24.1 against 25.4).
    static_assert(PANEL_SLABS == 2 * NS, "two rounds of the ring");
    const bool tail = RAG && k_left < BK; // the last slab is short: multiplied behind the loop
    const int nloop = tail ? nslabs - 1 : nslabs;
    for (int s0 = 0; s0 < nloop; s0 += PANEL_SLABS) {
        static_for<PANEL_SLABS>([&](auto sc) {
            constexpr int ps = decltype(sc)::value;
            constexpr int st = ps % NS;                   // stage of slab s
            constexpr int st1 = (st + 1) % NS;            // stage of slab s + 1
            constexpr int stn = (st + NS - 1) % NS;       // stage of slab s - 1 = stage of slab s + NS - 1
            constexpr int stp = (st + NS - 2) % NS;       // stage of slab s - 2 = stage of slab s + NS - 2
            using Par = std::integral_constant<int, st & 1>;        // register set of slab s's W operands
            using Nxt = std::integral_constant<int, (st & 1) ^ 1>;  // ... of slab s + 1's
            const int s = s0 + ps;
            if (s < nloop) {
                uint32_t y;
                uint32_t mk;
                // first step
                if constexpr (ps == 4 && !PRE) decode_other(g.ipw > 1);
                if constexpr (ps >= 3 && ps <= 5 && !PRE) decode_ask();
                mma(Par{}, I0{}, I0{}); read_x(st, I1{}, I0{}); y = mask_lo(Par{}, I1{}, mcur);
                mma(Par{}, I0{}, I1{}); read_x(st, I1{}, I1{}); mask_hi(Par{}, I1{}, y);
                if constexpr (SPREAD) issue_piece(stp, I2{});
                mma(Par{}, I0{}, I2{}); read_x(st, I1{}, I2{});
                mk = fetch_mask(s + 1); // mask bytes of the next slab (past the last one: not used)
                mma(Par{}, I0{}, I3{}); read_x(st, I1{}, I3{});
                if constexpr (SPREAD) issue_piece(stp, I3{});
                if constexpr (ps >= 3 && ps <= 5 && !PRE) decode_add();
                // factor slices of the next panel, requested at the panel's first slab: they have landed, for
                // every wavefront, behind the next iteration's wait and barrier
                if (ps == 0 && s0 + PANEL_SLABS < nslabs) {
                    load_factors();
                    wait_loads<(NS - 3) * 4 + (PRE ? 1 : HALF ? 6 : 2)>(); // slab s + 1 (younger: four, and two or three factor loads, HALF six, PRE one)
                } else
                    wait_loads<(NS - 3) * 4>(); // slab s + 1 has landed (four younger loads may still be in flight)
                LRBI_BARRIER();
                // second step
                mma(Par{}, I1{}, I0{}); read_x(st1, I0{}, I0{}); read_w(st1, Nxt{}, I0{}); read_w(st1, Nxt{}, I1{});
                issue_piece(stn, I0{});
                mma(Par{}, I1{}, I1{}); read_x(st1, I0{}, I1{}); mcur = my_bytes(mk);
                issue_piece(stn, I1{});
                mma(Par{}, I1{}, I2{}); read_x(st1, I0{}, I2{}); y = mask_lo(Nxt{}, I0{}, mcur);
                if constexpr (!SPREAD) issue_piece(stn, I2{});
                mma(Par{}, I1{}, I3{}); read_x(st1, I0{}, I3{}); mask_hi(Nxt{}, I0{}, y);
                if constexpr (!SPREAD) issue_piece(stn, I3{});
                // mask of the next panel: its words at slab 2, written in front of slab 6's barrier, first read at slab 7
                if constexpr (ps == 2 && !PRE) decode_words();
                if constexpr (ps == 5 && !PRE) decode_store(s / PANEL_SLABS + 1);
            }
        });
    }
#undef LRBI_SB
#undef LRBI_BARRIER
    if constexpr (RAG) {
        if (tail) { // its first operands are in registers, as in front of any other slab
            static_for<NS>([&](auto sc) {
                constexpr int st = decltype(sc)::value;
                using Par = std::integral_constant<int, st & 1>;
                if (last % NS != st) return;
                static_for<FN>([&](auto a) { read_x(st, I1{}, a); });
                mask_hi(Par{}, I1{}, mask_lo(Par{}, I1{}, mcur));
                static_for<2>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value;
                    const bool in = 16 * (2 * kg + j) + 8 * lg < k_left; // the eight rows of X that this lane holds
                    static_for<FN>([&](auto a_c) {
                        constexpr int a = decltype(a_c)::value;
                        if (!in) xf[j][a] = u32x4{0u, 0u, 0u, 0u};
                        mma(Par{}, j_c, a_c);
                    });
                });
            });
        }
    }
    wait_loads<0>(); // nothing may still be landing in LDS
    __syncthreads();

    // ---- the two halves of the reduction range: wavefronts 4 .. 7 hand their sums to wavefronts 0 .. 3 through LDS
    {
        float *red = (float *)smem + (size_t)wq * (FN * 16 * 64) + lane; // [wq][a][v][lane]; the stages are dead now
        if (kg == 1) {
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int v = 0; v < 16; ++v) red[(a * 16 + v) * 64] = acc[a][v];
        }
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int a = 0; a < FN; ++a)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][v] += red[(a * 16 + v) * 64];
    }

    // ---- epilogue: lane holds, per 32-column block a, columns n = 8 (v / 4) + 4 lg + (v % 4) of output row l32.
    // The wavefront's 32 x 128 block goes through its own strip of LDS (rounded to the output type first, or as
    // fp32 for a partial plane) and leaves as 16-byte pieces of whole rows.
    const int64_t row0 = m0 + wq * 32;
    if (SPLIT) {
        constexpr int RS = 128 * 4 + 16; // bytes per staged row
        unsigned char *strip = smem + 65536 + wq * (32 * RS);
#pragma unroll
        for (int a = 0; a < FN; ++a)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                *reinterpret_cast<float4 *>(strip + l32 * RS + (a * 32 + 8 * v4 + 4 * lg) * 4) =
                    make_float4(acc[a][4 * v4 + 0], acc[a][4 * v4 + 1], acc[a][4 * v4 + 2], acc[a][4 * v4 + 3]);
        // (the strip is private to the wavefront: its own LDS operations complete in order)
#pragma unroll
        for (int i = 0; i < 16; ++i) { // 2 rows per instruction: 32 lanes x 16 bytes per row
            const int rr = 2 * i + lg, col = n0 + 4 * l32;
            const float4 o = *reinterpret_cast<const float4 *>(strip + rr * RS + l32 * 16);
            // (non-temporal: the planes are read once, by another kernel; measured 0.6-0.8 us of the call on a
            // 4096 x 9216 matrix at 128 columns, most of it the end of this kernel)
            typedef float nt_f4 __attribute__((ext_vector_type(4)));
            nt_f4 ov = {o.x, o.y, o.z, o.w};
            if (col < ldp && (!RAG || row0 + rr < g.m)) __builtin_nontemporal_store(ov, reinterpret_cast<nt_f4 *>(P + ((int64_t)slice * g.m + row0 + rr) * ldp + col));
        }
    } else {
        constexpr int RS = 128 * 2 + 8;
        unsigned char *strip = smem + 65536 + wq * (32 * RS);
#pragma unroll
        for (int a = 0; a < FN; ++a)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                uint16_t o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = cvt_store(Tag{}, acc[a][4 * v4 + e]);
                *reinterpret_cast<uint2 *>(strip + l32 * RS + (a * 32 + 8 * v4 + 4 * lg) * 2) = *reinterpret_cast<uint2 *>(o);
            }
        const int l16 = lane & 15, rq = lane >> 4;
        const bool y16 = y_vec_ok && (((uintptr_t)Y & 15) == 0) && (ldy % 8 == 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) { // 4 rows per instruction: 16 lanes x 16 bytes per row
            const int rr = 4 * i + rq, col = n0 + 8 * l16;
            const uint2 lo = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16);
            const uint2 hi = *reinterpret_cast<const uint2 *>(strip + rr * RS + l16 * 16 + 8);
            uint16_t *yp = Y + (row0 + rr) * ldy + col;
            if (RAG && row0 + rr >= g.m) continue;
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

// tile shapes the pipelined kernel's blocking lines up with: tile rows in blocks of 128, tile widths a multiple of
// 128, or of 64 (gathered per half unit); the matrix may end inside a tile, its rows are whole 16-byte pieces
bool pipe_shape_ok(const Geom &g)
{
    if ((g.r % PIPE_BM) != 0 || g.k > FAST_MAX_K) return false;
    return (g.c % 64) == 0 && g.n % 8 == 0;
}

// true when the pipelined kernel serves this call: aligned tile shapes, X readable in 16-byte pieces, offsets
// that fit the kernel's 32-bit per-lane byte offsets
bool pipe_ok(const Geom &g, const void *dIz, const void *dX, int64_t ldw, int64_t ldx, int64_t N)
{
    if (!pipe_shape_ok(g)) return false;
    if ((((uintptr_t)dX & 15) != 0) || (ldx % 8 != 0) || (N % 8 != 0) || N < 8) return false;
    if (((uintptr_t)dIz & 15) != 0) return false; // the I_z slices are fetched in 16-byte pieces
    if (ldw > (1 << 22) || ldx > (1 << 22)) return false;
    // byte offsets into the packed factors are kept in 32 bits
    const int64_t tiles = (int64_t)g.tile_rows * g.tile_cols;
    if (tiles * g.k * g.izw * 4 >= (int64_t)1 << 31 || tiles * g.r * g.ipw * 4 >= (int64_t)1 << 31) return false;
    return true;
}

// the same for the form that reads a decoded mask: any tile shape and rank.  A lane's byte offset into the mask rows of its
// tile has 32 bits as well: the last byte of 128 rows lies below 2^32.
bool pipe_given_ok(const Geom &g, const void *dX, int64_t ldw, int64_t ldx, int64_t N, int64_t mask_pitch_bytes)
{
    if ((((uintptr_t)dX & 15) != 0) || (ldx % 8 != 0) || (N % 8 != 0) || N < 8 || g.n % 8 != 0) return false;
    return ldw <= (1 << 22) && ldx <= (1 << 22) && mask_pitch_bytes <= ((int64_t)1 << 32) / PIPE_BM;
}

template <typename Tag, int NS, bool SPREAD, bool CONV, bool EMIT = false, bool HALF = false, bool RAG = false, bool PRE = false>
static int launch_pipe_t(const Geom &g, const MfmaPlan &plan, const void *dW, int64_t ldw, const uint32_t *dIp,
                         const uint32_t *dIz, const void *dX, int64_t ldx, int64_t N, void *dY, int64_t ldy,
                         void *dWorkspace, const ConvGeom &cg, hipStream_t stream, MaskOut mo = {nullptr, 0})
{
    const int64_t mblocks = (g.m + PIPE_BM - 1) / PIPE_BM;
    const int64_t nblocks = (N + PIPE_BN - 1) / PIPE_BN;
    const int64_t blocks = mblocks * nblocks * plan.splitk;
    if (blocks > 0x7FFFFFFF) return LRBI_ERR_SHAPE;
    const bool split = plan.splitk > 1 || plan.planes_only;
    const int y_vec_ok = (((uintptr_t)dY & 7) == 0) && (ldy % 4 == 0);
    // Groups of four tile rows where the tiles make several rounds or have the chip to themselves.  Slices whose tiles are dealt
    // to the XCDs in one piece each, and convolutions of two or three tile rows, go row after row (us, groups against rows: 256 x
    // 4608, two images of 28 x 28, nine slices 18.3 / 16.8, 40 of 10 x 10 on 256 x 2304, four slices 20.7 / 19.8; 384 x 4608, 13 of
    // 14 x 14 24.9 / 22.9, 96 of 28 x 28 316 / 305; 512 x 4096, N = 2048, four slices 22.6 / 21.2; 4096 x 9216, N = 512 49.6 / 47.7; but
    // 1500 x 4104, N = 512 20.9 / 21.6; without slices 4096 x 9216, N = 2048 164 / 172, 256 x 4608, 20 of 28 x 28 42.7 / 44.2).
    const bool xcd = blocks % 8 == 0;
    const bool rows = plan.splitk > 1 ? (xcd || (CONV && mblocks < 4)) : (CONV && mblocks == 3);
    const int order = (xcd ? kOrderXcd : 0) | (rows ? kOrderRows : 0);
    const int64_t ldp = (N + 3) / 4 * 4;
    const size_t smem = SmemDma<NS, HALF>::bytes;
    auto kern = split ? mfma_gemm_pipe_kernel<Tag, NS, SPREAD, true, CONV, EMIT, HALF, RAG, PRE>
                      : mfma_gemm_pipe_kernel<Tag, NS, SPREAD, false, CONV, EMIT, HALF, RAG, PRE>;
    LRBI_SET_MAX_LDS(kern, smem);
    LRBI_LAUNCH(kern, dim3((unsigned)blocks), dim3(PIPE_THREADS), smem, stream, g, (const uint16_t *)dW, ldw, dIp, dIz,
                (const uint16_t *)dX, ldx, (int)N, (uint16_t *)dY, ldy, (float *)dWorkspace, ldp, (int)mblocks,
                (int)nblocks, plan.kper, order, y_vec_ok, cg, (uint4 *)mo.ptr, mo.pitch16);
    return LRBI_OK;
}

// variant 0, 1: a slab's loads issued in a burst right after the barrier (longest time to land: weights streaming
// from HBM); 2: loads spread evenly over the iteration (operands coming from L2).
// The caller adds the partial planes when the plan is split.
int launch_pipe_gemm(const Geom &g, const MfmaPlan &plan, lrbi_dtype dt, int variant, const void *dW, int64_t ldw,
                     const uint32_t *dIp, const uint32_t *dIz, const void *dX, int64_t ldx, int64_t N, void *dY,
                     int64_t ldy, void *dWorkspace, hipStream_t stream, MaskOut mo)
{
    const ConvGeom none = {0, 0, 0};
    if (plan.mask_given) { // the mask is in mo already
        if (dt == LRBI_F16)
            return launch_pipe_t<F16Tag, 4, true, false, false, false, true, true>(g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy,
                                                                                    dWorkspace, none, stream, mo);
        if (dt == LRBI_BF16)
            return launch_pipe_t<BF16Tag, 4, true, false, false, false, true, true>(g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy,
                                                                                     dWorkspace, none, stream, mo);
        return LRBI_ERR_DTYPE;
    }
    if (g.ragged || g.n % 128 != 0) { // cut-off tiles or panels: one variant per dtype and kind of unit, with or without the mask
#define LRBI_PIPE_RAG(TAG, EM, HF)                                                                                           \
    launch_pipe_t<TAG, 4, true, false, EM, HF, true>(g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy, dWorkspace, none, stream, mo)
        const bool half = g.c % 128 != 0;
        if (dt == LRBI_F16) {
            if (mo.ptr) return half ? LRBI_PIPE_RAG(F16Tag, true, true) : LRBI_PIPE_RAG(F16Tag, true, false);
            return half ? LRBI_PIPE_RAG(F16Tag, false, true) : LRBI_PIPE_RAG(F16Tag, false, false);
        }
        if (dt == LRBI_BF16) {
            if (mo.ptr) return half ? LRBI_PIPE_RAG(BF16Tag, true, true) : LRBI_PIPE_RAG(BF16Tag, true, false);
            return half ? LRBI_PIPE_RAG(BF16Tag, false, true) : LRBI_PIPE_RAG(BF16Tag, false, false);
        }
#undef LRBI_PIPE_RAG
        return LRBI_ERR_DTYPE;
    }
    if (g.c % 128 != 0) { // half units: one variant per dtype (loads spread over the iteration), with or without the mask
#define LRBI_PIPE_ARGS g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy, dWorkspace, none, stream, mo
        if (dt == LRBI_F16)
            return mo.ptr ? launch_pipe_t<F16Tag, 4, true, false, true, true>(LRBI_PIPE_ARGS)
                          : launch_pipe_t<F16Tag, 4, true, false, false, true>(LRBI_PIPE_ARGS);
        if (dt == LRBI_BF16)
            return mo.ptr ? launch_pipe_t<BF16Tag, 4, true, false, true, true>(LRBI_PIPE_ARGS)
                          : launch_pipe_t<BF16Tag, 4, true, false, false, true>(LRBI_PIPE_ARGS);
#undef LRBI_PIPE_ARGS
        return LRBI_ERR_DTYPE;
    }
    if (mo.ptr) { // the mask as a by-product: one variant per dtype (loads spread over the iteration)
        if (dt == LRBI_F16)
            return launch_pipe_t<F16Tag, 4, true, false, true>(g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy, dWorkspace,
                                                               none, stream, mo);
        if (dt == LRBI_BF16)
            return launch_pipe_t<BF16Tag, 4, true, false, true>(g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy, dWorkspace,
                                                                none, stream, mo);
        return LRBI_ERR_DTYPE;
    }
#define LRBI_PIPE_ARGS g, plan, dW, ldw, dIp, dIz, dX, ldx, N, dY, ldy, dWorkspace, none, stream
    if (dt == LRBI_F16) {
        if (variant <= 1) return launch_pipe_t<F16Tag, 4, false, false>(LRBI_PIPE_ARGS);
        return launch_pipe_t<F16Tag, 4, true, false>(LRBI_PIPE_ARGS);
    }
    if (dt == LRBI_BF16) {
        if (variant <= 1) return launch_pipe_t<BF16Tag, 4, false, false>(LRBI_PIPE_ARGS);
        return launch_pipe_t<BF16Tag, 4, true, false>(LRBI_PIPE_ARGS);
    }
#undef LRBI_PIPE_ARGS
    return LRBI_ERR_DTYPE;
}

// true when the pipelined kernel serves the convolution form: aligned tile shapes, 64 channels or a multiple,
// the weight matrix's 9 * cin columns, offsets that fit the kernel's 32-bit per-lane byte offsets
bool pipe_conv_ok(const Geom &g, const ConvGeom &cg, int64_t batch, const void *dIz, const void *dAct, int64_t ldw)
{
    if ((g.c % 128) != 0 || (g.r % PIPE_BM) != 0 || g.k > FAST_MAX_K || g.ragged) return false;
    if (cg.cin <= 0 || cg.cin % 64 != 0 || cg.H <= 0 || cg.Wd <= 0 || batch <= 0) return false;
    if (g.n != (int64_t)9 * cg.cin) return false;
    if ((((uintptr_t)dAct | (uintptr_t)dIz) & 15) != 0) return false;
    if (ldw > (1 << 22)) return false;
    const int64_t act_bytes = batch * (cg.H + 2) * (int64_t)(cg.Wd + 2) * cg.cin * 2;
    if (act_bytes >= ((int64_t)1 << 32) || batch * cg.H * (int64_t)cg.Wd > 0x7FFFFF00) return false;
    const int64_t tiles = (int64_t)g.tile_rows * g.tile_cols;
    if (tiles * g.k * g.izw * 4 >= (int64_t)1 << 31 || tiles * g.r * g.ipw * 4 >= (int64_t)1 << 31) return false;
    return true;
}

// the convolution form (operands from L2: loads spread over the iteration); N = batch * H * Wd columns
int launch_pipe_conv(const Geom &g, const MfmaPlan &plan, lrbi_dtype dt, const ConvGeom &cg, const void *dW, int64_t ldw,
                     const uint32_t *dIp, const uint32_t *dIz, const void *dAct, int64_t N, void *dY, int64_t ldy,
                     void *dWorkspace, hipStream_t stream)
{
    if (dt == LRBI_F16)
        return launch_pipe_t<F16Tag, 4, true, true>(g, plan, dW, ldw, dIp, dIz, dAct, 0, N, dY, ldy, dWorkspace, cg, stream);
    if (dt == LRBI_BF16)
        return launch_pipe_t<BF16Tag, 4, true, true>(g, plan, dW, ldw, dIp, dIz, dAct, 0, N, dY, ldy, dWorkspace, cg, stream);
    return LRBI_ERR_DTYPE;
}

} // namespace lrbi
