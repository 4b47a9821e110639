// The identity bottleneck block of a network's first stage (1x1 conv from 256 to 64 channels, 3x3 conv, 1x1 conv back to 256
// with the block input as skip operand, Section 4.1) as one kernel of small workgroups: four waves take tiles of at most 64 (on few pictures 32)
// pixels through the three layers, and two workgroups share a compute unit, so that one's loads and barriers run beside the
// other's arithmetic.
//
//   tile     TH x TW output pixels (at most 64 or 32), patch (TH+2) x (TW+2) input pixels (at most 96 or 64); two patch buffers, the next
//            tile's patch is copied global -> LDS while this tile runs
//   phase 1  a = BReLU/requant(W1 x + b1) on the patch: six (chunk, pixel group) items over four waves; patch pixels
//            outside the image become zeros (the 3x3 layer's padding)
//   phase 2  b = BReLU/requant(W2 (*) a + b2) on the tile, one item per wave; b replaces a
//   phase 3  y = epilogue(W3 b + b3, skip): two of the eight chunks of 32 channels per wave; the skip operand is the block input,
//            in LDS already, and every lane replaces the sixteen bytes it has merged by its result; y leaves in whole rows
//
// A wave's share of the three layers' weights is 30 fragments = 120 registers, loaded once for the workgroup's whole life.
//
// What bounds it: vector work.  The last layer's epilogue is 368 instructions per wave and tile, the other two 132, and what
// is left for positions has been taken out of the tile: where a patch's rows lie in memory is worked out by one thread per
// row into a table in LDS, where a copy's and a store's pieces lie in a tile once per workgroup.  64 x 56 x 56 pixels: 46 us with
// eight waves on tiles of 128 pixels (conv_block64.hip), 46 with three workgroups per compute unit that fetch their weights per
// tile (9 of a tile's 19 k clocks), 41 here, 39 to bytes.  Biases and weights are requested before anything else, from arguments that the hardware puts into registers:
// behind the tile's arguments and the first patch they came some 1500 clocks later (7.2 -> 6.9 us at one picture, 42.6 -> 41.9 at 64).
//
// PROJ: the block that opens the stage (64 input channels, the skip operand a projection of them, "after convolution").  Its last layer's sums
// pass through vector instructions twice, once at the projection's ratio; an item's four steps (projection, rescale, products, epilogue) are
// dealt out so that another item's products are made beside them.  28 weight fragments a wave; y has a region of LDS of its own.
// 56 x 56 pixels, 1 / 9 / 64 pictures, launches behind one another: 8.4 / 9.3 / 38.2 us with eight waves on tiles of 128 pixels (conv_block64.hip), 5.8 / 8.2 / 33.5 here, 4.65 at
// one picture in tiles of 32 pixels (a trace of the network, where each has cold weights, gives 1 to 5 us more to either).
#include "conv_common.h"

#include <algorithm>
#include <type_traits>

namespace icnn {

constexpr int kB64sMid = 64, kB64sWide = 256;
constexpr int b64s_rows(int og) { return og == 2 ? 96 : 64; }         // patch rows of a tile of 32 og output pixel slots
constexpr int kB64sYP = kB64sWide + 16, kB64sAP = kB64sMid + 16;      // row pitches: padded as in conv_tri.hip
constexpr int b64s_patch_bytes(int og, bool proj) { return (b64s_rows(og) * ((proj ? kB64sAP : kB64sYP) / 16) + 63) / 64 * 1024; }
constexpr int b64s_lds_bytes(int og, bool proj)
{
    return 2 * b64s_patch_bytes(og, proj) + b64s_rows(og) * kB64sAP + (2 * kB64sMid + (proj ? 2 : 1) * kB64sWide) * 4 + 2 * 128 * 4 + (proj ? 32 * og * kB64sYP : 0);
}

// The three layers requantise as a product's high word (rq_fast) and the skip operand is rescaled likewise (sk).  BYTE: all of them to bytes (requant_fits_byte).
// PROJ: the block that opens the stage: 64 input channels, the skip operand a projection pj of the block input whose rescale shifts by less than 32
// OG: groups of 32 output pixels of a tile
template <int OG, bool PROJ, bool BYTE>
__global__ __launch_bounds__(256, 2) void conv_block64s_kernel(const uint8_t *const x, const uint8_t *const wp1, const uint8_t *const wp2,
                                                               const uint8_t *const wp3, const int32_t *const bias1, const int32_t *const bias2,
                                                               const int32_t *const bias3, const BlockArgs g, const SkipMul sk, const ConvArgs a1,
                                                               const ConvArgs a2, const ConvArgs a3, const ProjArgs pj)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    constexpr int MID = kB64sMid, C = kB64sWide, CIN = PROJ ? MID : C, XP = CIN + 16, YP = kB64sYP, AP = kB64sAP;
    constexpr int XBYTES = b64s_patch_bytes(OG, PROJ), ROWS = b64s_rows(OG);

    // LDS: two patches of x (in the end y on the tile's rows) | a on the patch, then b on the tile | biases [64] [64] [256] (PROJ: [256] of the
    // projection) | two tables of patch rows | PROJ: y on the tile, which has no room in a patch of 64 channels
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const abuf = lds + 2 * XBYTES;
    int32_t *const btab = (int32_t *)(abuf + ROWS * AP);
    unsigned *const rtab = (unsigned *)(btab + 2 * MID + (PROJ ? 2 : 1) * C);
    [[maybe_unused]] uint8_t *const ybuf = (uint8_t *)(rtab + 2 * 128);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    // ---- biases and this wave's weights, for the workgroup's whole life: requested first, from arguments that arrive in registers
    const int c12 = wave & 1, pg = (wave >> 1) ^ (int)((blockIdx.x >> 8) & 1);          // chunk of layers 1 and 2; pixel group in phase 2 and first one in
                                                       // phase 1, where group 0's waves take a second one (the other waves of the second workgroup on a compute unit)
    v4i w1[CIN / 32], w2[18], w3[2][2];
    [[maybe_unused]] v4i wq[2][2];                     // the projection's
    int bv[2];
    [[maybe_unused]] int bq;
    static_assert(MID == 64, "a wave's biases are one layer's");
    bv[0] = (wave == 0 ? bias1 : wave == 1 ? bias2 : bias3 + 64 * (wave - 2))[lane];
    bv[1] = bias3[min(tid + 2 * MID, C - 1)];
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    {
        const int l16 = lane * 16;
        const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc((void *)(wp1 + (size_t)c12 * (CIN / 64) * kChunkBytes), 0, CIN / 64 * kChunkBytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc((void *)(wp2 + (size_t)c12 * 9 * kChunkBytes), 0, 9 * kChunkBytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t r3 = __builtin_amdgcn_make_buffer_rsrc((void *)(wp3 + (size_t)wave * 2 * kChunkBytes), 0, 2 * kChunkBytes, 0x00020000);
#pragma unroll
        for (int f = 0; f < CIN / 32; ++f) w1[f] = __builtin_amdgcn_raw_buffer_load_b128(r1, l16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
#pragma unroll
        for (int f = 0; f < 18; ++f) w2[f] = __builtin_amdgcn_raw_buffer_load_b128(r2, l16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
#pragma unroll
        for (int f = 0; f < 4; ++f) w3[f >> 1][f & 1] = __builtin_amdgcn_raw_buffer_load_b128(r3, l16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (PROJ) {                              // (their arguments come late, with the tile's)
        bq = pj.bias[tid];
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void *)(pj.wp + (size_t)wave * 2 * kChunkBytes), 0, 2 * kChunkBytes, 0x00020000);
#pragma unroll
        for (int f = 0; f < 4; ++f) wq[f >> 1][f & 1] = __builtin_amdgcn_raw_buffer_load_b128(rq, lane * 16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
    }
    in_registers(g.per_xcd, g.n_tiles, g.tiles_per_img, g.tiles_x, g.TH, g.TW, g.PW, g.inv_pw, g.inv_tw, g.H, g.W, g.x_cs, g.x_bytes, g.k1, a3.out_cs, a3.out_co, a3.out);

    auto sync = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // XCD-contiguous walk, as in the other fused kernels
    auto tile_of = [&](int v) { return (v & 7) * g.per_xcd + (v >> 3); };
    auto valid = [&](int v) { return (v >> 3) < g.per_xcd && tile_of(v) < g.n_tiles; };
    auto tile_origin = [&](int v, int &n, int &y0, int &x0) {
        const int t = tile_of(v);
        n = t / g.tiles_per_img;
        const int r = t - n * g.tiles_per_img;
        const int ty = r / g.tiles_x;
        y0 = ty * g.TH;
        x0 = (r - ty * g.tiles_x) * g.TW;
    };
    if (!valid(blockIdx.x)) return;

    // ---- the patch of a tile.  Table: the offset of every row in memory, one thread per row (one more stands for the padding behind the last).
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, g.x_bytes, 0x00020000);
    auto write_rows = [&](int v, int b) __attribute__((always_inline)) {
        if (tid <= ROWS) {
            int n, y0, x0;
            tile_origin(v, n, y0, x0);
            const int py = (int)(((unsigned)tid * g.inv_pw) >> 16), px = tid - py * g.PW;
            const int iy = y0 - 1 + py, ix = x0 - 1 + px;
            const bool ok = py < g.TH + 2 && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
            rtab[b * 128 + tid] = ok ? (unsigned)(((n * g.H + iy) * g.W + ix) * g.x_cs) : OOB;
        }
    };
    // Copies of 1 KiB: 16-byte piece i of the region is piece i % 17 (PROJ: 5) of row i / 17; the last one is padding, which takes any bytes (an offset
    // of 1 GiB beside the row: inside the tensor or read as zeros).
    constexpr int COPIES = XBYTES / 1024, CPW = (COPIES + 3) / 4;
    int c_row[CPW], c_off[CPW];                        // of this lane's piece of copy wave + 4 q: table entry, offset in the row
#pragma unroll
    for (int q = 0; q < CPW; ++q) {
        const int i = (wave + 4 * q) * 64 + lane;
        const int row = (int)(((unsigned)i * (PROJ ? 209716u : 61681u)) >> 20), piece = i - row * (XP / 16);       // / 17, / 5: exact below 2^12
        c_row[q] = min(row, ROWS);
        c_off[q] = piece < CIN / 16 ? piece * 16 : 0x40000000;
    }
    auto issue_patch = [&](int b) __attribute__((always_inline)) {
        unsigned off[CPW];
#pragma unroll
        for (int q = 0; q < CPW; ++q) off[q] = rtab[b * 128 + c_row[q]] + (unsigned)c_off[q];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < CPW; ++q)
            if (wave + 4 * q < COPIES)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(lds + b * XBYTES + (wave + 4 * q) * 1024), 16,
                                                         off[q], 0, 0, 0);
    };

    write_rows(blockIdx.x, 0);
    if (valid(blockIdx.x + (int)gridDim.x)) write_rows(blockIdx.x + (int)gridDim.x, 1);
    sync();
    issue_patch(0);
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (tid + q * 256 < 2 * MID + C) btab[tid + q * 256] = bv[q];

    if constexpr (PROJ) btab[2 * MID + C + tid] = bq;

    // patch row of this lane's pixels q = 32 j + col (slots beyond the tile: of pixel 0)
    int prow[OG];
    bool in[OG];
#pragma unroll
    for (int j = 0; j < OG; ++j) {
        const int q = 32 * j + col;
        in[j] = q < g.TH * g.TW;
        const int ty = in[j] ? (int)(((unsigned)q * g.inv_tw) >> 16) : 0;
        prow[j] = (ty + 1) * g.PW + (in[j] ? q - ty * g.TW : 0) + 1;
    }
    // where this lane's pieces of y lie: four pixels' whole rows per store (slots beyond the tile: nowhere, whatever the picture's height)
    constexpr int STORES = 2 * OG;
    int s_lds[STORES];
    unsigned s_out[STORES];
    short s_y[STORES], s_x[STORES];
#pragma unroll
    for (int c = 0; c < STORES; ++c) {
        const int q = (wave + 4 * c) * 4 + (lane >> 4);
        const bool slot = q < g.TH * g.TW;
        const int ty = slot ? (int)(((unsigned)q * g.inv_tw) >> 16) : 0, tx = slot ? q - ty * g.TW : 0;
        s_lds[c] = (PROJ ? q : (ty + 1) * g.PW + tx + 1) * YP + (lane & 15) * 16;
        s_y[c] = (short)ty;
        s_x[c] = (short)tx;
        s_out[c] = slot ? (unsigned)((ty * g.W + tx) * a3.out_cs + (lane & 15) * 16) : OOB;
    }

    int buf = 0;
    for (int v = blockIdx.x; valid(v); v += gridDim.x, buf ^= 1) {
    int n, y0, x0;
    tile_origin(v, n, y0, x0);
    uint8_t *const xb = lds + buf * XBYTES;
    asm volatile("" ::: "memory");
    if (v == (int)blockIdx.x) ICNN_WAIT_VMCNT(0);      // this wave's copies of the patch have landed (the weights, requested before them, too);
    else ICNN_WAIT_VMCNT(STORES);                      // younger are the last tile's stores
    sync();                                            // ... everybody's; and nobody reads the last tile's y or b any more
    {
        const int v1 = v + (int)gridDim.x, v2 = v1 + (int)gridDim.x;
        if (valid(v1)) issue_patch(buf ^ 1);
        if (valid(v2)) write_rows(v2, buf);            // (this tile's table has been used up)
    }

    // ---------------- phase 1: a = requant(W1 x + b1) on patch rows 32 pg .. + 32, and on the last 32 for the waves of group 0
#pragma unroll
    for (int rep = 0; rep < OG; ++rep) {
        if (rep && pg) break;
        const int row = 32 * (rep ? 2 : pg) + col;
        const uint8_t *const xr = xb + row * XP + half * 16;
        constexpr int NF = CIN / 32, NB = NF < 4 ? NF : 4;
        v4i bf[NB];
#pragma unroll
        for (int h = 0; h < NB; ++h) bf[h] = *(const v4i *)(xr + h * 32);
        v16i acc = bias16(btab + c12 * 32 + half * 16);
        __builtin_amdgcn_sched_barrier(0);
        static_for<NF>([&](auto h_tag) __attribute__((always_inline)) {
            constexpr int h = decltype(h_tag)::value;
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w1[h], bf[h % NB], acc, 0, 0, 0);
            asm volatile("" : "+v"(acc));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (h + NB < NF) bf[h % NB] = *(const v4i *)(xr + (h + NB) * 32);
            __builtin_amdgcn_sched_barrier(0);
        });
        mfma_drain(acc);
        const int py = (int)(((unsigned)row * g.inv_pw) >> 16), px = row - py * g.PW;
        const int iy = y0 - 1 + py, ix = x0 - 1 + px;
        v4i w = epilogue_hi16<0, BYTE>(a1, sk, acc, v4i{0, 0, 0, 0});
        if (!((unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W)) w = v4i{0, 0, 0, 0};
        *(v4i *)(abuf + row * AP + c12 * 32 + half * 16) = w;
        __builtin_amdgcn_sched_barrier(0);
    }
    sync();

    // ---------------- phase 2: b = requant(W2 (*) a + b2) on output slots 32 pg .. + 32 (one group of pixels: two of the waves)
    const bool has_group = OG == 2 || !pg;
    v16i acc2;
    if (has_group) {
        const uint8_t *const ar = abuf + (pg ? prow[OG - 1] : prow[0]) * AP + half * 16;
        v4i bf[6];
        auto frag = [&](auto f_tag) __attribute__((always_inline)) {
            constexpr int f = decltype(f_tag)::value, t = f >> 1;
            bf[f % 6] = *(const v4i *)(ar + ((t / 3 - 1) * g.PW + t % 3 - 1) * AP + (f & 1) * 32);
        };
        static_for<6>(frag);
        acc2 = bias16(btab + MID + c12 * 32 + half * 16);
        __builtin_amdgcn_sched_barrier(0);
        static_for<18>([&](auto f_tag) __attribute__((always_inline)) {
            constexpr int f = decltype(f_tag)::value;
            acc2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(w2[f], bf[f % 6], acc2, 0, 0, 0);
            asm volatile("" : "+v"(acc2));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (f + 6 < 18) frag(std::integral_constant<int, f + 6>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    sync();                                            // every wave has its last fragments of a: b may overwrite it
    if (has_group) {
        mfma_drain(acc2);
        *(v4i *)(abuf + (32 * pg + col) * AP + c12 * 32 + half * 16) = epilogue_hi16<0, BYTE>(a2, sk, acc2, v4i{0, 0, 0, 0});   // slots beyond the tile hold values nobody stores
    }
    sync();

    // ---------------- phase 3: y = epilogue(W3 b + b3, skip) on chunks 2 wave and 2 wave + 1
    {
        v4i bf[OG][2];
#pragma unroll
        for (int j = 0; j < OG; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) bf[j][h] = *(const v4i *)(abuf + (32 * j + col) * AP + half * 16 + h * 32);
        v16i acc[2];
        if constexpr (PROJ) {
            v4i xf[OG][2];                             // the pixels' own rows of the patch
#pragma unroll
            for (int j = 0; j < OG; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) xf[j][h] = *(const v4i *)(xb + prow[j] * XP + half * 16 + h * 32);
            // item i: chunk i / OG, pixel group i % OG, in four steps; while one item's sums are in vector instructions, another's products are made
            auto project = [&](auto i_tag) __attribute__((always_inline)) {
                constexpr int c = decltype(i_tag)::value / OG, j = decltype(i_tag)::value % OG, k = decltype(i_tag)::value & 1;
                acc[k] = bias16(btab + 2 * MID + C + (2 * wave + c) * 32 + half * 16);
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wq[c][h], xf[j][h], acc[k], 0, 0, 0);
                asm volatile("" : "+v"(acc[k]));
                __builtin_amdgcn_sched_barrier(0);
            };
            // the projection's sum at the main path's ratio, on the last layer's bias; that layer's products on top
            auto rescale = [&](auto i_tag) __attribute__((always_inline)) {
                constexpr int c = decltype(i_tag)::value / OG, j = decltype(i_tag)::value % OG, k = decltype(i_tag)::value & 1;
                const v16i b3 = bias16(btab + 2 * MID + (2 * wave + c) * 32 + half * 16);
                mfma_drain(acc[k]);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[k][r] = rsr64_low((int64_t)acc[k][r] * pj.res_mul, pj.res_shift) + b3[r];
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w3[c][h], bf[j][h], acc[k], 0, 0, 0);
                asm volatile("" : "+v"(acc[k]));
                __builtin_amdgcn_sched_barrier(0);
            };
            auto finish = [&](auto i_tag) __attribute__((always_inline)) {
                constexpr int c = decltype(i_tag)::value / OG, j = decltype(i_tag)::value % OG, k = decltype(i_tag)::value & 1;
                mfma_drain(acc[k]);
                *(v4i *)(ybuf + (32 * j + col) * YP + (2 * wave + c) * 32 + half * 16) = epilogue_hi16<0, BYTE>(a3, sk, acc[k], v4i{0, 0, 0, 0});
                __builtin_amdgcn_sched_barrier(0);
            };
            constexpr std::integral_constant<int, 0> i0{};
            constexpr std::integral_constant<int, 1> i1{};
            constexpr std::integral_constant<int, 2> i2{};
            constexpr std::integral_constant<int, 3> i3{};
            project(i0), project(i1);
            rescale(i0), rescale(i1);
            finish(i0);
            if constexpr (OG == 2) project(i2);
            finish(i1);
            if constexpr (OG == 2) {
                project(i3);
                rescale(i2), rescale(i3);
                finish(i2), finish(i3);
            }
        } else {
        v4i r8[2];
        // item i: chunk i / OG, pixel group i % OG; its products are issued before the epilogue of the item before it
        auto multiply = [&](auto i_tag) __attribute__((always_inline)) {
            constexpr int c = decltype(i_tag)::value / OG, j = decltype(i_tag)::value % OG, k = decltype(i_tag)::value & 1;
            acc[k] = bias16(btab + 2 * MID + (2 * wave + c) * 32 + half * 16);
            r8[k] = *(const v4i *)(xb + prow[j] * XP + (2 * wave + c) * 32 + half * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w3[c][h], bf[j][h], acc[k], 0, 0, 0);
            asm volatile("" : "+v"(acc[k]));
            __builtin_amdgcn_sched_barrier(0);
        };
        multiply(std::integral_constant<int, 0>{});
        static_for<2 * OG>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value, c = i / OG, j = i % OG, k = i & 1;
            if constexpr (i + 1 < 2 * OG) multiply(std::integral_constant<int, i + 1>{});
            mfma_drain(acc[k]);
            const v4i o = epilogue_hi16<1, BYTE>(a3, sk, acc[k], r8[k]);
            if (in[j]) *(v4i *)(xb + prow[j] * XP + (2 * wave + c) * 32 + half * 16) = o;
            __builtin_amdgcn_sched_barrier(0);
        });
        }
    }
    sync();                                            // y is complete

    // y leaves LDS
    {
        // (through a descriptor of the tile's own: pieces outside the image are dropped there, so the stores are always as many)
        const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
            (uint8_t *)a3.out + (size_t)(unsigned)((n * g.H + y0) * g.W + x0) * a3.out_cs + a3.out_co, 0, 0x7fffff00, 0x00020000);
#pragma unroll
        for (int c = 0; c < STORES; ++c) {
            const v4i o = *(const v4i *)((PROJ ? ybuf : xb) + s_lds[c]);
            const bool ok = y0 + s_y[c] < g.H && x0 + s_x[c] < g.W;
            __builtin_amdgcn_raw_buffer_store_b128(o, rs_y, ok ? s_out[c] : OOB, 0, 0);
        }
    }
    }
#endif
}

// ------------------------------------------------------------------ dispatch
// Tiles of 32 pixels where each has a compute unit for itself: a launch then takes what one tile takes.  And where tiles of 64 would come two to a unit: 32 pixels on two
// workgroups to a unit, and up to half of them with a second tile.  56 x 56 pixels, us in tiles of 32 / 64, identity block (opening block 0.3 to 0.5 less):
// 1, 2 pictures 4.95 / 6.15, 5.07 / 6.22; 3, 4 (tiles of 64 have a unit each) 6.47 / 6.36, 6.58 / 6.50; 5, 6, 7 6.77 / 8.10, 7.59 / 8.25, 7.79 / 8.40; 8, 9
// 9.72 / 8.54, 9.99 / 8.81.
constexpr long long kB64sUnits = 256;
static bool block64s_small(long long tiles32, long long tiles64)
{
    return tiles32 <= kB64sUnits || (tiles64 > kB64sUnits && tiles32 <= 3 * kB64sUnits);
}

// A tile of 32 og pixels, in t, whose stores can be made: their offsets from the tile's first pixel are 32 bits, up to the descriptor's 0x7fffff00 bytes
constexpr long long kB64sStores = 0x7fffff00LL - kB64sWide;
static bool block64s_tile(const BlockArgs &g, const ConvArgs &a3, int og, BlockArgs &t)
{
    t = g;
    return conv_block_tile(g.H, g.W, 32 * og, b64s_rows(og), t) && ((t.TH - 1LL) * g.W + t.TW - 1) * a3.out_cs <= kB64sStores;
}
// (A tile has at most 64 rows: it is searched for only where that many could pass the limit, at a pitch of 256 pictures from 133000 columns on.)
static bool block64s_stores_fit(const BlockArgs &g, const ConvArgs &a3)
{
    BlockArgs t;
    return (63LL * g.W + 64) * a3.out_cs <= kB64sStores || block64s_tile(g, a3, 2, t);
}

// 256 -> 64 -> 64 -> 256 channels, per-layer requantisation, an 8-bit output, the block input itself as skip operand (unsigned 8-bit, joined
// before requantisation) or none
bool conv_block64s_takes(const BlockArgs &g, const ConvArgs &a1, const ConvArgs &a2, const ConvArgs &a3)
{
    if (a1.Cin != kB64sWide || a1.Cout != kB64sMid || a3.Cout != kB64sWide || a3.pc) return false;
    if (a3.out_mode == 3 || !a3.epi_vec || a3.epi_mode / 4 == 2 || !a1.rq_fast || !a2.rq_fast || !a3.rq_fast) return false;
    if (!block64s_stores_fit(g, a3)) return false;
    if (a3.res_mode == 0) return true;
    return (const uint8_t *)a3.res == g.x && a3.res_cs == g.x_cs && make_skip_mul(a3.res_mul, a3.res_shift).ok;
}

// The block that opens the stage, 64 -> 64 -> 64 -> 256 channels with a 64 -> 256 projection, per-layer requantisation and an 8-bit output: every such block
// whose arithmetic the kernel has, since it is the faster one at any number of pictures (times above).  Shifts of 32 and more: a word of the product
// alone holds them, in another instruction.
bool conv_block64s_proj_takes(const BlockArgs &g, const ConvArgs &a1, const ConvArgs &a2, const ConvArgs &a3, const ProjArgs &pj)
{
    return conv_block64_proj_takes(a1, a3, pj) && a1.rq_fast && a2.rq_fast && a3.rq_fast && !a3.pc && pj.res_shift < 32 && block64s_stores_fit(g, a3);
}

// pj: the projection of an opening block, else null
hipError_t launch_conv_block64s(const BlockArgs &g, const ConvArgs &a1, const ConvArgs &a2, const ConvArgs &a3, const ProjArgs *pj, hipStream_t st)
{
    if (!(pj ? conv_block64s_proj_takes(g, a1, a2, a3, *pj) : conv_block64s_takes(g, a1, a2, a3))) return hipErrorInvalidValue;
    // (a search takes 0.1 to 0.2 us of the host: as few as the choice needs)
    BlockArgs gx, large;
    const auto tiles_of = [&](int og, BlockArgs &t) { return block64s_tile(g, a3, og, t) ? (long long)t.tiles_per_img * g.N : -1; };
    const int forced = g_tuning.block64s_tile;
    long long tiles = forced == 2 ? -1 : tiles_of(1, gx);
    int og = 1;
    if (tiles < 0 || (!forced && tiles > kB64sUnits)) {
        const long long tiles64 = tiles_of(2, large);
        if (tiles < 0 || !block64s_small(tiles, tiles64)) og = 2, gx = large, tiles = tiles64;
    }
    if (tiles < 0 || tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
    gx.n_tiles = (int)tiles;
    gx.per_xcd = (int)((tiles + 7) / 8);
    static_assert(b64s_lds_bytes(2, false) <= 64 * 1024 && b64s_lds_bytes(2, true) <= 64 * 1024, "no permission needed");
    const SkipMul sk = a3.res_mode ? make_skip_mul(a3.res_mul, a3.res_shift) : SkipMul{0, 0, 0};     // (without an operand: adds zero)
    const auto go = [&](auto og_tag, auto byte_tag) {
        constexpr int OG = decltype(og_tag)::value;
        constexpr bool BYTE = decltype(byte_tag)::value;
        hipLaunchKernelGGL((pj ? conv_block64s_kernel<OG, true, BYTE> : conv_block64s_kernel<OG, false, BYTE>), dim3((unsigned)std::min(8 * gx.per_xcd, 512)), dim3(256),
                           b64s_lds_bytes(OG, pj != nullptr), st, gx.x, a1.wp, a2.wp, a3.wp, a1.bias, a2.bias, a3.bias, gx, sk, a1, a2, a3, pj ? *pj : ProjArgs{});
    };
    const bool byte = requant_fits_byte(a1) && requant_fits_byte(a2) && requant_fits_byte(a3);
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    if (og == 1) byte ? go(one, std::true_type{}) : go(one, std::false_type{});
    else byte ? go(two, std::true_type{}) : go(two, std::false_type{});
    return hipGetLastError();
}

}  // namespace icnn
