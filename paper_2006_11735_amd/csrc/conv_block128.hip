// The identity bottleneck block of a network's second stage (1x1 conv from 512 to 128 channels, 3x3 conv, 1x1 conv back to
// 512 with the block input as skip operand, Section 4.1) as one kernel of small workgroups: four waves take a tile of at
// most 64 pixels through the three layers, and two workgroups share a compute unit, so that one's loads, barriers and
// vector work run beside the other's matrix instructions.
//
//   tile     TH x TW output pixels (at most 64, or 32 where there are few), patch (TH+2) x (TW+2) input pixels (at most 96, 64), copied to LDS once
//   phase 1  a = BReLU/requant(W1 x + b1) on the patch; patch pixels outside the image become zeros (the 3x3 layer's padding)
//   phase 2  b = BReLU/requant(W2 (*) a + b2) on the tile, tap = patch row offset; b replaces a
//   phase 3  y = epilogue(W3 b + b3, skip), 128 of the 512 channels at a time; the skip operand is the block input, in LDS
//            already, and every lane replaces the sixteen bytes it has merged by its result; y leaves in whole rows
//
// Each wave owns 32 of the 128 channels of a phase on all the tile's pixels, so a weight byte is needed by one wave of the
// workgroup only and goes from memory straight into that wave's registers, in packed order (which is the fragment order),
// four groups of two K steps ahead of its products and across the phases.  No K loop has a barrier.  LDS rows are padded by
// 16 bytes, as in conv_tri.hip.
//
// What bounds it: per tile 4.9 k clocks of matrix work, 4.4 k of the compute unit's path from L2 (279 KB of weights at 64
// bytes per clock), and 3.5 k of vector work in the last layer's epilogue, shared by the two workgroups of a compute unit.
#include "conv_common.h"

#include <type_traits>

namespace icnn {

constexpr int kB128Mid = 128, kB128Wide = 512;
// a tile of OG groups of 32 output pixel slots, patch rows in one group more
constexpr int kB128XP = kB128Wide + 16, kB128AP = kB128Mid + 16;
constexpr int b128_rows(int og) { return 32 * (og + 1); }
constexpr int b128_x_bytes(int og) { return (b128_rows(og) * (kB128XP / 16) + 63) / 64 * 1024; }

// HI: the three layers requantise as a product's high word (rq_fast) and the skip operand is rescaled likewise (g.sk), the last layer's
// epilogue dealt out between matrix instructions; else any 8-bit form.  BYTE: HI, and all of them to bytes (requant_fits_byte)
template <int OG, bool HI, bool BYTE>
__global__ __launch_bounds__(256, 2) void conv_block128_kernel(const uint8_t *x, const uint8_t *w1_packed, const unsigned hw, const unsigned shape, const int x_cs,
                                                               const int n_tiles, const int tiles_per_img, const unsigned mul_tpi, const int tiles_x,
                                                               const unsigned mul_tx, const unsigned shifts, const unsigned inv_pw, const BlockArgs ga,
                                                               const SkipMul sk, const ConvArgs a1, const ConvArgs a2, const ConvArgs a3)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    constexpr int MID = kB128Mid, C = kB128Wide, XP = kB128XP, AP = kB128AP;
    constexpr int PG = OG + 1, XBYTES = b128_x_bytes(OG);
    constexpr int NG = 4 + 9 + 4;                      // groups of two K steps: first layer, taps, chunks of the last layer

    // LDS: patch of x (in the end y on the tile's rows) | a on the patch, then b on the tile | biases [128] [128] [512]
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const abuf = lds + XBYTES;
    int32_t *const btab = (int32_t *)(abuf + b128_rows(OG) * AP);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    auto sync = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    struct { int H, W, TH, TW, PW, x_cs; unsigned inv_tw, inv_pw; } g = {(int)(hw & 0xffff), (int)(hw >> 16), (int)(shape & 0xff), (int)(shape >> 8 & 0xff),
                                                                        (int)(shape >> 16), x_cs, 0, inv_pw};
    // XCD x takes a contiguous range of tiles, so that the halos neighbouring patches share meet in one L2
    const int tile = (int)(blockIdx.x & 7) * ((n_tiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    const int n = fast_div_packed(tile, mul_tpi, shifts & 0xff, shifts >> 8 & 0xff);
    int y0, x0;
    {
        const int r = tile - n * tiles_per_img;
        const int ty = fast_div_packed(r, mul_tx, shifts >> 16 & 0xff, shifts >> 24);
        y0 = ty * g.TH;
        x0 = (r - ty * tiles_x) * g.TW;
    }

    // ---- weights: group k of this wave's chunk (its 32 channels), two K steps of two fragments, in slot k & 3 of the ring
    const uint8_t *const w1 = w1_packed + (size_t)wave * (8 * kChunkBytes);
    const uint8_t *const w2 = a2.wp + (size_t)wave * (18 * kChunkBytes);
    const uint8_t *const w3 = a3.wp + (size_t)wave * (2 * kChunkBytes);        // channels ch * 128 + ...: + ch * 8 steps
    v4i ring[4][4];
    const int lane16 = lane * 16;
    auto group_at = [&](auto k_tag) {
        constexpr int k = decltype(k_tag)::value;
        const uint8_t *const p = k < 4 ? w1 + k * (2 * kChunkBytes) : k < 13 ? w2 + (k - 4) * (2 * kChunkBytes) : w3 + (k - 13) * (8 * kChunkBytes);
        return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 2 * kChunkBytes, 0x00020000);
    };
    auto load_frag = [&](auto k_tag, auto f_tag) __attribute__((always_inline)) {
        constexpr int k = decltype(k_tag)::value, f = decltype(f_tag)::value;
        if constexpr (k < NG)
            ring[k & 3][f] = __builtin_amdgcn_raw_buffer_load_b128(group_at(k_tag), lane16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
    };

    // ---- prologue: patch, biases and the ring's first groups in flight together; what the patch and the ring need are leading arguments, which are in
    // registers when a wave starts, and the other arguments arrive meanwhile
    {
        const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);     // (every place inside the tensor lies below 2 GiB, OOB above)
        // 16-byte piece i of the patch region is piece i % 33 of row i / 33; the last one is padding
#pragma unroll 2
        for (int c = wave; c < XBYTES / 1024; c += 4) {
            const int i = c * 64 + lane;
            const int row = (int)(((unsigned)i * 63551u) >> 21), piece = i - row * 33;         // / 33, exact below 6000
            const int py = (int)(((unsigned)row * g.inv_pw) >> 16), px = row - py * g.PW;
            const int iy = y0 - 1 + py, ix = x0 - 1 + px;
            const bool ok = piece < 32 && py < g.TH + 2 && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
            const unsigned off = ok ? (unsigned)(((n * g.H + iy) * g.W + ix) * g.x_cs) + piece * 16 : OOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(lds + c * 1024), 16, off, 0, 0, 0);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        in_registers(a1.bias, a2.bias, a3.bias, a2.wp, a3.wp, a3.res_mode, a3.out, a3.out_cs, a3.out_co, ga.inv_tw);
        if constexpr (HI) in_registers(sk.k, sk.rnd, a1.mul_hi, a1.lo, a1.hi, a2.mul_hi, a2.lo, a2.hi, a3.mul_hi, a3.lo, a3.hi);
        g.inv_tw = ga.inv_tw;
        int bv[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int i = tid + q * 256;
            bv[q] = i < MID ? a1.bias[i] : (i < 2 * MID ? a2.bias[i - MID] : a3.bias[i - 2 * MID]);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        static_for<16>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value;
            load_frag(std::integral_constant<int, (i >> 2)>{}, std::integral_constant<int, (i & 3)>{});
        });
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 3; ++q) btab[tid + q * 256] = bv[q];
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(16);                           // this wave's copies of the patch have landed (the ring's loads are younger)
        sync();                                        // ... everybody's
    }

    const int co = wave * 32 + half * 16;              // this lane's sixteen channels inside the 128 of a phase
    auto finish = [&](const ConvArgs &a, const v16i &c) __attribute__((always_inline)) {
        if constexpr (HI) return epilogue_hi16<0, BYTE>(a, sk, c, v4i{0, 0, 0, 0});
        else return epilogue_bytes16<0>(a, c, v4i{0, 0, 0, 0});
    };
    // Group K of the ring on NJ pixel groups: row addresses ad, the group's 128 channels at `at` bytes into the row; behind every matrix
    // instruction one fragment of the half step (32 channels) AHEAD of it is read, at nad / nat beyond the group; behind every half step one
    // weight fragment of the group four on is fetched into the place of the one just used.
    auto group = [&](auto k_tag, auto &acc, auto &bf, const auto &ad, auto at_tag, const auto &nad, auto nat_tag) __attribute__((always_inline)) {
        constexpr int K = decltype(k_tag)::value, NJ = sizeof(acc) / sizeof(acc[0]), NB = sizeof(bf) / sizeof(bf[0]), AHEAD = NB - 1;
        constexpr int AT = decltype(at_tag)::value, NAT = decltype(nat_tag)::value;
        static_for<4>([&](auto h_tag) __attribute__((always_inline)) {
            constexpr int h = decltype(h_tag)::value, hn = h + AHEAD;
            static_for<NJ>([&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[K & 3][h], bf[h % NB][j], acc[j], 0, 0, 0);
                asm volatile("" : "+v"(acc[j]));       // here, not wherever the sums are needed
                __builtin_amdgcn_sched_barrier(0);
                bf[hn % NB][j] = *(const v4i *)(lds + (hn < 4 ? ad[j] + AT + hn * 32 : nad[j] + NAT + (hn - 4) * 32));
                if constexpr (j == NJ - 1) load_frag(std::integral_constant<int, K + 4>{}, h_tag);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    auto first_frags = [&](auto &bf, const auto &ad) __attribute__((always_inline)) {
        constexpr int NB = sizeof(bf) / sizeof(bf[0]), NJ = sizeof(bf[0]) / sizeof(bf[0][0]);
#pragma unroll
        for (int h = 0; h < NB - 1; ++h)
#pragma unroll
            for (int j = 0; j < NJ; ++j) bf[h][j] = *(const v4i *)(lds + ad[j] + h * 32);
    };

    // ---------------- phase 1: a = requant(W1 x + b1) on the patch
    {
        v16i acc[PG];
        v4i bf[2][PG];
        int ad[PG];
#pragma unroll
        for (int j = 0; j < PG; ++j) {
            ad[j] = (32 * j + col) * XP + half * 16;
            acc[j] = bias16(btab + co);
        }
        first_frags(bf, ad);
        static_for<4>([&](auto k_tag) __attribute__((always_inline)) {
            constexpr int k = decltype(k_tag)::value;
            group(k_tag, acc, bf, ad, std::integral_constant<int, k * 128>{}, ad, std::integral_constant<int, (k < 3 ? k + 1 : k) * 128>{});
        });
        mfma_drain(acc);
        static_for<PG>([&](auto j_tag) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value;
            const int row = 32 * j + col;
            const int py = (int)(((unsigned)row * g.inv_pw) >> 16), px = row - py * g.PW;
            const int iy = y0 - 1 + py, ix = x0 - 1 + px;
            v4i w = finish(a1, acc[j]);
            if (!((unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W)) w = v4i{0, 0, 0, 0};
            *(v4i *)(abuf + row * AP + co) = w;
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    sync();

    // ---------------- phase 2: b = requant(W2 (*) a + b2) on the tile's pixel slots
    int prow[OG];                                      // patch row of this lane's pixels q = 32 j + col (slots beyond the tile: of pixel 0)
    bool in[OG];
#pragma unroll
    for (int j = 0; j < OG; ++j) {
        const int q = 32 * j + col;
        in[j] = q < g.TH * g.TW;
        const int ty = in[j] ? (int)(((unsigned)q * g.inv_tw) >> 16) : 0;
        prow[j] = (ty + 1) * g.PW + (in[j] ? q - ty * g.TW : 0) + 1;
    }
    {
        v16i acc[OG];
        v4i bf[4][OG];
        int ad[OG], nad[OG];
#pragma unroll
        for (int j = 0; j < OG; ++j) {
            ad[j] = XBYTES + (prow[j] - g.PW - 1) * AP + half * 16;
            acc[j] = bias16(btab + MID + co);
        }
        first_frags(bf, ad);
        using Z = std::integral_constant<int, 0>;
        static_for<9>([&](auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value;
#pragma unroll
            for (int j = 0; j < OG; ++j) nad[j] = t == 8 ? ad[j] : ad[j] + (t % 3 == 2 ? (g.PW - 2) * AP : AP);
            group(std::integral_constant<int, 4 + t>{}, acc, bf, ad, Z{}, nad, Z{});
#pragma unroll
            for (int j = 0; j < OG; ++j) ad[j] = nad[j];
        });
        sync();                                        // every wave has its last fragments of a: b may overwrite it
        mfma_drain(acc);
        static_for<OG>([&](auto j_tag) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value;
            *(v4i *)(abuf + (32 * j + col) * AP + co) = finish(a2, acc[j]);        // slots beyond the tile hold values nobody stores
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    sync();

    // ---------------- phase 3: y = epilogue(W3 b + b3, skip), one pixel group of a chunk after the other
    {
        const bool has_res = a3.res_mode != 0;
        v16i c2[2];                                    // the group being multiplied, the one being finished
        v4i fr[4], r8[2];
        int w[4];
        const int ad0 = XBYTES + col * AP + half * 16;
#pragma unroll
        for (int h = 0; h < 3; ++h) fr[h] = *(const v4i *)(lds + ad0 + h * 32);
        static_for<4 * OG>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value, ch = i / OG, j = i % OG, K = 13 + ch, now = i & 1;
            constexpr int before = i == 0 ? 0 : (i - 1) % OG, next = (i + 1) % OG;                             // the pixel groups of the items beside it
            c2[now] = bias16(btab + 2 * MID + ch * MID + co);
            static_for<4>([&](auto h_tag) __attribute__((always_inline)) {
                constexpr int h = decltype(h_tag)::value, hn = h + 3;
                c2[now] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[K & 3][h], fr[h], c2[now], 0, 0, 0);
                asm volatile("" : "+v"(c2[now]));
                __builtin_amdgcn_sched_barrier(0);
                fr[hn & 3] = *(const v4i *)(lds + ad0 + (hn < 4 ? j : next) * (32 * AP) + (hn & 3) * 32);
                if constexpr (h == 1) r8[now] = *(const v4i *)(lds + prow[j] * XP + ch * MID + co);
                if constexpr (HI && i > 0) epilogue_hi_slice<1, 4 * h, 4, BYTE>(a3, sk, c2[now ^ 1], r8[now ^ 1], w);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (HI) {
                if constexpr (i > 0)
                    if (in[before]) *(v4i *)(lds + prow[before] * XP + ((i - 1) / OG) * MID + co) = v4i{w[0], w[1], w[2], w[3]};
                mfma_drain(c2[now]);
            } else {
                mfma_drain(c2[now]);
                const v4i o = has_res ? epilogue_bytes16<1>(a3, c2[now], r8[now]) : epilogue_bytes16<0>(a3, c2[now], r8[now]);
                if (in[j]) *(v4i *)(lds + prow[j] * XP + ch * MID + co) = o;
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (HI) {
            constexpr int last = (4 * OG - 1) & 1;
            const v4i o = epilogue_hi16<1, BYTE>(a3, sk, c2[last], r8[last]);
            if (in[OG - 1]) *(v4i *)(lds + prow[OG - 1] * XP + 3 * MID + co) = o;
        }
    }
    sync();                                            // y is complete

    // y leaves LDS two pixels' whole rows per store
#pragma unroll 4
    for (int c = wave; c < 16 * OG; c += 4) {
        const int q = 2 * c + half, piece = col * 16;
        const int ty = (int)(((unsigned)q * g.inv_tw) >> 16), tx = q - ty * g.TW;
        const int oy = y0 + ty, ox = x0 + tx;
        if (q < g.TH * g.TW && oy < g.H && ox < g.W)
            *(v4i *)((uint8_t *)a3.out + (size_t)((n * g.H + oy) * g.W + ox) * a3.out_cs + a3.out_co + piece) =
                *(const v4i *)(lds + ((ty + 1) * g.PW + tx + 1) * XP + piece);
    }
#endif
}

// ------------------------------------------------------------------ dispatch
constexpr long long kB128SmallTiles = 256;

// 512 -> 128 -> 128 -> 512 channels, an 8-bit output, the block input itself as skip operand (unsigned 8-bit, joined before requantisation
// with a rescale that fits 32 bits) or none
bool conv_block128_takes(const BlockArgs &g, const ConvArgs &a1, const ConvArgs &a3)
{
    if (a1.Cin != kB128Wide || a1.Cout != kB128Mid || a3.Cout != kB128Wide || a3.pc) return false;
    if (a3.out_mode == 3 || !a3.epi_vec || a3.epi_mode / 4 == 2) return false;
    if (g.H > 0xffff || g.W > 0xffff || g.x_bytes >= 0x7fffff00u) return false;
    return a3.res_mode == 0 || ((const uint8_t *)a3.res == g.x && a3.res_cs == g.x_cs);
}

hipError_t launch_conv_block128(const BlockArgs &g, const ConvArgs &a1, const ConvArgs &a2, const ConvArgs &a3, hipStream_t st)
{
    if (!conv_block128_takes(g, a1, a3)) return hipErrorInvalidValue;
    // Tiles of 32 pixels where there is a compute unit for each: a workgroup's own time is what a launch takes then.  50 layers, us, 64 / 32 pixels: one image (28 tiles of 32
    // pixels) 169.3 / 160.8, four 205.1 / 198.9, nine (252) 238.1 / 231.0, 12 (336) 275.8 / 277.4, 32 384.9 / 397.2.
    BlockArgs gx = g;
    long long tiles = 0;
    const auto tile = [&](int og) {
        gx = g;
        if (!conv_block_tile(g.H, g.W, 32 * og, b128_rows(og), gx)) return false;
        tiles = (long long)gx.tiles_per_img * g.N;
        return true;
    };
    int og = 1;
    if (g_tuning.block128_tile ? g_tuning.block128_tile == 2 || !tile(1) : !tile(1) || tiles > kB128SmallTiles) {
        og = 2;
        if (!tile(2)) return hipErrorInvalidValue;
    }
    if (tiles > 0x7fffffffLL - 8) return hipErrorInvalidValue;
    gx.n_tiles = (int)tiles;
    gx.per_xcd = (int)((tiles + 7) / 8);
    const size_t lds_bytes = b128_x_bytes(og) + b128_rows(og) * kB128AP + (2 * kB128Mid + kB128Wide) * 4;
    const SkipMul sk = a3.res_mode ? make_skip_mul(a3.res_mul, a3.res_shift) : SkipMul{0, 0, 0};     // (without an operand: adds zero)
    auto go = [&](auto kernel) -> hipError_t {
        const hipError_t e = allow_large_lds((const void *)kernel);
        if (e != hipSuccess) return e;
        const FastDiv tpi = make_fast_div((unsigned)gx.tiles_per_img), tx = make_fast_div((unsigned)gx.tiles_x);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * gx.per_xcd)), dim3(256), lds_bytes, st, g.x, a1.wp, (unsigned)gx.H | (unsigned)gx.W << 16,
                           (unsigned)gx.TH | (unsigned)gx.TW << 8 | (unsigned)gx.PW << 16, gx.x_cs, gx.n_tiles, gx.tiles_per_img, tpi.mul, gx.tiles_x, tx.mul,
                           tpi.s1 | tpi.s2 << 8 | tx.s1 << 16 | tx.s2 << 24, gx.inv_pw, gx, sk, a1, a2, a3);
        return hipGetLastError();
    };
    const bool hi = a1.rq_fast && a2.rq_fast && a3.rq_fast && (a3.res_mode == 0 || sk.ok) && !g_tuning.block_any_form;
    const bool byte = hi && requant_fits_byte(a1) && requant_fits_byte(a2) && requant_fits_byte(a3);
    auto by_form = [&](auto og_tag) {
        constexpr int OG = decltype(og_tag)::value;
        return byte ? go(conv_block128_kernel<OG, true, true>) : hi ? go(conv_block128_kernel<OG, true, false>) : go(conv_block128_kernel<OG, false, false>);
    };
    return og == 1 ? by_form(std::integral_constant<int, 1>{}) : by_form(std::integral_constant<int, 2>{});
}

}  // namespace icnn
