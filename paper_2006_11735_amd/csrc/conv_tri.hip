// The second half of one bottleneck block and the first layer of the next as ONE kernel: 3x3 convolution (256 -> 256
// channels), 1x1 convolution (256 -> 1024, skip operand merged in its epilogue, Section 4.1) and the 1x1 convolution
// (1024 -> 256) that opens the next block and reads nothing but that result.  Cut this way, between a block's first two
// layers instead of between blocks, nothing is computed twice: the only neighbours' values a tile needs are the 3x3
// layer's input, which is in memory, and the two pointwise layers stay on the tile.
//
//   tile     PX consecutive pixels of the flattened N*H*W axis (32, 64, 96 or 112); patch: these and the W + 1 pixels
//            before and behind them, so that tap (kh, kw) of a pixel is the patch row (kh - 1) * W + kw - 1 away; a tap
//            beyond the image's edge reads a row of zeros instead, chosen by a mask of nine bits per pixel
//   phase 1  b = BReLU/requant(W2 (*) t + b2) on the tile, from the patch in LDS; b replaces the patch
//   phase 2  y = epilogue(W3 b + b3, skip), 256 of the 1024 channels at a time; the skip operand's tile was copied to LDS
//            meanwhile and every lane replaces the sixteen bytes it has merged by its result
//   phase 3  z = BReLU/requant(W1 y + b1) from y in LDS, while y goes to memory in whole rows
//
// Every wave owns 32 of the 256 output channels of a phase, on all the tile's pixels, so a weight byte is needed by one
// wave of the workgroup only and goes from memory straight into that wave's registers, in packed order (which is the
// fragment order), eight K steps ahead of its products and across the phases.  No K loop has a barrier.  LDS rows are
// padded by 16 bytes: consecutive rows start one bank group apart, so the fragment reads of any 16 consecutive pixels are
// free of conflicts and a row's channels are constant offsets from one address.
#include "conv_common.h"

#include <algorithm>
#include <type_traits>

namespace icnn {

// The kernel's arguments in their order (late_argument): a parameter more, or of another type, does not compile (tri_members)
struct TriKernelArgs {
    const uint8_t *x, *w2;
    const int32_t *bias2, *bias3, *bias1;
    int M, in_cs;
    unsigned shape, tiles;
    int grid;
    const uint8_t *w3, *w1;
    TriArgs ga;
    ConvArgs a2, a3, a1;
};

// FORM: 1 all layers requantise as a product's high word (rq_fast), the skip operand rescaled likewise (g.sk), the block's last layer between matrix instructions; 3 as 1, all
// layers to bytes (requant_fits_byte); 0 any form, chosen at run time; 2 per output channel.  NEXT: the next block's first layer is included.
template <int NP, bool NEXT, int FORM>                 // NP: pixel groups of 32 (the fourth one half used)
__global__ __launch_bounds__(512, 2) void conv_tri_kernel(const uint8_t *x, const uint8_t *w2_packed, const int32_t *bias2, const int32_t *bias3, const int32_t *bias1,
                                                          const int M, const int in_cs, const unsigned shape, const unsigned tiles, const int grid,
                                                          const uint8_t *w3_packed, const uint8_t *w1_packed, const TriArgs, const ConvArgs, const ConvArgs, const ConvArgs)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    constexpr int MID = kTriMid, C = kTriWide, PX = tri_pixels(NP);
    constexpr bool HI = FORM == 1 || FORM == 3, BYTE = FORM == 3;
    constexpr int AP = MID + 16, YP = C + 16;          // row pitches of the patch (later b) and of the skip operand (later y)
    constexpr int S2 = 9 * 4, S1 = 16;                 // K steps of 64 of a wave's chunk: 3x3 layer, next block's layer (last layer: 4 per chunk)

    // what the patch, the biases and the ring need are leading arguments: in registers when a wave starts, the others arrive meanwhile
    struct { int W, rows, patch_bytes, n_tiles, per_xcd, touch; } g = {(int)(shape & 0x3ff), (int)(shape >> 10 & 0x7ff), (int)(shape >> 21 & 0xff) * 1024,
                                                                       (int)(tiles), (int)((tiles + 7) >> 3), NP == 1 ? (int)(shape >> 29 & 1) : 0};
    // LDS: patch, then b | skip operand, then y | biases: [256] 3x3 layer, [1024] last, [256] next
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int yb = g.patch_bytes;
    int32_t *const btab = (int32_t *)(lds + yb + PX * YP);
    // FORM 2 with ga.table (epilogue_pc_hi16): factors in the same order, skip multipliers and byte positions of the last layer, a word per wave: all of
    // its channels take that form.  (12544 pixels, per channel: 33 us with the packed parameters fetched from memory for every 32 pixels, 27.5 so.)
    int32_t *const atab = btab + 2 * MID + C, *const ktab = atab + 2 * MID + C, *const votes = ktab + C;
    uint8_t *const ptab = (uint8_t *)(votes + 8);
    [[maybe_unused]] bool one_product = false;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    // XCD-contiguous walk, as in the other fused kernels
    auto tile_of = [&](int v) { return (v & 7) * g.per_xcd + (v >> 3); };
    auto valid = [&](int v) { return (v >> 3) < g.per_xcd && tile_of(v) < g.n_tiles; };
    // every LDS access of this wave is over before the others go on (fragment reads in flight included)
    auto sync = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- copies global -> LDS, 1 KiB per wave-wide copy
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);      // (every place inside the tensor lies below 2 GiB, OOB above)
    TriArgs ga;
    ConvArgs a2, a3, a1;                               // read behind the first requests, the last two behind the 3x3 layer
    bool has_res = false;
    // 16-byte piece i of the patch region is piece i % 17 of row i / 17; the seventeenth is padding.  Row r is pixel p0 - W - 1 + r; pixels
    // outside the tensor, the padding and the rows behind the last one (the first of them is the row of zeros) get zeros.
    auto issue_patch = [&](int p0) {
        int l = lane;
        asm volatile("" : "+v"(l));                    // (worked out here: left alone, the compiler keeps it all in registers)
        const int first = p0 - g.W - 1;
#pragma unroll 1
        for (int c = wave; c < g.patch_bytes / 1024; c += 8) {
            const int i = c * 64 + l;
            const int row = (int)(((unsigned)i * 61681u) >> 20), piece = i - row * 17;         // / 17, exact below 2^16
            const int p = first + row;
            const unsigned off = piece < 16 && row < g.rows && (unsigned)p < (unsigned)M ? (unsigned)p * (unsigned)in_cs + piece * 16 : OOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(lds + c * 1024), 16, off, 0, 0, 0);
        }
    };
    // a pixel's whole skip operand per copy
    auto issue_skip = [&](int p0) {
        const int n = min(PX, M - p0);
        const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void *)a3.res, 0, ga.res_bytes, 0x00020000);
#pragma unroll 1
        for (int q = wave; q < n; q += 8)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_r, (__attribute__((address_space(3))) void *)(lds + yb + q * YP), 16, lane * 16,
                                                     (unsigned)(p0 + q) * (unsigned)a3.res_cs, 0, 0);
    };

    // ---- weights: this wave's 32-channel chunk of every layer, two fragments per K step, a ring of eight steps
    // An XCD's workgroups start together and would ask its L2 for the same lines, which come from beyond it, all at once.  So each begins at another
    // tap and goes round, and at another quarter of the next block's layer (another order of the last layer's chunks changed nothing).  Tiles of 32 pixels,
    // which need a tap's weights twice as soon, touch them all first instead: every wave its share, a 128-byte line per lane, workgroups without a tile
    // included.  The 152-layer network, us, touched / from one place / in turn / touched and in turn: 8 images 713 / - / 764 / 718, 16 784 / 943 / 823 / 788,
    // 32 930 / 1060 / 928 / 920; tiles of 64 pixels, 64 images 1345 / 1475 / 1315 / 1340, 96 1824 / - / 1799 / 1813; launches side by side are not touched for
    // (2048 -> 2150 at two halves of 96).
    const int place = NP > 1 ? (int)(blockIdx.x >> 3) : 0, t0 = (int)((unsigned)place % 9u), k0 = place & 3;
    auto next_tap = [](int t, int n) { return t + n >= 9 ? t + n - 9 : t + n; };
    const uint8_t *const w2 = w2_packed + (size_t)wave * (S2 * kChunkBytes);
    const uint8_t *w3 = nullptr, *w1 = nullptr;        // channels ch * 256 + ... of the last layer: + ch * 32 steps
    v4i ring[8][2];                                    // two groups of four steps
    // (through a descriptor of the four steps at p: the address costs scalar instructions only, 36 clocks per matrix instruction of a SIMD in
    // the K loops against 45 with 64-bit vector addresses)
    auto steps_at = [&](const uint8_t *p) { return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 4 * kChunkBytes, 0x00020000); };
    const int lane16 = lane * 16;
    // fragment f of the ring (its steps' two fragments in order), from the group of four steps behind rs
    auto load_frag = [&](auto f_tag, __amdgpu_buffer_rsrc_t rs) __attribute__((always_inline)) {
        constexpr int f = decltype(f_tag)::value;
        ring[f >> 1][f & 1] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane16 + (f & 1) * 1024, ((f >> 1) & 3) * kChunkBytes, 0);
    };

    // (behind the patch's copies and before the ring's, so they are over when the ring's first fragments are here; what they fetch lands in the skip
    // operand's place before it does)
    auto touch_weights = [&]() {
        constexpr int N2 = 8 * S2 * kChunkBytes / 8192, N3 = 32 * 4 * kChunkBytes / 8192, N1 = NEXT ? 8 * S1 * kChunkBytes / 8192 : 0;
        for (int i = (int)(blockIdx.x >> 3) * 8 + wave; i < N2 + N3 + N1; i += grid) {
            const uint8_t *const p = i < N2 ? w2_packed + i * 8192 : i < N2 + N3 ? w3_packed + (i - N2) * 8192 : w1_packed + (i - N2 - N3) * 8192;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 8192, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + yb + wave * 256), 4, lane * 128, 0, 0, 0);
        }
    };

    // ---- this lane's pixels q = 32 j + col of the tile; slots beyond the tile stay on its last pixel and are never stored
    auto slot = [&](int j) { return min(32 * j + col, PX - 1); };
    const int co = wave * 32 + half * 16;              // its sixteen channels inside the 256 of a phase
    auto init = [&](v16i &c, const int32_t *tab) __attribute__((always_inline)) { c = bias16(tab + co); };

    v16i acc[NP];
    // half steps (32 channels) whose fragments are in flight: a half step is 32 NP clocks of matrix work, twice that beside the SIMD's other wave
    constexpr int NB = NP >= 3 ? 2 : NP == 2 ? 4 : 8, AHEAD = NB - 1;
    v4i bf[NB][NP];
    auto read_frag = [&](auto h_tag, auto j_tag, const int (&ad)[NP]) __attribute__((always_inline)) {
        constexpr int h = decltype(h_tag)::value, j = decltype(j_tag)::value;
        bf[h % NB][j] = *(const v4i *)(lds + ad[j] + h * 32);
    };
    auto first_frags = [&](const int (&ad)[NP]) __attribute__((always_inline)) {
        static_for<AHEAD>([&](auto h_tag) __attribute__((always_inline)) {
            static_for<NP>([&](auto j_tag) __attribute__((always_inline)) { read_frag(h_tag, j_tag, ad); });
        });
    };
    // Four K steps = 256 channels of the rows at ad: behind every matrix instruction, in its shadow, one fragment of the half step AHEAD of it is
    // read (beyond the group: of the next group, at nad), behind every half step one weight fragment fetched from nx, eight steps on.
    auto group = [&](auto half_tag, const int (&ad)[NP], const int (&nad)[NP], const uint8_t *nx) __attribute__((always_inline)) {
        constexpr int R0 = 4 * decltype(half_tag)::value;       // the ring's half that this group multiplies
        const __amdgpu_buffer_rsrc_t rs = steps_at(nx);
        static_for<8>([&](auto h_tag) __attribute__((always_inline)) {
            constexpr int h = decltype(h_tag)::value;
            static_for<NP>([&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value, hn = h + AHEAD;
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[R0 + (h >> 1)][h & 1], bf[h % NB][j], acc[j], 0, 0, 0);
                asm volatile("" : "+v"(acc[j]));       // here, not wherever the sums are needed
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (hn < 8) read_frag(std::integral_constant<int, hn>{}, j_tag, ad);
                else read_frag(std::integral_constant<int, hn - 8>{}, j_tag, nad);
                if constexpr (j == NP - 1) load_frag(std::integral_constant<int, R0 * 2 + h>{}, rs);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;

    // sixteen bytes of layer a at this lane's pixel, RES: with a skip operand
    // (FORM 2: its packed parameters, its place in atab; only the last layer, at MID of it, has an operand)
    auto finish = [&](const ConvArgs &a, auto res_tag, const v16i &c, const v4i &r8, [[maybe_unused]] const int32_t *pc, [[maybe_unused]] int at) __attribute__((always_inline)) {
        constexpr int RES = decltype(res_tag)::value;
        if constexpr (FORM == 2) {
            if (one_product) return epilogue_pc_hi16<RES>(a, atab + at, ktab + (at - MID), ptab + (at - MID), c, r8);
            return epilogue_pc_bytes16<RES>(a, c, r8, pc);
        }
        else if constexpr (HI) return epilogue_hi16<RES, BYTE>(a, ga.sk, c, r8);
        else return epilogue_bytes16<RES>(a, c, r8);
    };

    if (!valid(blockIdx.x)) {
        if (g.touch) touch_weights();
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(0);
        return;
    }
    // The patch, the biases and the ring are requested from arguments that are in registers when a wave starts, and nothing of it waits for the others, which
    // come some 1500 clocks later: with those asked for in between the patch was requested at 3000 clocks of a tile's 38000 and all of it here
    // at 7900, now at 900 and 5600.
    {
        issue_patch(tile_of(blockIdx.x) * PX);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        int bv[3];                                     // requested before the ring, written to the table behind the ring's loads
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int i = tid + q * 512;
            bv[q] = i < MID ? bias2[i] : (i < MID + C ? bias3[i - MID] : NEXT ? bias1[i - MID - C] : 0);
        }
        if (g.touch) touch_weights();
        auto read_arguments = [&]() __attribute__((always_inline)) {
            ga = late_argument<TriArgs>(offsetof(TriKernelArgs, ga));
            a2 = late_argument<ConvArgs>(offsetof(TriKernelArgs, a2));
            a3 = late_argument<ConvArgs>(offsetof(TriKernelArgs, a3));
            a1 = late_argument<ConvArgs>(offsetof(TriKernelArgs, a1));
            has_res = a3.res_mode != 0;
            w3 = late_argument<const uint8_t *>(offsetof(TriKernelArgs, w3)) + (size_t)wave * (4 * kChunkBytes);
            w1 = NEXT ? late_argument<const uint8_t *>(offsetof(TriKernelArgs, w1)) + (size_t)wave * (S1 * kChunkBytes) : w2;
        };
        if constexpr (FORM == 2) read_arguments();
        [[maybe_unused]] int factor[3] = {0, 0, 0}, rescale[3] = {0, 0, 0}, position[3] = {0, 0, 0};
        [[maybe_unused]] bool mine = true;
        if constexpr (FORM == 2) {
            if (ga.table) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int i = tid + q * 512;
                    if (i < MID) mine &= pc_hi_channel(a2.pc, i, false, factor[q], rescale[q], position[q]);
                    else if (i < MID + C) mine &= pc_hi_channel(a3.pc, i - MID, has_res, factor[q], rescale[q], position[q]);
                    else if (NEXT) mine &= pc_hi_channel(a1.pc, i - MID - C, false, factor[q], rescale[q], position[q]);
                }
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const __amdgpu_buffer_rsrc_t rs0 = steps_at(w2 + t0 * (4 * kChunkBytes)), rs1 = steps_at(w2 + next_tap(t0, 1) * (4 * kChunkBytes));
        static_for<16>([&](auto f_tag) __attribute__((always_inline)) { load_frag(f_tag, decltype(f_tag)::value < 8 ? rs0 : rs1); });
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FORM != 2) read_arguments();
        in_registers(a3.res_mode, a2.H, a2.div_howo.mul, a2.div_howo.s1, a2.div_howo.s2, a2.div_wo.mul, a2.div_wo.s1, a2.div_wo.s2, a3.res, a3.res_cs, ga.res_bytes);
#pragma unroll
        for (int q = 0; q < 3; ++q) btab[tid + q * 512] = bv[q];
        if constexpr (FORM == 2) {
            if (ga.table) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int i = tid + q * 512;
                    atab[i] = factor[q];
                    if (i >= MID && i < MID + C) {
                        ktab[i - MID] = rescale[q];
                        ptab[i - MID] = (uint8_t)position[q];
                    }
                }
                const bool all = __builtin_amdgcn_ballot_w64(!mine) == 0;
                if (lane == 0) votes[wave] = all;
            }
        }
        asm volatile("" ::: "memory");
    }

    for (int v = blockIdx.x; valid(v); v += grid) {
        const int p0 = tile_of(v) * PX;
        int taps[NP];                                  // bit t: tap t of the pixel lies in its image
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int p = min(p0 + 32 * j + col, M - 1);
            const int r = p - fast_div(p, a2.div_howo) * (a2.H * g.W);
            const int y = fast_div(r, a2.div_wo), x = r - y * g.W;
            const int cols = (x > 0 ? 1 : 0) | 2 | (x + 1 < g.W ? 4 : 0);
            taps[j] = (y > 0 ? cols : 0) | cols << 3 | (y + 1 < a2.H ? cols << 6 : 0);
        }
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(16);                           // this wave's copies of the patch have landed: sixteen younger loads at least are the ring's
        sync();                                        // ... everybody's; and nobody reads the last tile's y any more
        if (has_res) issue_skip(p0);
        if constexpr (FORM == 2) {
            if (ga.table) {
                int all = 1;
#pragma unroll
                for (int k = 0; k < 8; ++k) all &= votes[k];
                one_product = __builtin_amdgcn_readfirstlane(all) != 0;
            }
        }

        // ---------------- phase 1: 3x3
#pragma unroll
        for (int j = 0; j < NP; ++j) init(acc[j], btab);
        {
            const int zero = g.rows * AP + half * 16;
            int centre[NP], ad[NP], nad[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) centre[j] = (slot(j) + g.W + 1) * AP + half * 16;
            auto tap = [&](int (&d)[NP], int t, int off) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NP; ++j) d[j] = (taps[j] >> t) & 1 ? centre[j] + off : zero;
            };
            int kw = t0 % 3, tc = t0;
            int off = ((t0 / 3 - 1) * g.W + kw - 1) * AP;
            tap(ad, t0, off);
            first_frags(ad);
            auto one = [&](auto half_tag, int t) __attribute__((always_inline)) {
                if (t < 8) {
                    off += AP;
                    if (++kw == 3) { kw = 0; off += (g.W - 3) * AP; }
                    if (++tc == 9) { tc = 0; off = -(g.W + 1) * AP; }
                }
                tap(nad, tc, off);
                group(half_tag, ad, nad, t < 7 ? w2 + next_tap(t0, t + 2) * (4 * kChunkBytes) : w3 + (t - 7) * (32 * kChunkBytes));
#pragma unroll
                for (int j = 0; j < NP; ++j) ad[j] = nad[j];
            };
#pragma unroll 1
            for (int t = 0; t < 8; t += 2) {
                one(H0{}, t);
                one(H1{}, t + 1);
            }
            // (what the next phases want of the arguments: read here, under the last tap's products)
            a3 = late_argument<ConvArgs>(offsetof(TriKernelArgs, a3));
            a1 = late_argument<ConvArgs>(offsetof(TriKernelArgs, a1));
            one(H0{}, 8);
        }
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(16);                           // the skip operand's copies (all older than the ring's loads) have landed
        sync();                                        // ... everybody's, and every wave has its last fragments of the patch: b may overwrite it
        mfma_drain(acc);
        static_for<NP>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            const v4i w = finish(a2, H0{}, acc[j], v4i{0, 0, 0, 0}, a2.pc + (2 * wave + half) * kPcGroupInts, co);
            if (32 * j + 31 < PX || 32 * j + col < PX) *(v4i *)(lds + (32 * j + col) * AP + co) = w;
            __builtin_amdgcn_sched_barrier(0);
        });
        sync();

        // ---------------- phase 2: 1x1, 256 output channels at a time, one pixel group of a chunk after the other
        {
            int ad[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) ad[j] = slot(j) * AP + half * 16;
            const int at0 = yb + co;                   // this lane's bytes of chunk ch at pixel q: + q * YP + ch * 256
            // the next fragments of b: four half steps in flight, across the groups
            v4i fr[4];
            v16i c2[2];                                // the group being multiplied, the one being finished
            v4i r8[2];
            int w[4];
#pragma unroll
            for (int h = 0; h < 3; ++h) fr[h] = *(const v4i *)(lds + ad[0] + h * 32);
            // group J of chunk ch (PAR: the parity of its number); the one before it (OJ, of chunk och) is finished meanwhile
            auto item = [&](auto half_tag, auto j_tag, auto par_tag, auto first_tag, int ch) __attribute__((always_inline)) {
                constexpr int R0 = 4 * decltype(half_tag)::value, j = decltype(j_tag)::value, PAR = decltype(par_tag)::value;
                constexpr int oj = j == 0 ? NP - 1 : j - 1, nj = j + 1 < NP ? j + 1 : 0;
                const bool old = !decltype(first_tag)::value || ch > 0;        // there is a group before it
                init(c2[PAR], btab + MID + ch * MID);
                const __amdgpu_buffer_rsrc_t rs = steps_at(ch + 2 < C / MID ? w3 + (ch + 2) * (32 * kChunkBytes) : NEXT ? w1 + ((k0 + ch + 2 - C / MID) & 3) * (4 * kChunkBytes) :
                                                            w2 + next_tap(t0, ch + 2 - C / MID) * (4 * kChunkBytes));
                static_for<8>([&](auto h_tag) __attribute__((always_inline)) {
                    constexpr int h = decltype(h_tag)::value, hn = h + 3;
                    c2[PAR] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[R0 + (h >> 1)][h & 1], fr[h & 3], c2[PAR], 0, 0, 0);
                    asm volatile("" : "+v"(c2[PAR]));
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (hn < 8) fr[hn & 3] = *(const v4i *)(lds + ad[j] + hn * 32);
                    else fr[hn & 3] = *(const v4i *)(lds + ad[nj] + (hn - 8) * 32);
                    if constexpr (j == NP - 1) load_frag(std::integral_constant<int, R0 * 2 + h>{}, rs);
                    if constexpr (h == 4) r8[PAR] = *(const v4i *)(lds + at0 + slot(j) * YP + ch * MID);
                    if constexpr (HI)
                        if (old) epilogue_hi_slice<1, 2 * h, 2, BYTE>(a3, ga.sk, c2[PAR ^ 1], r8[PAR ^ 1], w);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (HI) {
                    if (old && (32 * oj + 31 < PX || 32 * oj + col < PX))
                        *(v4i *)(lds + at0 + (32 * oj + col) * YP + (j == 0 ? ch - 1 : ch) * MID) = v4i{w[0], w[1], w[2], w[3]};
                    mfma_drain(c2[PAR]);
                } else {
                    mfma_drain(c2[PAR]);
                    const int32_t *pc = a3.pc + ((ch * 8 + wave) * 2 + half) * kPcGroupInts;
                    const int at = MID + ch * MID + co;
                    const v4i o = has_res ? finish(a3, H1{}, c2[PAR], r8[PAR], pc, at) : finish(a3, H0{}, c2[PAR], r8[PAR], pc, at);
                    if (32 * j + 31 < PX || 32 * j + col < PX) *(v4i *)(lds + at0 + (32 * j + col) * YP + ch * MID) = o;
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto chunk = [&](auto half_tag, auto odd_tag, auto first_tag, int ch) __attribute__((always_inline)) {
                constexpr int P0 = decltype(odd_tag)::value * NP;
                // b goes to memory as well: four pixels per wave-wide store, dealt over waves and chunks
                if (a2.out) {
                    int l = lane;
                    asm volatile("" : "+v"(l));
                    const int q = (wave + 8 * ch) * 4 + (l >> 4), piece = (l & 15) * 16;
                    if (ch < NP && q < PX && p0 + q < M)
                        *(v4i *)((uint8_t *)a2.out + (size_t)(p0 + q) * a2.out_cs + a2.out_co + piece) = *(const v4i *)(lds + q * AP + piece);
                }
                static_for<NP>([&](auto j_tag) __attribute__((always_inline)) {
                    constexpr int j = decltype(j_tag)::value;
                    item(half_tag, j_tag, std::integral_constant<int, (P0 + j) & 1>{}, std::integral_constant<bool, decltype(first_tag)::value && j == 0>{}, ch);
                });
            };
#pragma unroll
            for (int ch = 0; ch < C / MID; ch += 2) {  // (nine groups of the ring so far)
                chunk(H1{}, H0{}, std::true_type{}, ch);
                chunk(H0{}, H1{}, std::false_type{}, ch + 1);
            }
            if constexpr (HI) {
                constexpr int PAR = (2 * NP - 1) & 1;
                const v4i o = finish(a3, H1{}, c2[PAR], r8[PAR], nullptr, 0);
                if (32 * NP - 1 < PX || 32 * (NP - 1) + col < PX) *(v4i *)(lds + at0 + (32 * (NP - 1) + col) * YP + 3 * MID) = o;
            }
        }
        sync();                                        // y is complete; nobody reads b any more

        // y leaves LDS one pixel's whole row per store
        auto store_y = [&](int q) __attribute__((always_inline)) {
            if (q < PX && p0 + q < M)
                *(v4i *)((uint8_t *)a3.out + (size_t)(p0 + q) * a3.out_cs + a3.out_co + lane16) = *(const v4i *)(lds + yb + q * YP + lane16);
        };
        const int vn = v + grid;
        if constexpr (NEXT) {
            if (valid(vn)) issue_patch(tile_of(vn) * PX);      // travels during this phase
            // ---------------- phase 3: 1x1, K = 1024
            int ad[NP], nad[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                ad[j] = yb + slot(j) * YP + half * 16 + k0 * 256;
                init(acc[j], btab + MID + C);
            }
            first_frags(ad);
            auto quarter = [&](auto half_tag, int k) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NP; ++j) nad[j] = k + k0 == 3 ? ad[j] - 768 : ad[j] + 256;
                constexpr int PER = (PX + 31) / 32;
                for (int c = k * PER; c < (k + 1) * PER; ++c) store_y(wave + 8 * c);
                group(half_tag, ad, nad, k < 2 ? w1 + ((k + k0 + 2) & 3) * (4 * kChunkBytes) : w2 + next_tap(t0, k - 2) * (4 * kChunkBytes));
#pragma unroll
                for (int j = 0; j < NP; ++j) ad[j] = nad[j];
            };
#pragma unroll 1
            for (int k = 0; k < 4; k += 2) {
                quarter(H1{}, k);
                quarter(H0{}, k + 1);
            }
            mfma_drain(acc);
            static_for<NP>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                const v4i w = finish(a1, H0{}, acc[j], v4i{0, 0, 0, 0}, a1.pc + (2 * wave + half) * kPcGroupInts, MID + C + co);
                const int q = 32 * j + col;
                if (q < PX && p0 + q < M) *(v4i *)((uint8_t *)a1.out + (size_t)(p0 + q) * a1.out_cs + a1.out_co + co) = w;
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
#pragma unroll 2
            for (int c = 0; c < (PX + 7) / 8; ++c) store_y(wave + 8 * c);
            if (valid(vn)) {
                issue_patch(tile_of(vn) * PX);         // (b is no longer read)
                asm volatile("" ::: "memory");
                ICNN_WAIT_VMCNT(0);
            }
        }
        if (!valid(vn)) break;
        // an odd number of groups: the next tile's first four steps are in the ring's other half
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const v4i w = ring[r][f];
                ring[r][f] = ring[r + 4][f];
                ring[r + 4][f] = w;
            }
    }
#endif
}

// TriKernelArgs' members are the kernel's parameters
inline auto tri_members(TriKernelArgs k)
{
    auto [x, w2, bias2, bias3, bias1, M, in_cs, shape, tiles, grid, w3, w1, ga, a2, a3, a1] = k;
    return Types<decltype(x), decltype(w2), decltype(bias2), decltype(bias3), decltype(bias1), decltype(M), decltype(in_cs), decltype(shape), decltype(tiles), decltype(grid),
                 decltype(w3), decltype(w1), decltype(ga), decltype(a2), decltype(a3), decltype(a1)>();
}
static_assert(std::is_same_v<decltype(tri_members(TriKernelArgs())), decltype(parameters_of(&conv_tri_kernel<1, true, 1>))>, "late_argument reads by this struct");

// ------------------------------------------------------------------ dispatch
namespace {
size_t tri_lds_bytes(const TriArgs &g) { return (size_t)g.patch_bytes + (size_t)tri_pixels(g.np) * (kTriWide + 16) + (2 * kTriMid + kTriWide) * 4; }

bool tri_shape(long long M, int W, int np, TriArgs &g)
{
    const int px = tri_pixels(np);
    g.np = np;
    g.touch = 0;
    g.W = W;
    g.rows = px + 2 * (W + 1);
    g.patch_bytes = ((g.rows + 1) * 17 + 63) / 64 * 1024;
    if (g.rows > 1024 || tri_lds_bytes(g) > 160 * 1024) return false;
    const long long tiles = (M + px - 1) / px;
    g.n_tiles = (int)tiles;
    g.per_xcd = (int)((tiles + 7) / 8);
    return true;
}
}  // namespace

// Which tile.  One round of tiles on the 256 compute units takes 14, 19, 25 or 31 us by tile (28 for two rounds of the smallest), whatever their
// number: the cheapest in rounds.  The 152-layer network, us, 32 / 64 / 96 / 112 pixels: 769 / 903 / 1093 / 1260 at 16 images, 842 / 962 / 1146 / 1326 at 24, 1043 / 1108 / 1274 / 1448
// at 40, 1386 / 1172 / 1337 / 1515 at 48, 1510 / 1308 / 1466 / 1633 at 64, 1447 / 1260 / 1412 / 1597 at 72 (24, 72 and 84 on a faster machine).  With several launches side by side, the
// smallest of the first three tiles that gives all of them a compute unit each (two halves of 84 images: 1729 / 1460 / 1474 / 1661, of 96: 1897 / 1716 / 1695 / 1836), and
// where none does the same rule as alone (of 128: 2410 / 1996 / 2201 / 2224).  Every one of these goes to its best tile or within 1.1 % of it; beyond, the figures leave
// the rule: 168 images 3078 / 2575 / 2709 / 2818 (it takes 96 pixels), 256 4438 / 3796 / 3661 / 3922 (112).
bool conv_tri_plan(long long M, int W, int lanes, TriArgs &g)
{
    if (M < 1 || M > 0x7fffffffLL - 256 || W > 1000) return false;
    auto touch = [&]() { g.touch = lanes == 1 && g.np == 1; return true; };
    if (g_tuning.tri_tile) return tri_shape(M, W, g_tuning.tri_tile, g) && touch();
    static const int cost[5] = {0, 14, 19, 25, 31};
    long long best = -1;
    TriArgs t = g;
    for (int np = 1; np <= 4; ++np) {
        if (!tri_shape(M, W, np, t)) break;
        if (lanes > 1 && np < 4 && (long long)t.n_tiles * lanes <= 256) {
            g = t;
            return true;
        }
        const long long c = ((long long)t.n_tiles + 255) / 256 * cost[np];
        if (best < 0 || c < best) {
            best = c;
            g = t;
        }
    }
    return best >= 0 && touch();
}

// a1: the next block's first layer, or null.  The caller has checked widths (256 -> 256 -> 1024 -> 256), kinds and alignment.
hipError_t launch_conv_tri(const TriArgs &g, const ConvArgs &a2, const ConvArgs &a3, const ConvArgs *a1, hipStream_t st)
{
    if (a2.Cin != kTriMid || a2.Cout != kTriMid || a3.Cin != kTriMid || a3.Cout != kTriWide || (a1 && (a1->Cin != kTriWide || a1->Cout != kTriMid)) ||
        g.n_tiles < 1 || g.np < 1 || g.np > 4 || g.W != a2.W || g.rows != tri_pixels(g.np) + 2 * (g.W + 1) ||
        (long long)g.n_tiles * tri_pixels(g.np) < a2.M || tri_lds_bytes(g) > 160 * 1024)
        return hipErrorInvalidValue;
    // (17 workgroups per XCD touch all of the weights at once; more without a tile would only wait for compute units)
    const int slots = std::min(256, std::max(8 * g.per_xcd, g.touch ? 136 : 0));
    ConvArgs b2 = a2;
    TriArgs q = g;
    q.sk = a3.res_mode ? make_skip_mul(a3.res_mul, a3.res_shift) : SkipMul{0, 0, 0};      // (without an operand the arithmetic runs on zeros)
    b2.div_howo = make_fast_div((unsigned)(a2.H * a2.W));
    b2.div_wo = make_fast_div((unsigned)a2.W);
    // (the biggest tile leaves no room for the tables)
    const size_t tables = (2 * kTriMid + 2 * kTriWide + 8) * 4 + kTriWide;
    q.table = a3.pc && tri_lds_bytes(g) + tables <= 160 * 1024;
    const size_t lds_bytes = tri_lds_bytes(g) + (q.table ? tables : 0);
    int form = a3.pc ? 2 : a2.rq_fast && a3.rq_fast && (!a3.res_mode || q.sk.ok) && (!a1 || a1->rq_fast) ? 1 : 0;
    if (form == 1 && requant_fits_byte(a2) && requant_fits_byte(a3) && (!a1 || requant_fits_byte(*a1))) form = 3;
    auto go = [&](auto kernel) -> hipError_t {
        const hipError_t e = allow_large_lds((const void *)kernel);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)slots), dim3(512), lds_bytes, st, a2.x, a2.wp, a2.bias, a3.bias, a1 ? a1->bias : a2.bias, a2.M, a2.in_cs,
                           (unsigned)g.W | (unsigned)g.rows << 10 | (unsigned)(g.patch_bytes / 1024) << 21 | (g.touch ? 1u << 29 : 0u), (unsigned)g.n_tiles, slots, a3.wp,
                           a1 ? a1->wp : a2.wp, q, b2, a3, a1 ? *a1 : a2);
        return hipGetLastError();
    };
    auto by_form = [&](auto np_tag, auto next_tag) {
        constexpr int NP = decltype(np_tag)::value;
        constexpr bool NEXT = decltype(next_tag)::value;
        return form == 2 ? go(conv_tri_kernel<NP, NEXT, 2>) : form == 3 ? go(conv_tri_kernel<NP, NEXT, 3>) : form == 1 ? go(conv_tri_kernel<NP, NEXT, 1>) : go(conv_tri_kernel<NP, NEXT, 0>);
    };
    auto by_next = [&](auto np_tag) { return a1 ? by_form(np_tag, std::true_type{}) : by_form(np_tag, std::false_type{}); };
    switch (g.np) {
    case 1: return by_next(std::integral_constant<int, 1>{});
    case 2: return by_next(std::integral_constant<int, 2>{});
    case 3: return by_next(std::integral_constant<int, 3>{});
    default: return by_next(std::integral_constant<int, 4>{});
    }
}

}  // namespace icnn
