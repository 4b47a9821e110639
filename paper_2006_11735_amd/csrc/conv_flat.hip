// A 3x3 or 1x1 layer of stride 1 or 2 whose weights go from memory straight into the registers of the one wave of a workgroup that
// multiplies them, and whose input crosses the compute unit's memory path once per 128 output channels.
//
//   tile     PX consecutive pixels of the flattened N*Ho*Wo axis; patch (3x3): these and the W + 1 pixels before and behind
//            them, so that tap (kh, kw) of a pixel is the patch row (kh - 1) * W + kw - 1 away; a tap beyond the image's edge
//            reads a row of zeros instead, chosen by a mask of nine bits per pixel.  Stride 2: the input as four planes of the output's
//            size, the pixels of even and odd rows and columns; the tile's pixels in the first, with one, Wo and Wo + 1 more before them
//            in the others, and a tap is a row's distance again.  The whole patch, all channels, lies in
//            LDS before the K loop begins, rows padded by 16 bytes (any 16 consecutive rows start in different banks)
//   waves    four: WC along the output channels, 32 each; 4 / WC along the pixels, 64 each
//   K loop   groups of G steps of 64; every group of weights is fetched eight K steps ahead; no barrier
//
// Two or three workgroups share a compute unit: one's copies and epilogue run beside another's matrix instructions.  What bounds it is the
// compute unit's memory path (64 to 72 bytes a clock): a 3x3 of 256 channels takes 295 KB of weights and 30 KB of patch per 64 pixels x 128
// channels, 4608 clocks of matrix instructions on its four units.
//
// Per output channel (FORM 2) each wave works its 32 channels' factors out once, into LDS, and finishes with the products of FORM 1 where they
// are exact for all of them (otherwise with epilogue_pc_tiles, which fetches the packed parameters from memory four channels at a time): 64 images
// of 28 x 28, 128 -> 512 with skip operand, 25.4 us in the tile kernel, 15.6 here, 15.2 with one pair per layer.
#include "conv_common.h"

#include <algorithm>
#include <type_traits>

namespace icnn {

struct FlatArgs {
    int rows, patch_bytes;        // patch rows; bytes of it in LDS with the row of zeros behind, in whole KiB
    SkipMul sk;
};
// What the patch's copies, the biases and the weights need, passed as single arguments, which are in registers when a wave starts; the other arguments
// come by scalar loads and are waited for behind those requests.  (86 instructions at some 9 clocks and two rounds of scalar loads before the first
// request, 157 and four before the first weights; us at 64 images, before / now: 1024 -> 256 on 14 x 14 8.8 / 8.0, 2048 -> 512 on 7 x 7 9.9 / 8.8, 512 -> 2048
// 10.5 / 9.8, 3x3 of 512 channels 13.2 / 12.5, at stride 2 16.3 / 15.6; launches of several rounds gain less, 128 -> 512 on 28 x 28 per channel 16.6 / 15.9.)
struct FlatFirst {
    const uint8_t *x, *wp;
    const int32_t *bias, *pc;
    int M, in_cs;
    unsigned shape;               // patch rows (11 bits), KiB of it (8), image width (13)
    unsigned div_mul;             // a workgroup's number by channel tiles, or by pixel tiles where neighbouring workgroups share channels
    unsigned tiles;               // channel tiles (16 bits), that division's shifts (8, 6), whether it is by pixel tiles, whether there is a skip operand
};

constexpr int kFlatTables = 4 * 72 * 4;                // of four waves' 32 channels
constexpr int kFlatSums = 4 * 32 * (32 * 4 + 16);      // 32 pixels' int32 sums of four waves

// KK: kernel size; NG groups of G steps: cin = 64 G NG / KK^2.  FORM: 1 requantisation as a product's high word (rq_fast), an unsigned 8-bit skip
// operand before it rescaled likewise (g.sk) or none, 8-bit output; 5 as 1, to bytes (requant_fits_byte); 0 any form of one pair per layer; 2 per output channel; 3 as 1 with an int32
// skip operand; 4 int32 sums.
// S: stride, both ways.
template <int KK, int NG, int G, int WC, int FORM, int S>
__global__ __launch_bounds__(256, 2) void conv_flat_kernel(const uint8_t *x, const uint8_t *weights, const int32_t *bias, const int32_t *pc, const int M,
                                                           const int in_cs, const unsigned shape, const unsigned div_mul, const unsigned tiles,
                                                           const ConvArgs a, const FlatArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    constexpr int CIN = 64 * G * NG / (KK * KK), GP = NG / (KK * KK);      // groups per tap
    constexpr int AP = CIN + 16, PIECES = AP / 16, PX = 64 * (4 / WC), NS = 8 / G;
    constexpr int T = NG * G;                          // K steps
    constexpr bool HI = FORM == 1 || FORM == 5, BYTE = FORM == 5;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    const int rows = (int)(shape & 0x7ff), patch_bytes = (int)(shape >> 11 & 0xff) * 1024, W = (int)(shape >> 19);

    // LDS: patch | biases of the tile's channels | FORM 2: factors, skip multipliers | stride 2: where each patch row is in the input
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    int32_t *const btab = (int32_t *)(lds + patch_bytes);
    int32_t *const ptab = btab + 128 + wave * 72;                          // FORM 2: this wave's 32 factors, 32 skip multipliers and positions
    unsigned *const rtab = (unsigned *)(lds + patch_bytes + 512 + (FORM == 2 ? kFlatTables : 0));

    // (as tile_of_block; the division by pixel tiles where the host found neighbours sharing channels the better order)
    const int n_ct = (int)(tiles & 0xffff), n_pt = (int)(((unsigned)M + PX - 1) / PX), n_tiles = n_ct * n_pt;
    const int logical = (int)(blockIdx.x & 7) * ((n_tiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (logical >= n_tiles) return;
    const bool by_pt = tiles >> 30 & 1;
    const int major = fast_div_packed(logical, div_mul, tiles >> 16 & 0xff, tiles >> 24 & 0x3f), minor = logical - major * (by_pt ? n_pt : n_ct);
    const int ct = by_pt ? major : minor, pt = by_pt ? minor : major;
    const int p0 = pt * PX;
    const int wc = wave % WC, pw = p0 + (wave / WC) * 64;                  // this wave's channels in the tile, first pixel
    const int co_tile = ct * (WC * 32), co_wave = co_tile + wc * 32;

    // ---- weights: group k of this wave's chunk in slot k % NS of the ring
    const uint8_t *const wp = weights + (size_t)(co_wave >> 5) * (T * kChunkBytes);
    v4i ring[NS][2 * G];
    const int lane16 = lane * 16;
    auto load_frag = [&](auto k_tag, auto f_tag) __attribute__((always_inline)) {
        constexpr int k = decltype(k_tag)::value, f = decltype(f_tag)::value;
        if constexpr (k < NG) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(wp + k * (G * kChunkBytes)), 0, G * kChunkBytes, 0x00020000);
            ring[k % NS][f] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
        }
    };

    // ---- prologue: patch, biases and the ring's first groups in flight together.  Stride 2, whose patch rows take the other arguments to find: the ring first
    constexpr int FIRST = NS < NG ? NS : NG;
    auto start_ring = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        static_for<FIRST * 2 * G>([&](auto i_tag) __attribute__((always_inline)) {
            constexpr int i = decltype(i_tag)::value;
            load_frag(std::integral_constant<int, i / (2 * G)>{}, std::integral_constant<int, i % (2 * G)>{});
        });
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // stride 2: first patch rows of the pixels of odd columns, odd rows, both
    [[maybe_unused]] int eo = 0, oe = 0, oo = 0;
    if constexpr (S == 2) {
        start_ring();
        in_registers(a.Ho, a.Wo, a.H, a.div_howo.mul, a.div_howo.s1, a.div_howo.s2, a.div_wo.mul, a.div_wo.s1, a.div_wo.s2);
        eo = PX; oe = 2 * PX + 1; oo = 3 * PX + 1 + a.Wo;
        for (int r = tid; r < rows; r += 256) {
            const int odd_y = KK == 3 && r >= oe, odd_x = KK == 3 && (r >= oo || (r >= eo && r < oe));
            const int p = p0 + (KK == 1 || r < eo ? r : r < oe ? r - eo - 1 : r < oo ? r - oe - a.Wo : r - oo - a.Wo - 1);
            unsigned off = OOB;
            if ((unsigned)p < (unsigned)M) {
                const int n = fast_div(p, a.div_howo), at = p - n * (a.Ho * a.Wo), y = fast_div(at, a.div_wo);
                const int iy = 2 * y + odd_y, ix = 2 * (at - y * a.Wo) + odd_x;
                if (iy < a.H && ix < W) off = (unsigned)((n * a.H + iy) * W + ix) * (unsigned)in_cs;
            }
            rtab[r] = off;
        }
        // (the barrier is for the table alone: the ring's loads stay in flight)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    {
        // (every place inside the tensor lies below 2 GiB, OOB above)
        const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);
        const int first = KK == 3 ? p0 - W - 1 : p0;
        // 16-byte piece i of the patch region is piece i % PIECES of row i / PIECES, the last of a row padding; pixels outside the tensor, the
        // padding and the rows behind the last one (the first of them is the row of zeros) get zeros
        int row = tid / PIECES, piece = tid - row * PIECES;
        for (int c = wave; c < patch_bytes / 1024; c += 4) {
            unsigned off;
            if constexpr (S == 2) {
                off = piece < PIECES - 1 && row < rows ? rtab[min(row, rows - 1)] + piece * 16 : OOB;
            } else {
                const int p = first + row;
                off = piece < PIECES - 1 && row < rows && (unsigned)p < (unsigned)M ? (unsigned)p * (unsigned)in_cs + piece * 16 : OOB;
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(lds + c * 1024), 16, off, 0, 0, 0);
            row += 256 / PIECES;
            piece += 256 % PIECES;
            if (piece >= PIECES) { piece -= PIECES; ++row; }
        }
    }
    const int bv = bias[co_tile + min(tid, WC * 32 - 1)];
    [[maybe_unused]] int factor = 0, rescale = 0, position = 0;
    [[maybe_unused]] bool one_product = false;
    if constexpr (FORM == 2) one_product = pc_hi_channel(pc, co_wave + col, tiles >> 31, factor, rescale, position);
    if constexpr (S == 1) start_ring();
    in_registers(a.Ho, a.Wo, a.H, a.div_howo.mul, a.div_howo.s1, a.div_howo.s2, a.div_wo.mul, a.div_wo.s1, a.div_wo.s2, a.res_mode, a.res, a.res_cs, a.out, a.out_cs,
                 a.out_co, a.lo, a.hi);
    if constexpr (HI) in_registers(a.mul_hi, g.sk.k, g.sk.rnd);
    if (tid < WC * 32) btab[tid] = bv;
    if constexpr (FORM == 2) {
        ptab[lane] = half ? rescale : factor;
        if (half == 0) ((uint8_t *)(ptab + 64))[col] = (uint8_t)position;
        one_product = a.pc_fast_ok && __builtin_amdgcn_ballot_w64(!one_product) == 0;
    }
    // this lane's pixels
    int taps[2], q[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        q[j] = (wave / WC) * 64 + 32 * j + col;
        if constexpr (KK == 3) {
            const int p = min(p0 + q[j], M - 1);
            const int r = p - fast_div(p, a.div_howo) * (a.Ho * a.Wo);
            const int y = fast_div(r, a.div_wo), x = r - y * a.Wo;
            const int cols = (x > 0 ? 1 : 0) | 2 | (S * x + 1 < W ? 4 : 0);
            taps[j] = (y > 0 ? cols : 0) | cols << 3 | (S * y + 1 < a.H ? cols << 6 : 0);
        }
    }
    v4i res8[1][2];
    [[maybe_unused]] v4i res32[2][4];
    if constexpr (FORM == 3) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                res32[j][i] = *(const v4i *)((const int32_t *)a.res + ((size_t)min(pw + 32 * j + 8 * i + (lane >> 3), M - 1) * a.res_cs + co_wave + 4 * (lane & 7)));
    } else if constexpr (HI) {
        if (a.res_mode != 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                res8[0][j] = p0 + q[j] < M ? *(const v4i *)((const uint8_t *)a.res + ((size_t)(p0 + q[j]) * a.res_cs + co_wave + half * 16)) : v4i{0, 0, 0, 0};
        }
    } else {
        prefetch_res8<1, 2>(a, co_wave, pw, lane, res8);
    }
    asm volatile("" ::: "memory");
    ICNN_WAIT_VMCNT((S == 1 ? 2 * G * FIRST : 0));     // this wave's copies of the patch have landed: as many younger loads at least are the ring's
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();                      // ... everybody's
    asm volatile("" ::: "memory");

    // ---- K loop
    v16i acc[1][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[0][j] = bias16(btab + wc * 32 + half * 16);
    {
        constexpr int NB = 2 * G < 4 ? 2 * G : 4, AHEAD = NB - 1, H = 2 * G;       // fragments in flight; half steps (32 channels) of a group
        v4i bf[NB][2];
        const int zero = rows * AP + half * 16;
        int ad[2], nad[2];
        auto tap = [&](auto t_tag, int (&d)[2]) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value, kh = t / 3, kw = t % 3;
            const int from = KK == 1 ? 0 : S == 1 ? kh * W + kw :
                             (kh == 1 ? kw == 1 ? 0 : eo : (kw == 1 ? oe : oo) + (kh == 2 ? a.Wo : 0)) + (kw == 2 ? 1 : 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int at = (q[j] + from) * AP + half * 16;
                d[j] = KK == 1 || (taps[j] >> t) & 1 ? at : zero;
            }
        };
        tap(std::integral_constant<int, 0>{}, ad);
#pragma unroll
        for (int h = 0; h < AHEAD; ++h)
#pragma unroll
            for (int j = 0; j < 2; ++j) bf[h][j] = *(const v4i *)(lds + ad[j] + h * 32);
        static_for<NG>([&](auto k_tag) __attribute__((always_inline)) {
            constexpr int k = decltype(k_tag)::value, part = KK == 3 ? k % GP : k, next = KK == 3 ? (k + 1) % GP : k + 1;
            constexpr int AT = part * (G * 64), NAT = k + 1 < NG ? next * (G * 64) : AT;
            if constexpr (KK == 3 && next == 0 && k + 1 < NG) tap(std::integral_constant<int, (k + 1) / GP>{}, nad);
            else {
                nad[0] = ad[0];
                nad[1] = ad[1];
            }
            static_for<H>([&](auto h_tag) __attribute__((always_inline)) {
                constexpr int h = decltype(h_tag)::value, hn = h + AHEAD;
                static_for<2>([&](auto j_tag) __attribute__((always_inline)) {
                    constexpr int j = decltype(j_tag)::value;
                    acc[0][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[k % NS][h], bf[h % NB][j], acc[0][j], 0, 0, 0);
                    asm volatile("" : "+v"(acc[0][j]));        // here, not wherever the sums are needed
                    __builtin_amdgcn_sched_barrier(0);
                    bf[hn % NB][j] = *(const v4i *)(lds + (hn < H ? ad[j] + AT + hn * 32 : nad[j] + NAT + (hn - H) * 32));
                    if constexpr (j == 1) load_frag(std::integral_constant<int, k + NS>{}, h_tag);
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            ad[0] = nad[0];
            ad[1] = nad[1];
        });
    }
    mfma_drain(acc);
    // int32 sums, stored (FORM 4) or joined (FORM 3): a pixel's 32 are 128 bytes, of which a lane has half in its accumulators.  They pass through LDS, so
    // that an access to memory has eight whole lines and not a quarter of 64 halves.  (A region of the wave's own; its LDS accesses keep their order.)
    constexpr int SP = 32 * 4 + 16;
    [[maybe_unused]] uint8_t *const sums = lds + patch_bytes + 512 + (S == 2 ? (rows * 4 + 511) / 512 * 512 : 0) + wave * (32 * SP);
    [[maybe_unused]] const int px = lane >> 3, piece = (lane & 7) * 16;
    if constexpr (FORM == 4) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(v4i *)(sums + col * SP + half * 64 + i * 16) = v4i{acc[0][j][4 * i], acc[0][j][4 * i + 1], acc[0][j][4 * i + 2], acc[0][j][4 * i + 3]};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v4i v = *(const v4i *)(sums + (8 * i + px) * SP + piece);
                const int p = pw + 32 * j + 8 * i + px;
                if (p < M) *(v4i *)((uint8_t *)((int32_t *)a.out + (size_t)p * a.out_cs + a.out_co + co_wave) + piece) = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    } else if constexpr (FORM == 3) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            v4i r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) *(v4i *)(sums + (8 * i + px) * SP + piece) = res32[j][i];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = *(const v4i *)(sums + col * SP + half * 64 + i * 16);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const v4i w = epilogue_skip_s32(a, acc[0][j], r);
            if (p0 + q[j] < M) *(v4i *)((uint8_t *)a.out + (size_t)(p0 + q[j]) * a.out_cs + a.out_co + co_wave + half * 16) = w;
        }
    } else if constexpr (HI) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const v4i w = a.res_mode != 0 ? epilogue_hi16<1, BYTE>(a, g.sk, acc[0][j], res8[0][j]) : epilogue_hi16<0, BYTE>(a, g.sk, acc[0][j], v4i{0, 0, 0, 0});
            if (p0 + q[j] < M) *(v4i *)((uint8_t *)a.out + (size_t)(p0 + q[j]) * a.out_cs + a.out_co + co_wave + half * 16) = w;
        }
    } else if constexpr (FORM == 2) {
        if (one_product) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const v4i w = a.res_mode != 0 ? epilogue_pc_hi16<1>(a, ptab + half * 16, ptab + 32 + half * 16, (const uint8_t *)(ptab + 64) + half * 16, acc[0][j], res8[0][j])
                                              : epilogue_pc_hi16<0>(a, ptab + half * 16, ptab, nullptr, acc[0][j], v4i{0, 0, 0, 0});
                if (p0 + q[j] < M) *(v4i *)((uint8_t *)a.out + (size_t)(p0 + q[j]) * a.out_cs + a.out_co + co_wave + half * 16) = w;
            }
        } else {
            epilogue_pc_tiles<1, 2>(a, acc, co_wave, pw, lane, res8, pc, 0);
        }
    } else {
        epilogue_tiles<1, 2>(a, acc, co_wave, pw, lane, res8);
    }
#endif
}

// ------------------------------------------------------------------ dispatch
namespace {
bool flat_shape(const ConvArgs &a, FlatArgs &g, size_t &lds_bytes)
{
    const int wc = a.Cout == 64 ? 2 : 4, px = 64 * (4 / wc), pieces = a.Cin / 16 + 1;
    g.rows = a.KH == 1 ? px : a.sh == 1 ? px + 2 * (a.W + 1) : 4 * px + 2 * (a.Wo + 1);
    g.patch_bytes = ((g.rows + 1) * pieces + 63) / 64 * 1024;
    lds_bytes = g.patch_bytes + 512 + (a.pc ? kFlatTables : 0) + (a.sh == 2 ? (g.rows * 4 + 511) / 512 * 512 : 0);
    return lds_bytes <= 160 * 1024 && g.rows <= 0x7ff;
}
}  // namespace

static bool flat_takes(const ConvArgs &a, bool direct_ok)
{
    FlatArgs g;
    size_t lds_bytes;
    if (!direct_ok || a.frag_xor || a.in_xor || a.sh < 1 || a.sh > 2 || a.sw != a.sh || a.KH != a.KW || a.ph != a.KH / 2 || a.pw != a.KW / 2 || !a.vec_bias) return false;
    if (a.x_bytes >= 0x7fffff00u || a.wp_bytes >= 0x7fffff00u || a.M > 0x7fffffff - 256 || a.W > 4096 || a.Cout / 64 > 0xffff) return false;
    if (a.Cout % 128 != 0 && !(a.Cout == 64 && a.Cin == 64 && a.KH == 3 && a.sh == 1)) return false;
    const int c = a.Cin;
    if (a.KH == 3 ? c != 64 && c != 128 && c != 256 && c != 512 : a.KH != 1 || (c != 128 && c != 256 && c != 512 && (a.sh == 1 ? c != 1024 && c != 2048 : c != 64))) return false;
    return flat_shape(a, g, lds_bytes);
}

// A layer of 64 channels whose tiles are all on the chip at once, three to a compute unit.  Against two-dimensional tiles (there / here; smaller layers are level): 16, 20, 24
// and 31 images of 56 x 56 5.8 / 5.1, 8.1 / 5.6, 8.5 / 6.8, 8.8 / 7.0; 256 x 256 6.4 / 6.2, two of 200 x 200 8.5 / 7.1; with two to a unit, 300 x 300, 8.6 / 8.9; in two rounds
// 400 x 400 11.7 / 13.8.
static bool flat_one_round(const ConvArgs &a)
{
    FlatArgs g;
    size_t lds_bytes;
    return a.Cout == 64 && a.M > 45056 && a.M <= 768 * 128 && flat_shape(a, g, lds_bytes) && 3 * lds_bytes <= 160 * 1024;
}

// Every layer it takes but two kinds (microseconds the other kernel / this one, weights and maps cold in L2).  Those of few enough pixels for the
// few-pixel kernel: the rule and its figures stand beside it (conv_lat_before_flat).  Layers of 64 channels on large
// pictures go to the kernel that keeps their weights (conv_keep_applies) or to two-dimensional tiles, but for one round of this kernel's workgroups
// (flat_one_round).  The others: 3x3 of 256 channels on 14 x 14, 16 / 32 / 64 / 128 images 9.9 / 6.8, 11.4 / 7.4,
// 13.2 / 10.8, 22.5 / 18.9; of 512 on 7 x 7, 64 images 14.3 / 10.7; of 128 on 28 x 28, 9 / 64 images 8.4 / 5.5, 16.1 / 12.6; 256 -> 1024 on 14 x 14,
// 9 / 64 images 5.4 / 3.9, 13.0 / 9.5; 512 -> 256 on 28 x 28, 9 / 64 images 6.1 / 4.6, 16.1 / 14.1; 128 -> 512, 15.6 / 11.2; 1024 -> 512 and 512 -> 128
// within 4 % where they have 12544 and 50176 pixels, 9 % faster at 9408.  Stride 2, 64 images: 3x3 of 128 channels on 56 x 56 16.1 / 15.3, of 256 on
// 28 x 28 16.5 / 12.1, of 512 on 14 x 14 19.6 / 12.8 (and 128 images 26.6 / 23.9); 128 -> 256 on 28 x 28 11.2 / 8.2, 256 -> 512 on 14 x 14 12.4 / 8.6;
// 1x1, 64 -> 128 on 56 x 56 14.5 / 13.4, 256 -> 512 on 14 x 14 7.6 / 6.1.  A 1x1 patch of 2048 channels leaves room for one workgroup on a compute
// unit: 64 / 80 / 96 / 128 images of 7 x 7 (196, 248, 300, 392 workgroups) 10.4 / 8.0, 10.8 / 8.4, 14.4 / 13.7, 12.5 / 14.1: one round of them only.
bool conv_flat_applies(const ConvArgs &a, bool direct_ok)
{
    if (g_tuning.flat == 2) return false;
    if (g_tuning.flat == 1) return flat_takes(a, direct_ok);
    if (conv_lat_before_flat(a)) return false;
    if (g_tuning.tile >= 0 || g_tuning.stages || g_tuning.ksplit || g_tuning.deep_always || g_tuning.halo_always || g_tuning.halo_tile ||
        g_tuning.plane_always || g_tuning.lat || !flat_takes(a, direct_ok))
        return false;
    if (a.Cin == 2048 && (long long)(a.Cout / 128) * ((a.M + 63) / 64) > 256) return false;
    return a.pc || a.res_mode != 0 || g_tuning.no_plane || !conv_plane_applies(a) || flat_one_round(a);
}

hipError_t launch_conv_flat(const ConvArgs &args, hipStream_t st)
{
    ConvArgs a = args;
    FlatArgs g;
    size_t lds_bytes;
    if (!flat_takes(a, true) || !flat_shape(a, g, lds_bytes)) return hipErrorInvalidValue;
    const bool narrow = a.Cout == 64;
    if (!finish_args(a, narrow ? 64 : 128, narrow ? 128 : 64)) return hipErrorInvalidValue;
    a.div_howo = make_fast_div((unsigned)(a.Ho * a.Wo));
    a.div_wo = make_fast_div((unsigned)a.Wo);
    // What the eight L2s fetch: weights eight times and the input once, or the other way round as far as the channel tiles go.  (3x3 of 512
    // channels on 64 images of 7 x 7, 20.5 MB against 11 MB.)
    const double wt = a.wp_bytes, in = a.x_bytes;
    const bool by_pt = a.n_ct > 1 && wt * 8 + in > wt * std::max(8 / a.n_ct, 1) + in * std::min(a.n_ct, 8);
    g.sk = SkipMul{0, 0, 0};
    if (a.res_mode == 1 && a.res_dtype == 0) g.sk = make_skip_mul(a.res_mul, a.res_shift);
    const int form = a.pc ? 2 : a.rq_fast && a.epi_vec && (a.res_mode == 0 || g.sk.ok) ? requant_fits_byte(a) ? 5 : 1 : 0;
    const FastDiv by = make_fast_div((unsigned)(by_pt ? a.n_tiles / a.n_ct : a.n_ct));
    const FlatFirst f = {a.x, a.wp, a.bias, a.pc, a.M, a.in_cs, (unsigned)g.rows | (unsigned)(g.patch_bytes / 1024) << 11 | (unsigned)a.W << 19, by.mul,
                         (unsigned)a.n_ct | by.s1 << 16 | by.s2 << 24 | (by_pt ? 1u << 30 : 0u) | (a.res_mode ? 1u << 31 : 0u)};
    auto go = [&](auto kernel) -> hipError_t {
        if (lds_bytes > 64 * 1024) {
            const hipError_t e = allow_large_lds((const void *)kernel);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * a.per_xcd)), dim3(256), lds_bytes, st, f.x, f.wp, f.bias, f.pc, f.M, f.in_cs, f.shape, f.div_mul, f.tiles, a, g);
        return hipGetLastError();
    };
#define ICNN_FLAT(KK, NG, G, WC, S) \
    (form == 5 ? go(conv_flat_kernel<KK, NG, G, WC, 5, S>) : form == 1 ? go(conv_flat_kernel<KK, NG, G, WC, 1, S>) : form == 2 ? go(conv_flat_kernel<KK, NG, G, WC, 2, S>) : go(conv_flat_kernel<KK, NG, G, WC, 0, S>))
    // The closing layer of a basic block beside its projection's int32 sums: two products in place of the general 64-bit steps, and the sums requested
    // before the K loop in whole lines (64 images, 128 channels on 28 x 28 18.4 -> 15.6 us, 256 on 14 x 14 13.9 -> 11.6, 512 on 7 x 7 14.0 -> 11.4;
    // with each lane asking for its own half lines 15.7, 12.8 and 11.4).
    if (a.KH == 3 && a.sh == 1 && !narrow && !a.pc && skip_s32_fits(a) && lds_bytes + kFlatSums <= 160 * 1024) {
        lds_bytes += kFlatSums;
        switch (a.Cin) {
        case 64: return go(conv_flat_kernel<3, 9, 1, 4, 3, 1>);
        case 128: return go(conv_flat_kernel<3, 9, 2, 4, 3, 1>);
        case 256: return go(conv_flat_kernel<3, 9, 4, 4, 3, 1>);
        default: return go(conv_flat_kernel<3, 18, 4, 4, 3, 1>);
        }
    }
    if (a.KH == 3 && a.sh == 1) {
        switch (a.Cin) {
        case 64: return narrow ? ICNN_FLAT(3, 9, 1, 2, 1) : ICNN_FLAT(3, 9, 1, 4, 1);
        case 128: return ICNN_FLAT(3, 9, 2, 4, 1);
        case 256: return ICNN_FLAT(3, 9, 4, 4, 1);
        default: return ICNN_FLAT(3, 18, 4, 4, 1);
        }
    }
    if (a.KH == 3) {
        switch (a.Cin) {
        case 64: return ICNN_FLAT(3, 9, 1, 4, 2);
        case 128: return ICNN_FLAT(3, 9, 2, 4, 2);
        case 256: return ICNN_FLAT(3, 9, 4, 4, 2);
        default: return ICNN_FLAT(3, 18, 4, 4, 2);
        }
    }
    if (a.sh == 1) {
        switch (a.Cin) {
        case 128: return ICNN_FLAT(1, 1, 2, 4, 1);
        case 256: return ICNN_FLAT(1, 1, 4, 4, 1);
        case 512: return ICNN_FLAT(1, 2, 4, 4, 1);
        case 1024: return ICNN_FLAT(1, 4, 4, 4, 1);
        default: return ICNN_FLAT(1, 8, 4, 4, 1);
        }
    }
    // A projection's int32 sums, stored in whole lines (64 images: 64 -> 128 channels on 56 x 56 13.3 -> 7.3 us, 128 -> 256 on 28 x 28 8.8 -> 6.2,
    // 256 -> 512 on 14 x 14 6.3 -> 5.6).
    if (a.out_mode == 3 && a.res_mode == 0 && a.epi_vec && !a.pc) {
        lds_bytes += kFlatSums;
        switch (a.Cin) {
        case 64: return go(conv_flat_kernel<1, 1, 1, 4, 4, 2>);
        case 128: return go(conv_flat_kernel<1, 1, 2, 4, 4, 2>);
        case 256: return go(conv_flat_kernel<1, 1, 4, 4, 4, 2>);
        default: return go(conv_flat_kernel<1, 2, 4, 4, 4, 2>);
        }
    }
    switch (a.Cin) {
    case 64: return ICNN_FLAT(1, 1, 1, 4, 2);
    case 128: return ICNN_FLAT(1, 1, 2, 4, 2);
    case 256: return ICNN_FLAT(1, 1, 4, 4, 2);
    default: return ICNN_FLAT(1, 2, 4, 4, 2);
    }
#undef ICNN_FLAT
}

}  // namespace icnn
