// First layer of a classification network as ONE kernel: strided convolution of a raw picture (cin <= 4, kernel up
// to 8 pixels wide, stride 2), BReLU / requantisation (Sections 3.1, 3.2.1, 3.4.1), then the 3x3 / stride 2 /
// padding 1 max-pool that follows it.  Layer by layer the convolution writes its output (51 MB for a ResNet stem at
// batch 64), the pool reads it back, and the picture is first copied into a padded 4-channel tensor; here a wave keeps
// the convolution's rows in its accumulators and stores only the pooled ones.
//
// A wave's work is a strip of 14 pooled columns and some pooled rows of one picture, and it needs no other wave: no
// barrier, every wave at its own place.  14 pooled columns are 29 convolution columns (of the 32 of a matrix instruction)
// and 64 picture columns, one load per picture row.  Vector work bounds the kernel, so the order is the one with least of it:
//
//   picture  a row is one dword per pixel (channels padded to 4, "- 128" applied, zeros outside the picture), in LDS for
//            as long as it is needed: a ring of four groups of four rows, the group a pooled row further on travelling
//            meanwhile
//   conv     D[cout][column] with v_mfma_i32_32x32x32_i8, one K block of 32 per kernel row: eight pixels of four channels
//            (the packed weights of a small-cin layer have exactly this order, zeros in the padding).  The weights stay in
//            registers, and a picture row's fragment is read once for the two convolution rows a pooled row advances by
//   pool     down the columns on the sums themselves, one three-way maximum per output of two convolution rows (a
//            requantisation does not decrease, so it may follow the maximum); then half as many values as the convolution
//            has are requantised, go to LDS as bytes, and are pooled along the row, 16 channels of a pixel per lane
//
// Only the first convolution row of a strip is computed twice (once for the strip above).
//
// 64 pictures of 224 x 224 x 3, 64 channels of 7 x 7: 31 us in tiles of 7 x 8 pooled pixels behind barriers, with all convolution bytes in LDS and
// all of them requantised, 19 to 20 us so (nine pictures 8.5 -> 7.1, one 8.3 -> 4.5 us).  A SIMD's two waves take 28000 clocks: 5700 up to
// the first product (weights, kernel arguments, twelve picture rows), 13300 of matrix instructions, 12000 of vector ones.  Dealing the
// requantisation out between the products would hide it, but its operands, the sums being made and the weights are more registers than two
// waves have; with one chunk of channels a wave and three waves to a SIMD it is no faster (21.7 us), the picture being prepared twice.
#include "conv_common.h"

#include <type_traits>

namespace icnn {

constexpr int kStemPW = 14;                                  // pooled columns of a strip
constexpr int kStemMaxRows = 16;                             // pooled rows of a strip, at most
constexpr int kStemRing = 16 * 64 * 4 + 64;                  // picture rows of a wave, and what the unused columns read beyond the last
constexpr int kStemBytes = 32 * (64 + 16);                   // convolution bytes of a wave: rows 20 or 12 banks apart

struct StemArgs {
    int Hp, Wp;                 // pooled size
};

// CG: chunks of 32 channels that a wave computes, all of them or one; KR: kernel rows (packed weights beyond the kernel's are taken as zeros); FORM: 1 requantisation as a product's high word
// (rq_fast), 0 any one of one pair per layer, 2 per output channel (the packed parameters in LDS).  units: strips of all pictures, a strip's number being
// (picture * segs + segment) * strips + strip, times the waves that share one.
template <int CG, int KR, int FORM>
__global__ __launch_bounds__(256, 2) void conv_stem_pool_kernel(const uint8_t *x, const uint8_t *weights, const int H, const int W, const int in_cs,
                                                                const int units, const int strips, const int segs, const unsigned strips_mul,
                                                                const unsigned segs_mul, const unsigned packed, const unsigned pads,
                                                                const ConvArgs a, const StemArgs g)
{
    constexpr int ROW_PITCH = CG * 32 + 16;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t *const ring = lds + wave * (kStemRing + kStemBytes);
    uint8_t *const cbuf = ring + kStemRing;
    int32_t *const pct = (int32_t *)(lds + 4 * (kStemRing + kStemBytes));

    const int u = (int)blockIdx.x * 4 + wave, share = (int)(packed >> 18 & 1);       // share: two waves to a strip, a chunk each
    const int first = u & share, KH = (int)(packed >> 19), co = 32 * first;
    // ---- weights: [chunk][K step][half step] of a KiB, a kernel row each
    v4i wt[CG][KR];
    {
        auto row = [&](int c, int kh) {
            return *(const v4i *)(weights + (size_t)((first + c) * ((KH + 1) / 2 * kChunkBytes) + kh * 1024) + lane * 16);
        };
        if (KH == KR) {
#pragma unroll
            for (int c = 0; c < CG; ++c)
#pragma unroll
                for (int kh = 0; kh < KR; ++kh) wt[c][kh] = row(c, kh);
        } else {
#pragma unroll
            for (int c = 0; c < CG; ++c)
#pragma unroll
                for (int kh = 0; kh < KR; ++kh) wt[c][kh] = kh < KH ? row(c, kh) : v4i{0, 0, 0, 0};
        }
    }
    if constexpr (FORM == 2) {
        copy_pc_groups<256>(pct, a.pc, a.Cout / 16, tid);
        __syncthreads();
    }
    if (u >= units) return;
    const int strip = u >> share;

    const int q = fast_div_packed(strip, strips_mul, packed >> 10 & 1, packed >> 5 & 31);
    const int px0 = (strip - q * strips) * kStemPW;
    const int n = fast_div_packed(q, segs_mul, packed >> 16 & 1, packed >> 11 & 31);
    const int rows = (int)(packed & 31), py0 = (q - n * segs) * rows;
    int ph = (int)(pads & 0xffff), pw = (int)(pads >> 16);
    if (packed >> 17 & 1) { ph = a.ph; pw = a.pw; }

    // ---- picture rows: group b is rows iy0 + 4 b to iy0 + 4 b + 3, a lane per column
    const int iy0 = 4 * py0 - 2 - ph, ix = 4 * px0 - 2 - pw + lane;
    const bool col_ok = (unsigned)ix < (unsigned)W;
    const uint32_t voff = col_ok ? (uint32_t)ix * (uint32_t)in_cs : 0u;
    uint32_t word[4][4];
    bool inner[4];
    typedef uint32_t u32_a1 __attribute__((aligned(1)));
    const uint32_t pitch = (uint32_t)W * (uint32_t)in_cs, early = 4u - (uint32_t)a.Cin;
    const uint32_t cmask = 0xffffffffu >> 8 * early;                     // the pixel's own channels
    const uint32_t keep = col_ok ? cmask : 0u, flip = a.in_xor;
    // A pixel is the upper bytes of one unaligned dword that ends with it.  Groups that lie in the picture take it like that.  In the
    // others a row outside reads the nearest one and counts as zeros, and the tensor's first dword, where a pixel's would begin before
    // the tensor, serves in its place (the tensor has four bytes at least).
    auto row_offset = [&](int iy) { return (uint32_t)(n * H + min(max(iy, 0), H - 1)) * pitch; };
    auto fetch = [&](uint32_t (&w)[4], bool &in, int b) {
        const int iy = iy0 + 4 * b;
        const uint32_t first = (uint32_t)(n * H + iy) * pitch;
        in = iy >= 0 && iy + 3 < H && first >= 4;
        if (in) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = *(const u32_a1 *)(x + (size_t)(first - early + (uint32_t)i * pitch) + voff);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t o = row_offset(iy + i) + voff;
                w[i] = *(const u32_a1 *)(x + (o - min(o, early)));
            }
        }
    };
    auto store = [&](const uint32_t (&w)[4], bool in, int b) {
        uint8_t *const p = ring + (b & 3) * 1024 + lane * 4;
        if (in) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(uint32_t *)(p + i * 256) = ((w[i] >> 8 * early) ^ flip) & keep;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int iy = iy0 + 4 * b + i;
                const uint32_t v = w[i] >> 8 * min(row_offset(iy) + voff, early);
                *(uint32_t *)(p + i * 256) = (unsigned)iy < (unsigned)H ? (v ^ flip) & keep : 0u;
            }
        }
    };
    // The unit keeps the order of a wave's LDS accesses; this keeps the compiler to it where lanes read what other lanes have stored.
    auto wave_order = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
#pragma unroll
    for (int b = 0; b < 4; ++b) fetch(word[b], inner[b], b);

    v16i bias[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) bias[c] = bias16(a.bias + co + c * 32 + half * 16);

    // bytes of columns outside the convolution's output are the pool's padding: zeros, written once
    const bool out_ok = (unsigned)(2 * px0 - 1 + col) < (unsigned)a.Wo;
    uint8_t *const mine = cbuf + col * ROW_PITCH + half * 16;
#pragma unroll
    for (int c = 0; c < CG; ++c) *(v4i *)(mine + c * 32) = v4i{0, 0, 0, 0};
    // the pooling lane's first pixel and channels
    constexpr int GPP = 2 * CG;                      // 16-channel groups per pixel
    const int pp = lane / GPP, cgp = lane - pp * GPP;
    const bool pool_ok = pp < kStemPW && px0 + pp < g.Wp;
    const uint8_t *const window = cbuf + 2 * min(pp, kStemPW - 1) * ROW_PITCH + cgp * 16;
    const size_t out_row = (size_t)g.Wp * a.out_cs;
    uint8_t *out = (uint8_t *)a.out + ((size_t)n * g.Hp + py0) * out_row + (size_t)px0 * a.out_cs + a.out_co + co;
    const size_t out_lane = (size_t)pp * a.out_cs + cgp * 16;

#pragma unroll
    for (int b = 0; b < 3; ++b) store(word[b], inner[b], b);
    wave_order();

    // fragment of picture row r (of four groups from b on): eight pixels from column 2 col on, this half of the wave four of them
    const uint8_t *const pix = ring + 8 * col + 16 * half;
    auto frag = [&](int b, int r) {
        const uint2 *p = (const uint2 *)(pix + ((b + (r >> 2)) & 3) * 1024 + (r & 3) * 256);
        const uint2 lo = p[0], hi = p[1];
        return v4i{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
    };

    // ---- the convolution row above the strip's first pair: pooled with it, if it exists
    v16i top[CG];
    if (py0 > 0) {
#pragma unroll
        for (int kh = 0; kh < KR; ++kh) {
            const v4i f = frag(0, kh);
#pragma unroll
            for (int c = 0; c < CG; ++c) top[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[c][kh], f, kh == 0 ? bias[c] : top[c], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) top[c][e] = -0x7fffffff - 1;
    }

    // ---- pooling along the row: a lane's three pixels, word d of its 16 channels.  Bytewise maximum in two halves, as 16-bit lanes: the
    // even bytes masked out of every loaded word; the odd bytes need no mask, because a lane's maximum is decided by its high byte (the
    // low byte only breaks ties) and only the high byte of the result is kept.
    auto read_window = [&](v4i (&w)[3]) {
#pragma unroll
        for (int jx = 0; jx < 3; ++jx) w[jx] = *(const v4i *)(window + jx * ROW_PITCH);
    };
    auto pool_word = [&](const v4i (&w)[3], int d) {
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        u16x2 me = __builtin_bit_cast(u16x2, (uint32_t)w[0][d] & 0x00ff00ffu), mo = __builtin_bit_cast(u16x2, (uint32_t)w[0][d]);
#pragma unroll
        for (int jx = 1; jx < 3; ++jx) {
            me = __builtin_elementwise_max(me, __builtin_bit_cast(u16x2, (uint32_t)w[jx][d] & 0x00ff00ffu));
            mo = __builtin_elementwise_max(mo, __builtin_bit_cast(u16x2, (uint32_t)w[jx][d]));
        }
        return (int)(__builtin_bit_cast(uint32_t, me) | (__builtin_bit_cast(uint32_t, mo) & 0xff00ff00u));
    };

    // ---- one pooled row: convolution rows 2 (py0 + s) and the next (local picture rows 2 and 4 on), the row before them in `above`;
    // the second one's sums are left in `below`.  The row before is pooled meanwhile.
    const int n_rows = min(rows, g.Hp - py0);
    // Group s + 3, requested a pooled row ago, is put into LDS (w_put); s + 4 is requested (w_get): requested and put within one row
    // it was waited for (19.6 us in place of 18.8).
    auto step = [&](const v16i (&above)[CG], v16i (&below)[CG], const uint32_t (&w_put)[4], bool in_put, uint32_t (&w_get)[4], bool &in_get, int s) {
        if (s + 2 < n_rows) fetch(w_get, in_get, s + 4);
        v16i acc[CG];
        v4i f = frag(s, 2), w3[3], o;
        read_window(w3);
        __builtin_amdgcn_sched_barrier(0);
        static_for<KR + 2>([&](auto rc) {
            constexpr int r = decltype(rc)::value + 2;
            v4i next = {};
            if constexpr (r < KR + 3) next = frag(s, r + 1);
            if constexpr (r - 2 < KR) {
#pragma unroll
                for (int c = 0; c < CG; ++c) acc[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[c][r - 2], f, r == 2 ? bias[c] : acc[c], 0, 0, 0);
            }
            if constexpr (r >= 4) {
#pragma unroll
                for (int c = 0; c < CG; ++c) below[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[c][r - 4], f, r == 4 ? bias[c] : below[c], 0, 0, 0);
            }
            if constexpr (r >= 4 && r < 8) {
                int v = pool_word(w3, r - 4);
                asm volatile("" : "+v"(v));          // here, between the products
                o[r - 4] = v;
            }
            f = next;
            __builtin_amdgcn_sched_barrier(0);
        });
        if (2 * (py0 + s) + 1 >= a.Ho) {             // the last pooled row of an odd convolution has no second row: the first again
            const v4i zero = {0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < CG; ++c) below[c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(zero, zero, acc[c], 0, 0, 0);
        }
        if (s > 0) {
            if (pool_ok) *(v4i *)(out + out_lane) = o;
            out += out_row;
        }
        mfma_drain(acc);
        mfma_drain(below);
        // ---- maximum of three rows, requantised
#pragma unroll
        for (int c = 0; c < CG; ++c) {
            v16i t;
#pragma unroll
            for (int e = 0; e < 16; ++e) t[e] = max(max(above[c][e], acc[c][e]), below[c][e]);
            v4i w;
            if constexpr (FORM == 2) w = epilogue_pc_bytes16<0>(a, t, v4i{0, 0, 0, 0}, pct + (2 * (first + c) + half) * kPcGroupInts);
            else if constexpr (FORM == 1) w = epilogue_bytes16<0, 1>(a, t, v4i{0, 0, 0, 0});
            else w = epilogue_bytes16<0>(a, t, v4i{0, 0, 0, 0});
            if (out_ok) *(v4i *)(mine + c * 32) = w;
        }
        if (s + 1 < n_rows) store(w_put, in_put, s + 3);
        wave_order();
    };
    // weights and biases are here before the loop: its first product would wait for the picture rows just requested too
#pragma unroll
    for (int c = 0; c < CG; ++c) {
#pragma unroll
        for (int kh = 0; kh < KR; ++kh) asm volatile("" : "+v"(wt[c][kh]));
        asm volatile("" : "+v"(bias[c]));
    }
    v16i bottom[CG];
    for (int s = 0; s < n_rows; s += 2) {
        step(top, bottom, word[3], inner[3], word[0], inner[0], s);
        if (s + 1 >= n_rows) break;
        step(bottom, top, word[0], inner[0], word[3], inner[3], s + 1);
    }
    v4i w3[3], o;
    read_window(w3);
#pragma unroll
    for (int d = 0; d < 4; ++d) o[d] = pool_word(w3, d);
    if (pool_ok) *(v4i *)(out + out_lane) = o;
}

// conv: a small-cin layer's arguments on the ORIGINAL picture (H, W, Cin, in_cs, KH, KW, pads, Ho, Wo as given;
// the packed weights in the small-cin order), out / out_cs / out_co describing the POOLED tensor.
hipError_t launch_conv_stem_pool(const ConvArgs &a, int hp, int wp, hipStream_t st)
{
    if (a.x_bytes < 4 || a.KH > 8 || a.KW > 8 || (a.Cout != 32 && a.Cout != 64) || a.ksteps != (a.KH * 32 + 63) / 64) return hipErrorInvalidValue;
    const StemArgs g = {hp, wp};
    const int strips = (wp + kStemPW - 1) / kStemPW;
    // Pooled rows per strip: as few as fill the chip's 2048 waves, for what a strip costs besides its rows (the row above, the first
    // picture rows, the weights: about a row and a half), in whole rounds.
    const long long across = (long long)strips * a.N;
    int rows = 1;
    double best = 0;
    for (int r = 1; r <= kStemMaxRows && r <= hp; ++r) {
        const long long waves = across * ((hp + r - 1) / r);
        const double cost = (double)((waves + 2047) / 2048) * (r + 1.5);
        if (r == 1 || cost < best) best = cost, rows = r;
    }
    const int segs = (hp + rows - 1) / rows;
    // Two waves share a strip of 64 channels where each can have a SIMD of its own (one picture of 224 x 224: 5.2 -> 4.4 us).  Beyond that the
    // picture rows and their fragments would be prepared twice on the same SIMDs (64 pictures: 18.8 -> 21.7 us).
    const bool share = a.Cout == 64 && 2 * across * segs <= 1024;
    const long long units = across * segs * (share ? 2 : 1);
    if (units < 1 || units > 0x7ffffff0LL) return hipErrorInvalidValue;
    const FastDiv ds = make_fast_div((unsigned)strips), dg = make_fast_div((unsigned)segs);
    const bool wide = a.ph > 0xffff || a.pw > 0xffff;
    const unsigned packed = (unsigned)rows | ds.s2 << 5 | ds.s1 << 10 | dg.s2 << 11 | dg.s1 << 16 | (unsigned)wide << 17 | (unsigned)share << 18 | (unsigned)a.KH << 19;
    const unsigned pads = wide ? 0u : (unsigned)a.ph | (unsigned)a.pw << 16;
    const size_t lds_bytes = 4 * (kStemRing + kStemBytes) + (a.pc ? (size_t)(a.Cout / 16) * kPcGroupInts * 4 : 0);
    auto go = [&](auto kernel) -> hipError_t {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((units + 3) / 4)), dim3(256), lds_bytes, st, a.x, a.wp, a.H, a.W, a.in_cs, (int)units, strips, segs,
                           ds.mul, dg.mul, packed, pads, a, g);
        return hipGetLastError();
    };
    auto rows_of = [&](auto cg, auto form) -> hipError_t {
        constexpr int CG = decltype(cg)::value;
        constexpr int FORM = decltype(form)::value;
        return a.KH <= 7 ? go(conv_stem_pool_kernel<CG, 7, FORM>) : go(conv_stem_pool_kernel<CG, 8, FORM>);
    };
    using std::integral_constant;
    auto form_of = [&](auto cg) -> hipError_t {
        if (a.pc) return rows_of(cg, integral_constant<int, 2>{});
        return a.rq_fast ? rows_of(cg, integral_constant<int, 1>{}) : rows_of(cg, integral_constant<int, 0>{});
    };
    return a.Cout == 64 && !share ? form_of(integral_constant<int, 2>{}) : form_of(integral_constant<int, 1>{});
}

}  // namespace icnn
