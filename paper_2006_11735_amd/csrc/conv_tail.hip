// The end of a restoration network in one launch: two branches of one 48-channel input (3x3, 16 channels, beside 1x1, 32 channels; their
// outputs concatenated to 48) and the single-channel 3x3 layer behind them.  On a 2560 x 1600 frame the 48-channel tensor between the two
// is 197 MB: one launch wrote it and another read it back, 96 + 80 us of which the matrix cores worked 20.
//
//   tile     16 rows x 32 columns of the middle tensor; a work unit is a column strip of the picture from a given row downwards, taken
//            tile by tile, so that no row of the middle tensor is computed twice (but for the two above a unit's first tile, which one
//            wave redoes); two of the 32 columns are borders of the neighbouring strips, 30 are outputs (7 % more work)
//   patch    the 18 x 34 input pixels under a tile, in LDS, zeros outside the picture; double-buffered by direct-to-LDS copies
//   K loop   v_mfma_i32_16x16x64_i8: 16 channels x 16 pixels, so neither 16-channel branch slice is padded to 32 rows (the 32x32 shapes
//            spend 512 clocks per tile row where these take 320).  All weights live in registers (nine fragments).  K order is the
//            packed order (tap, channel): fragment f holds the 16-byte pieces 4 f .. 4 f + 3 of the 27 a pixel's taps have, one per
//            quarter wave; the pieces of a kernel row are neighbours in LDS, so all fragments but two lie at base + constant.
//            The 1x1 branch's operand (the centre tap) is fragment 3.
//   last     a 3x3 layer with one output channel is, per pixel of its input, nine dot products over 48 channels (one per tap) whose values
//            belong to nine output pixels.  The requantised bytes of a pixel are in the lanes just as the B operand of another 16x16x64
//            product needs them (channel 4 q + r of slice j in byte r of word j of quarter q; the tap weights' K order is laid
//            out to match): one product per 16 pixels gives all nine.  The three taps of a kernel row are then added across neighbouring
//            lanes (quarter q holds kernel row q), and the three kernel rows through a ring of rows in LDS.
//   rows     a wave owns two tile rows and deals a row's requantisation out between the next row's products (also across tiles), so
//            the values of a tile are complete one tile later and its outputs are stored two tiles later.
//
// Accumulators are int32 throughout and the arithmetic of each layer is that of its own launch, so results are the same bit for bit.
#include "conv_common.h"

#include <type_traits>

namespace icnn {

constexpr int kTailTH = 16, kTailTW = 32, kTailOut = kTailTW - 2;       // tile rows, columns, columns that are outputs
constexpr int kTailCin = 48;
constexpr int kTailPW = kTailTW + 2, kTailPH = kTailTH + 2;             // patch
constexpr int kTailRowB = kTailPW * kTailCin;
constexpr int kTailPieces = kTailPH * kTailPW * (kTailCin / 16);
constexpr int kTailCopies = (kTailPieces + 63) / 64;                    // wave-wide 1 KiB copies
constexpr int kTailCpw = (kTailCopies + 7) / 8;
constexpr int kTailPatch = kTailCopies * 1024;
constexpr int kTailRing = 64;                                           // rows of partial sums in LDS (four tiles), 4 x 32 words each
constexpr int kTailLds = 2 * kTailPatch + kTailRing * 4 * kTailTW * 4;
// a wave's fragment reads reach past its rows' last pixel by one 16-byte piece (meeting zero weights): inside the LDS allocation
static_assert(kTailCpw == 4, "a tile's copies are dealt out over the two rows of a wave, two each");
static_assert(kTailLds <= 160 * 1024 && kTailRowB * kTailPH + 64 <= kTailLds, "LDS");

struct TailArgs {
    int strips, tiles_y;             // per picture
    int n_tiles, per_wg;             // all tiles; tiles per workgroup
    FastDiv div_tpi, div_ty;         // / (strips * tiles_y), / tiles_y
};

// four accumulators (consecutive channels) -> their requantised bytes as one word.  QUICK: the 32-bit form (ConvArgs::rq24)
template <bool QUICK>
__device__ __forceinline__ int tail_word(const ConvArgs &a, const v4i &acc)
{
    if constexpr (QUICK) {
        int w = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t x = __umul24((uint32_t)med3_v0s(acc[r], a.t_hi), (uint32_t)a.mul) + (uint32_t)a.rnd;
            if (r == 0) w = (int)(x >> a.shift);
            else shift_into_byte(w, x, a.shift, r);
        }
        return w;
    } else {
        int v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (a.rq_fast) v[r] = clampi64(((int64_t)acc[r] * a.mul_hi + 0x80000000LL) >> 32, a.lo, a.hi);
            else v[r] = clampi64(rsr64((int64_t)acc[r] * a.mul, a.shift), a.lo, a.hi);
        }
        return pack_low_bytes(v[0], v[1], v[2], v[3]);
    }
}

// value of the neighbouring lane in a row of 16 lanes, where the two 16-lane rows of `lo` and `hi` are columns 0..15 and 16..31
__device__ __forceinline__ int from_left_lo(int lo) { return __builtin_amdgcn_update_dpp(0, lo, 0x111, 0xf, 0xf, false); }
__device__ __forceinline__ int from_left_hi(int lo, int hi)
{
    return __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, lo, 0x121, 0xf, 0xf, false), hi, 0x111, 0xf, 0xf, false);
}
__device__ __forceinline__ int from_right_lo(int lo, int hi)
{
    return __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, hi, 0x12f, 0xf, 0xf, false), lo, 0x101, 0xf, 0xf, false);
}
__device__ __forceinline__ int from_right_hi(int hi) { return __builtin_amdgcn_update_dpp(0, hi, 0x101, 0xf, 0xf, false); }

template <bool QUICK>
__global__ __launch_bounds__(512, 1) void conv_tail_kernel(const ConvArgs a, const ConvArgs b, const ConvArgs c, const TailArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr unsigned OOB = 0x80000000u;            // beyond any buffer this kernel accepts (< 2 GiB)
    constexpr int F = 7;                             // fragments of 64 k-values: 27 pieces of 16 and one of zeros
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const pbuf = lds;
    int *const ring = (int *)(lds + 2 * kTailPatch);

    const int tid = threadIdx.x, lane = tid & 63, quad = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.x_bytes, 0x00020000);

    // the workgroups of an XCD (blockIdx.x & 7) take neighbouring ranges of tiles
    const int wg = ((int)blockIdx.x & 7) * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);
    const int t_end = min((wg + 1) * g.per_wg, g.n_tiles);
    int t_next = wg * g.per_wg;
    if (t_next >= t_end) return;

    struct Visit { int n, y0, x0, ty, real; };      // real: not the warm-up above a unit's first tile
    auto visit_of = [&](int t) {
        Visit v;
        v.n = fast_div(t, g.div_tpi);
        const int r = t - v.n * g.strips * g.tiles_y;
        const int s = fast_div(r, g.div_ty);
        v.ty = r - s * g.tiles_y;
        v.y0 = v.ty * kTailTH;
        v.x0 = s * kTailOut - 1;
        v.real = 1;
        return v;
    };

    int p_rel[kTailCpw], p_yx[kTailCpw];
#pragma unroll
    for (int i = 0; i < kTailCpw; ++i) {
        const int q = (wave + 8 * i) * 64 + lane;
        const int pix = q / 3, slot = q - pix * 3;
        const int py = pix / kTailPW, px = pix - py * kTailPW;
        p_rel[i] = (py * a.W + px) * a.in_cs + slot * 16;
        p_yx[i] = ((q < kTailPieces ? py : 0x7fff) << 16) | px;
    }
    auto issue_copy = [&](auto i_tag, const Visit &v, int base, int bufi) {
        constexpr int i = decltype(i_tag)::value;
        const int e = wave + 8 * i;
        if (e < kTailCopies) {                       // wave-uniform
            const int py = p_yx[i] >> 16;
            const int iy = v.y0 - 1 + py, ix = v.x0 - 1 + (p_yx[i] & 0xffff);
            // (a warm-up only needs the pixels under its last two rows)
            const bool ok = ((unsigned)iy < (unsigned)a.H) & ((unsigned)ix < (unsigned)a.W) & (v.real || py >= kTailTH - 2);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(pbuf + bufi * kTailPatch + e * 1024), 16,
                                                     ok ? (unsigned)(base + p_rel[i]) : OOB, 0, 0, 0);
        }
    };
    auto patch_base = [&](const Visit &v) { return ((v.n * a.H + v.y0 - 1) * a.W + v.x0 - 1) * a.in_cs; };

    // the first tile, or the two rows above it where it is not a strip's first
    Visit cur = visit_of(t_next);
    if (cur.ty > 0) {
        cur.ty -= 1; cur.y0 -= kTailTH; cur.real = 0;
    } else {
        ++t_next;
    }
    {
        const int base = patch_base(cur);
        static_for<kTailCpw>([&](auto i_tag) { issue_copy(i_tag, cur, base, 0); });
    }

    // ---- weights.  Fragment f, matrix row (= channel) i = lane & 15, pieces 4 f + quad: in the packed order that is K step f, half quad >> 1,
    // and slot 32 * (quad & 1) + the row that holds channel i (i + 16) of a 32-channel chunk.
    const int prow = (col & 3) + 8 * (col >> 2);
    const unsigned woff = (unsigned)((quad >> 1) * 1024 + ((quad & 1) * 32 + prow) * 16);
    v4i wa[F], wb[2], wt;
#pragma unroll
    for (int f = 0; f < F; ++f) wa[f] = *(const v4i *)(a.wp + f * kChunkBytes + woff);
    wb[0] = *(const v4i *)(b.wp + woff);
    wb[1] = *(const v4i *)(b.wp + woff + 4 * 16);
    {
        // tap weights: matrix row 4 kh + kw, K position 16 q + 4 j + r = channel 4 q + r of slice j of the middle tensor
        const int kh = col >> 2, kw = col & 3;
        const bool tap = kh < 3 && kw < 3;
        int w[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int ch = (j == 0 ? a.out_co : b.out_co + (j - 1) * 16) + quad * 4;
            const int k = (tap ? kh * 3 + kw : 0) * kTailCin + (ch & ~15);
            const unsigned o = (unsigned)(k >> 6) * kChunkBytes + (unsigned)((k >> 5) & 1) * 1024u + (unsigned)(((k >> 4) & 1) * 512) + (unsigned)(ch & 15);
            w[j] = *(const int *)(c.wp + o);
            if (!tap) w[j] = 0;
        }
        wt = v4i{w[0], w[1], w[2], 0};
    }
    v4i bias[3];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        bias[0][r] = a.bias[quad * 4 + r];
        bias[1][r] = b.bias[quad * 4 + r];
        bias[2][r] = b.bias[16 + quad * 4 + r];
    }
    const int bias_c = c.bias[0];

    // fragment read bases within a patch, first row of this wave: pieces 9 dy .. 9 dy + 8 are neighbours, fragments 2 and 4 straddle two kernel rows
    const int lin = 2 * wave * kTailRowB + col * kTailCin + quad * 16;
    const int lin2 = lin + (quad == 0 ? 8 * 16 : kTailRowB - 16);
    const int lin4 = lin + (quad < 2 ? kTailRowB + 7 * 16 : 2 * kTailRowB - 2 * 16);
    auto frag = [&](const uint8_t *P, auto f_tag, int j, int u) {        // tile row j of the wave, pixels 16 u ..
        constexpr int f = decltype(f_tag)::value;
        const int o = f == 2 ? lin2 : f == 4 ? lin4 : lin + (f < 2 ? f * 64 : f == 3 ? kTailRowB + 3 * 16 : 2 * kTailRowB + (f == 5 ? 2 * 16 : 6 * 16));
        return *(const v4i *)(P + o + j * kTailRowB + u * 16 * kTailCin);
    };

    // ---- a finished row: its accumulators wait for the next row's K loop
    v4i pend[2][3] = {};
    int pend_m[2] = {0, 0}, pend_slot = 0;
    bool have = false;
    int word[2][3];
    auto finish_word = [&](auto k_tag) {             // k = 0 .. 5: slice k % 3 of pixels 16 (k / 3) ..
        constexpr int k = decltype(k_tag)::value, u = k / 3, s = k % 3;
        word[u][s] = tail_word<QUICK>(s == 0 ? a : b, pend[u][s]) & pend_m[u];
    };
    auto finish_row = [&]() {                        // the nine taps' products, kernel rows summed, into the ring
        v4i t[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) t[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wt, v4i{word[u][0], word[u][1], word[u][2], 0}, v4i{0, 0, 0, 0}, 0, 0, 0);
        asm volatile("s_nop 15" : "+v"(t[0]), "+v"(t[1]));
        const int h0 = from_left_lo(t[0][0]) + t[0][1] + from_right_lo(t[0][2], t[1][2]);
        const int h1 = from_left_hi(t[0][0], t[1][0]) + t[1][1] + from_right_hi(t[1][2]);
        if (have) {
            int *const r = ring + ((pend_slot & (kTailRing - 1)) * 4 + quad) * kTailTW + col;
            r[0] = h0;
            r[16] = h1;
        }
    };

    // ---- outputs of visit v (number vn): rows y0 - 1 .. y0 + 14, and y0 + 15 where that is the picture's last
    const bool thin32 = c.out_mode != 3 && c.rq_fast && (c.res_mode == 0 || c.res_fast);
    const int orow = tid >> 5, ocol = tid & 31;
    auto out_pixel = [&](const Visit &v, int r, size_t &p) {
        const int y = v.y0 - 1 + r, x = v.x0 + ocol;
        p = ((size_t)v.n * a.H + y) * a.W + x;
        return v.real && y >= 0 && y < a.H && ocol >= 1 && ocol <= kTailOut && x < a.W;
    };
    auto fetch_res = [&](const Visit &v, int r) {
        size_t p;
        return c.res_mode != 0 && out_pixel(v, r, p) ? load_elem(c.res, p * c.res_cs, c.res_dtype) : 0;
    };
    auto emit = [&](const Visit &v, int vn, int r, int res) {
        size_t p;
        if (!out_pixel(v, r, p)) return;
        const int y = v.y0 - 1 + r;
        const int s = vn * kTailTH - 1 + r;          // ring row of picture row y
        auto part = [&](int ds, int kh) { return ring[(((s + ds) & (kTailRing - 1)) * 4 + kh) * kTailTW + ocol]; };
        int sum = part(0, 1);
        if (y > 0) sum += part(-1, 0);
        if (y + 1 < a.H) sum += part(1, 2);
        const size_t oo = p * c.out_cs + c.out_co;
        epilogue_one(c, sat32((int64_t)sum + bias_c), res, oo, thin32);
    };
    auto emit_visit = [&](const Visit &v, int vn, int res) {
        emit(v, vn, orow, res);
        if (v.ty == g.tiles_y - 1 && v.y0 + kTailTH == a.H && tid < 32) emit(v, vn, kTailTH, fetch_res(v, kTailTH));
    };

    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    Visit v1 = cur, v2 = cur;                        // the visits one and two before the current one
    v1.real = v2.real = 0;
    int buf = 0, vn = 0;
    for (;; ++vn) {
        const bool more = t_next < t_end;
        Visit nxt = cur;
        if (more) nxt = visit_of(t_next++);
        const int nbase = patch_base(nxt);
        const int res2 = fetch_res(v2, orow);
        const uint8_t *const P = pbuf + buf * kTailPatch;
        const bool active = cur.real || wave == 7;
        if (active) {
            int m[2];
            m[0] = (unsigned)(cur.x0 + col) < (unsigned)a.W ? -1 : 0;
            m[1] = (unsigned)(cur.x0 + 16 + col) < (unsigned)a.W ? -1 : 0;
            static_for<2>([&](auto j_tag) {
                constexpr int j = decltype(j_tag)::value;
                v4i acc[2][3];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int s = 0; s < 3; ++s) acc[u][s] = bias[s];
                v4i B[2][2];
#pragma unroll
                for (int u = 0; u < 2; ++u) B[0][u] = frag(P, std::integral_constant<int, 0>{}, j, u);
                static_for<F>([&](auto f_tag) {
                    constexpr int f = decltype(f_tag)::value, S = f & 1;
                    if constexpr (f + 1 < F) {
#pragma unroll
                        for (int u = 0; u < 2; ++u) B[S ^ 1][u] = frag(P, std::integral_constant<int, f + 1>{}, j, u);
                    }
                    if constexpr (f % 3 == 0 && j * 2 + f / 3 < kTailCpw && f < 6) {      // f = 0, 3: copies 2 j, 2 j + 1
                        if (more) issue_copy(std::integral_constant<int, j * 2 + f / 3>{}, nxt, nbase, buf ^ 1);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[f], B[S][u], acc[u][0], 0, 0, 0);
                    if constexpr (f == 3) {
#pragma unroll
                        for (int s = 0; s < 2; ++s)
#pragma unroll
                            for (int u = 0; u < 2; ++u) acc[u][1 + s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wb[s], B[S][u], acc[u][1 + s], 0, 0, 0);
                    }
                    if constexpr (f < 6) finish_word(f_tag);
                    else finish_row();
                    __builtin_amdgcn_sched_barrier(0);
                });
                // between the last product and the first reader (hand-written instructions, which the compiler does not keep apart)
                asm volatile("s_nop 15" : "+v"(acc[0][0]), "+v"(acc[1][0]), "+v"(acc[0][1]), "+v"(acc[1][1]), "+v"(acc[0][2]), "+v"(acc[1][2]));
                const bool rowok = cur.y0 + 2 * wave + j < a.H;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int s = 0; s < 3; ++s) pend[u][s] = acc[u][s];
                    pend_m[u] = rowok ? m[u] : 0;
                }
                pend_slot = vn * kTailTH + 2 * wave + j;
                have = true;
            });
        } else if (more) {
            static_for<kTailCpw>([&](auto i_tag) { issue_copy(i_tag, nxt, nbase, buf ^ 1); });
        }
        emit_visit(v2, vn - 2, res2);
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(0);                          // the next patch has landed (this wave's copies of it)
        __builtin_amdgcn_s_waitcnt(0xC07F);          // and this wave's reads of this one and its ring rows are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        v2 = v1;
        v1 = cur;
        if (!more) break;
        cur = nxt;
        buf ^= 1;
    }
    // the last rows, and the outputs of the last two visits
    static_for<6>([&](auto k_tag) { finish_word(k_tag); });
    finish_row();
    const int res2 = fetch_res(v2, orow), res1 = fetch_res(v1, orow);
    __syncthreads();
    emit_visit(v2, vn - 1, res2);
    emit_visit(v1, vn, res1);
#endif
}

// The layers of a launch: a, b as in conv_plane_twin_ok at 48 channels (16 outputs of 3x3, 32 of 1x1, unsigned bytes), c the single-channel
// 3x3 layer of their concatenation.
bool conv_tail_ok(const ConvArgs &a, const ConvArgs &b, const ConvArgs &c)
{
    if (!conv_plane_twin_ok(a, b) || a.KH != 3 || a.Cin != kTailCin || a.Cout != 16 || b.Cout != 32 || a.out_mode > 1 || b.out_mode > 1) return false;
    if (c.N != a.N || c.H != a.H || c.W != a.W || c.Ho != a.H || c.Wo != a.W || c.KH != 3 || c.KW != 3 || c.sh != 1 || c.sw != 1 || c.ph != 1 || c.pw != 1)
        return false;
    if (c.Cin != 48 || c.Cout != 1 || c.in_xor || c.frag_xor || c.pc || c.ksteps != 7) return false;
    // the two branches fill the 48 channels of the tensor between them
    return (a.out_co == 0 && b.out_co == 16) || (a.out_co == 32 && b.out_co == 0);
}

hipError_t launch_conv_tail(const ConvArgs &a, const ConvArgs &b, const ConvArgs &c, hipStream_t st)
{
    if (!conv_tail_ok(a, b, c)) return hipErrorInvalidValue;
    TailArgs g;
    g.strips = (a.W + kTailOut - 1) / kTailOut;
    g.tiles_y = (a.H + kTailTH - 1) / kTailTH;
    const long long tiles = (long long)g.strips * g.tiles_y * a.N;
    if (tiles < 1 || tiles > 0x7ffffff0LL) return hipErrorInvalidValue;
    g.n_tiles = (int)tiles;
    g.per_wg = (int)((tiles + 255) / 256);
    g.div_tpi = make_fast_div((unsigned)(g.strips * g.tiles_y));
    g.div_ty = make_fast_div((unsigned)g.tiles_y);
    const bool quick = a.rq24 && b.rq24;
    const auto kernel = quick ? conv_tail_kernel<true> : conv_tail_kernel<false>;
    const hipError_t e = allow_large_lds((const void *)kernel);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(256), dim3(512), kTailLds, st, a, b, c, g);
    return hipGetLastError();
}

}  // namespace icnn
