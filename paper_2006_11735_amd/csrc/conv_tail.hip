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
//   rows     sixteen waves own a tile row each and deal its requantisation out between the products of their row of the next tile, so the
//            values of a tile are complete one tile later and its outputs are stored two tiles later.  What bounds the kernel is
//            instruction issue (110 vector instructions per row, of which 72 requantise), hence four waves per SIMD: under rocprofv3 a
//            SIMD issues 0.129 vector instructions per clock, 52 % of what 64 lanes on 16 ALUs allow, beside 21 % of matrix work; LDS bank
//            conflicts (the 48-byte pixels of the fragment reads) hold 16 % of the clocks.
//
// Measured inside the network: 91 + 80 us for the two launches on 2560 x 1600, 80 us here (24 us on 720 x 1280).
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
constexpr int kTailCpw = (kTailCopies + 15) / 16;
constexpr int kTailPatch = kTailCopies * 1024;
constexpr int kTailRing = 64;                                           // rows of partial sums in LDS (four tiles), 4 x 32 words each
constexpr int kTailLds = 2 * kTailPatch + kTailRing * 4 * kTailTW * 4 + 48 * 4;
// a wave's fragment reads reach past its rows' last pixel by one 16-byte piece (meeting zero weights): inside the LDS allocation
static_assert(kTailCpw == 2, "a wave issues its copies at two places of its row");
static_assert(kTailLds <= 160 * 1024 && kTailRowB * kTailPH + 64 <= kTailLds, "LDS");

struct TailRequant { int mul, rnd, t_hi, shift, mul_hi, rq_fast, lo, hi; };      // of a branch, as in ConvArgs
struct TailArgs {
    const uint8_t *x, *wa, *wb, *wc, *res;
    const int32_t *bias_a, *bias_b, *bias_c;
    uint8_t *out;
    unsigned x_bytes, res_bytes, out_bytes;
    int H, W, in_cs, co_a, co_b;
    TailRequant a, b;
    // the last layer's 32-bit epilogue (QUICK): a skip operand joins before (pre = -1) or after (post = -1) requantisation, or there is none
    int res_cs, out_cs, out_co, res_mul, res_shift, pre, post, mul_hi, lo, hi;
    int strips, tiles_y;             // per picture
    int n_tiles, per_wg;             // all tiles; tiles per workgroup
    FastDiv div_tpi, div_ty;         // / (strips * tiles_y), / tiles_y
};

// four accumulators (consecutive channels) -> their requantised bytes as one word.  QUICK: the 32-bit form (ConvArgs::rq24)
template <bool QUICK>
__device__ __forceinline__ int tail_word(const TailRequant &a, const v4i &acc)
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
            if (a.rq_fast) v[r] = min(max((int)(((int64_t)acc[r] * a.mul_hi + 0x80000000LL) >> 32), a.lo), a.hi);
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

// QUICK: both branches by the 32-bit requantisation form and the last layer by TailArgs' epilogue; else `c` has the last layer's.
template <bool QUICK>
__global__ __launch_bounds__(1024) void conv_tail_kernel(const TailArgs g, const ConvArgs c)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr unsigned OOB = 0x80000000u;            // beyond any buffer this kernel accepts (< 2 GiB)
    constexpr int F = 7;                             // fragments of 64 k-values: 27 pieces of 16 and one of zeros
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const pbuf = lds;
    int *const ring = (int *)(lds + 2 * kTailPatch);
    int *const bias = ring + kTailRing * 4 * kTailTW;        // of the 16 + 32 branch channels

    const int tid = threadIdx.x, lane = tid & 63, quad = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)g.x, 0, g.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_res = __builtin_amdgcn_make_buffer_rsrc((void *)g.res, 0, g.res_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc((void *)g.out, 0, g.out_bytes, 0x00020000);

    // the workgroups of an XCD (blockIdx.x & 7) take neighbouring ranges of tiles
    const int wg = ((int)blockIdx.x & 7) * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);
    const int t_end = min((wg + 1) * g.per_wg, g.n_tiles);
    int t_next = wg * g.per_wg;
    if (t_next >= t_end) return;

    struct Visit { int row0, y0, x0, real; };       // picture's first row among all pictures' rows; real: not the warm-up above a unit's first tile
    auto visit_of = [&](int t) {
        Visit v;
        const int n = fast_div(t, g.div_tpi);
        const int r = t - n * g.strips * g.tiles_y;
        const int s = fast_div(r, g.div_ty);
        v.row0 = n * g.H;
        v.y0 = (r - s * g.tiles_y) * kTailTH;
        v.x0 = s * kTailOut - 1;
        v.real = 1;
        return v;
    };

    int p_rel[kTailCpw], p_yx[kTailCpw];
#pragma unroll
    for (int i = 0; i < kTailCpw; ++i) {
        const int q = (wave + 16 * i) * 64 + lane;
        const int pix = q / 3, slot = q - pix * 3;
        const int py = pix / kTailPW, px = pix - py * kTailPW;
        p_rel[i] = (py * g.W + px) * g.in_cs + slot * 16;
        p_yx[i] = ((q < kTailPieces ? py : 0x7fff) << 16) | px;
    }
    auto issue_copy = [&](auto i_tag, const Visit &v, int base, int bufi) {
        constexpr int i = decltype(i_tag)::value;
        const int e = wave + 16 * i;
        if (e < kTailCopies) {                       // wave-uniform
            const int py = p_yx[i] >> 16;
            const int iy = v.y0 - 1 + py, ix = v.x0 - 1 + (p_yx[i] & 0xffff);
            // (a warm-up only needs the pixels under its last two rows)
            const bool ok = ((unsigned)iy < (unsigned)g.H) & ((unsigned)ix < (unsigned)g.W) & (v.real || py >= kTailTH - 2);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(pbuf + bufi * kTailPatch + e * 1024), 16,
                                                     ok ? (unsigned)(base + p_rel[i]) : OOB, 0, 0, 0);
        }
    };
    auto patch_base = [&](const Visit &v) { return ((v.row0 + v.y0 - 1) * g.W + v.x0 - 1) * g.in_cs; };

    // the first tile, or the two rows above it where it is not a strip's first
    Visit cur = visit_of(t_next);
    if (cur.y0 > 0) {
        cur.y0 -= kTailTH; cur.real = 0;
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
    for (int f = 0; f < F; ++f) wa[f] = *(const v4i *)(g.wa + f * kChunkBytes + woff);
    wb[0] = *(const v4i *)(g.wb + woff);
    wb[1] = *(const v4i *)(g.wb + woff + 4 * 16);
    {
        // tap weights: matrix row 4 kh + kw, K position 16 q + 4 j + r = channel 4 q + r of slice j of the middle tensor
        const int kh = col >> 2, kw = col & 3;
        const bool tap = kh < 3 && kw < 3;
        int w[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int ch = (j == 0 ? g.co_a : g.co_b + (j - 1) * 16) + quad * 4;
            const int k = (tap ? kh * 3 + kw : 0) * kTailCin + (ch & ~15);
            const unsigned o = (unsigned)(k >> 6) * kChunkBytes + (unsigned)((k >> 5) & 1) * 1024u + (unsigned)(((k >> 4) & 1) * 512) + (unsigned)(ch & 15);
            w[j] = *(const int *)(g.wc + o);
            if (!tap) w[j] = 0;
        }
        wt = v4i{w[0], w[1], w[2], 0};
    }
    if (tid < 48) bias[tid] = tid < 16 ? g.bias_a[tid] : g.bias_b[tid - 16];
    const int bias_c = g.bias_c[0];

    // fragment read bases within a patch, this wave's row: pieces 9 dy .. 9 dy + 8 are neighbours, fragments 2 and 4 straddle two kernel rows
    const int lin = wave * kTailRowB + col * kTailCin + quad * 16;
    const int lin2 = lin + (quad == 0 ? 8 * 16 : kTailRowB - 16);
    const int lin4 = lin + (quad < 2 ? kTailRowB + 7 * 16 : 2 * kTailRowB - 2 * 16);
    auto frag = [&](const uint8_t *P, auto f_tag, int u) {               // pixels 16 u .. of the row
        constexpr int f = decltype(f_tag)::value;
        const int o = f == 2 ? lin2 : f == 4 ? lin4 : lin + (f < 2 ? f * 64 : f == 3 ? kTailRowB + 3 * 16 : 2 * kTailRowB + (f == 5 ? 2 * 16 : 6 * 16));
        return *(const v4i *)(P + o + u * 16 * kTailCin);
    };

    // ---- a finished row: its accumulators wait for the next row's K loop
    v4i pend[2][3] = {};
    int pend_m[2] = {0, 0}, pend_slot = 0;
    bool have = false;
    int word[2][3];
    auto finish_word = [&](auto k_tag) {             // k = 0 .. 5: slice k % 3 of pixels 16 (k / 3) ..
        constexpr int k = decltype(k_tag)::value, u = k / 3, s = k % 3;
        word[u][s] = tail_word<QUICK>(s == 0 ? g.a : g.b, pend[u][s]) & pend_m[u];
    };
    auto finish_row = [&]() {                        // the nine taps' products, those of a kernel row summed, into the ring
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

    // ---- outputs of visit v (number vn): rows y0 - 1 .. y0 + 14 (two per wave of the first half), and y0 + 15 where that is the picture's last
    const int orow = tid >> 5, ocol = tid & 31;
    const bool ocol_ok = ocol >= 1 && ocol <= kTailOut;
    auto out_pixel = [&](const Visit &v, int r) {   // its index, or -1
        const int y = v.y0 - 1 + r, x = v.x0 + ocol;
        const bool ok = v.real && ocol_ok && (unsigned)y < (unsigned)g.H && x < g.W;
        return ok ? (v.row0 + y) * g.W + x : -1;
    };
    auto fetch_res = [&](const Visit &v, int r) -> int {
        const int p = out_pixel(v, r);
        if constexpr (QUICK) return __builtin_amdgcn_raw_buffer_load_b8(rs_res, p >= 0 ? (unsigned)(p * g.res_cs) : OOB, 0, 0);
        else return p >= 0 && c.res_mode != 0 ? load_elem(c.res, (size_t)p * c.res_cs, c.res_dtype) : 0;
    };
    auto emit = [&](const Visit &v, int vn, int r, int res) {
        const int p = out_pixel(v, r);
        const int y = v.y0 - 1 + r;
        const int s = vn * kTailTH - 1 + r;          // ring row of picture row y
        auto part = [&](int ds, int kh) { return ring[(((s + ds) & (kTailRing - 1)) * 4 + kh) * kTailTW + ocol]; };
        const int above = part(-1, 0), here = part(0, 1), below = part(1, 2);
        const int sum = here + (y > 0 ? above : 0) + (y + 1 < g.H ? below : 0);
        if constexpr (QUICK) {
            const int skip = (int)(((uint32_t)res * (uint32_t)g.res_mul + (uint32_t)((1 << g.res_shift) >> 1)) >> g.res_shift);
            const int ti = sat32((int64_t)sum + bias_c + (skip & g.pre));
            const int q = __builtin_elementwise_add_sat((int)(((int64_t)ti * g.mul_hi + 0x80000000LL) >> 32), skip & g.post);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)min(max(q, g.lo), g.hi), rs_out, p >= 0 ? (unsigned)(p * g.out_cs + g.out_co) : OOB, 0, 0);
        } else if (p >= 0) {
            epilogue_one(c, sat32((int64_t)sum + bias_c), res, (size_t)p * c.out_cs + c.out_co, false);
        }
    };
    auto emit_visit = [&](const Visit &v, int vn, int res) {
        if (!v.real) return;
        if (wave < 8) emit(v, vn, orow, res);
        else if (wave == 8 && v.y0 + kTailTH == g.H && lane < 32) emit(v, vn, kTailTH, res);
    };
    // the skip operand of this lane's output of visit v
    auto visit_res = [&](const Visit &v) -> int { return wave < 9 ? fetch_res(v, wave < 8 ? orow : kTailTH) : 0; };

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
        const int res2 = visit_res(v2);
        const uint8_t *const P = pbuf + buf * kTailPatch;
        if (cur.real || wave >= 14) {
            v4i acc[2][3];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int s = 0; s < 3; ++s) acc[u][s] = *(const v4i *)(bias + s * 16 + quad * 4);
            v4i B[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u) B[0][u] = frag(P, std::integral_constant<int, 0>{}, u);
            static_for<F>([&](auto f_tag) {
                constexpr int f = decltype(f_tag)::value, S = f & 1;
                if constexpr (f + 1 < F) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) B[S ^ 1][u] = frag(P, std::integral_constant<int, f + 1>{}, u);
                }
                if constexpr (f == 0 || f == 3) {
                    if (more) issue_copy(std::integral_constant<int, f / 3>{}, nxt, nbase, buf ^ 1);
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
            const bool rowok = cur.y0 + wave < g.H;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int s = 0; s < 3; ++s) pend[u][s] = acc[u][s];
                pend_m[u] = rowok && (unsigned)(cur.x0 + 16 * u + col) < (unsigned)g.W ? -1 : 0;
            }
            pend_slot = vn * kTailTH + wave;
            have = true;
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
    const int res2 = visit_res(v2), res1 = visit_res(v1);
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
    g.x = a.x; g.x_bytes = a.x_bytes; g.wa = a.wp; g.wb = b.wp; g.wc = c.wp;
    g.bias_a = a.bias; g.bias_b = b.bias; g.bias_c = c.bias;
    g.H = a.H; g.W = a.W; g.in_cs = a.in_cs; g.co_a = a.out_co; g.co_b = b.out_co;
    auto requant = [](const ConvArgs &l) { return TailRequant{l.mul, l.rnd, l.t_hi, l.shift, l.mul_hi, l.rq_fast, l.lo, l.hi}; };
    g.a = requant(a); g.b = requant(b);
    g.res = (const uint8_t *)c.res; g.out = (uint8_t *)c.out;
    g.res_cs = c.res_cs; g.out_cs = c.out_cs; g.out_co = c.out_co;
    g.res_mul = c.res_mode ? c.res_mul : 0; g.res_shift = c.res_mode ? c.res_shift : 0;
    g.pre = c.res_mode == 1 ? -1 : 0; g.post = c.res_mode == 2 ? -1 : 0;
    g.mul_hi = c.mul_hi; g.lo = c.lo; g.hi = c.hi;
    const long long res_bytes = c.res_mode ? (long long)c.M * c.res_cs : 0, out_bytes = (long long)c.M * c.out_cs;
    g.res_bytes = (unsigned)res_bytes; g.out_bytes = (unsigned)out_bytes;
    g.strips = (a.W + kTailOut - 1) / kTailOut;
    g.tiles_y = (a.H + kTailTH - 1) / kTailTH;
    const long long tiles = (long long)g.strips * g.tiles_y * a.N;
    if (tiles < 1 || tiles > 0x7ffffff0LL) return hipErrorInvalidValue;
    g.n_tiles = (int)tiles;
    g.per_wg = (int)((tiles + 255) / 256);
    g.div_tpi = make_fast_div((unsigned)(g.strips * g.tiles_y));
    g.div_ty = make_fast_div((unsigned)g.tiles_y);
    const bool quick = a.rq24 && b.rq24 && c.out_mode <= 1 && c.rq_fast && (c.res_mode == 0 || (c.res_fast && c.res_dtype == 0)) &&
                       res_bytes < 0x7fffff00LL && out_bytes < 0x7fffff00LL;
    const auto kernel = quick ? conv_tail_kernel<true> : conv_tail_kernel<false>;
    const hipError_t e = allow_large_lds((const void *)kernel);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(256), dim3(1024), kTailLds, st, g, c);
    return hipGetLastError();
}

}  // namespace icnn
