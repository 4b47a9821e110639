// A run of 3x3 / stride 1 / padding 1 layers of 64 channels (the body of the super-resolution network) as ONE launch:
// a workgroup takes a spatial tile of the picture through up to six layers with the middle tensors only in LDS.
//
// One such layer on a 256 x 256 plane is 1 us of matrix-core time behind a launch that costs 6 us (launch gap, cold
// weights, first patch).  Here a workgroup computes TH x TW pixels of the last of L layers and, before them, what those
// need of every earlier layer: layer l's region is TH + 2 (L - 1 - l) by TW + 2 (L - 1 - l) pixels.  The recomputed border
// costs matrix time (1.28 x for three layers on 16 x 16 tiles), and saves L - 1 launches; conv_chain_split() weighs the
// two and cuts a run of layers into launches.
//
//   buffers  two activation buffers in LDS, rows of 24 pixels, 80 bytes per pixel (64 channels and 16 bytes of padding:
//            sixteen consecutive pixels hit every bank once, and every tap of a fragment read is an immediate offset
//            from one address per lane).  Layer 0 reads the patch copied straight from memory, every later layer what the
//            layer before wrote; pixels outside the picture are stored as zeros = the next layer's padding.
//   weights  36 KiB per layer, double-buffered, copied two layers ahead: layer 1's in the prologue, waited for at its last barrier; layer l + 2's from
//            the start of layer l on, into the place of layer l's, waited for at the barrier that ends layer l.  A wave multiplies one
//            32-channel chunk (wave & 1) and keeps its 18 weight fragments in registers for the layer, so the K loop
//            reads one activation fragment (1 KiB of LDS) per matrix instruction; behind each product of its last group it reads the
//            next layer's fragment into the place of the one just used.
//   work     layer l's pixels in groups of 32 (row-major over the region); wave w takes groups (w >> 1), + 4, ...
//   barrier  one per layer
//
// Measured on 256 x 256: a launch of four layers of the network 14 to 15 us (16.8 before the layers' parameters left the loop: a scalar load in it was waited for with the
// fragments; before the next layer's weights came behind the last products, 1000 clocks a layer; and before the next group's first fragments came
// behind the last products of the one before); on uniform random bytes, which are slower, two, three and four layers
// 8.9, 12.3 and 16.1.  That the prologue waits for layer 1's weights as well changes none of these.  Of 31 k clocks 4.5 pass before the first layer, 7.3 in a layer of 16 groups: 36 matrix
// instructions a round of groups and SIMD at 50 clocks, 33 without the rest of the loop; seven other instructions to each.  Unrolling the loop by two
// saves sixteen moves a group and is slower (14.5 / 15.5 us: more code than the instruction buffers of eight waves take).
#include "conv_common.h"

#include <type_traits>

namespace icnn {

constexpr int kChainRP = 24;                       // pixels per buffer row
constexpr int kChainPix = 80;                      // bytes per pixel in LDS
constexpr int kChainRow = kChainRP * kChainPix;
constexpr int kChainF = 18;                        // K fragments of 32 (9 taps x 64 channels)
constexpr int kChainWBytes = 2 * kChainF * 1024;   // packed weights of one layer
constexpr int kChainA = kChainRP * kChainRow;      // the first layer's input, up to 24 rows
constexpr int kChainB = (kChainRP - 2) * kChainRow;
constexpr int kChainLds = 2 * kChainWBytes + kChainA + kChainB + kChainMaxLayers * 64 * 4;
static_assert(kChainLds <= 160 * 1024, "LDS");

// PIPE: every layer requantises as a product's high word (ConvArgs::rq_fast; the host checks).  A wave then deals the requantisation of
// its previous pixel group out between the matrix instructions of the next: the barrier per layer keeps the two waves of a SIMD in
// step, so both multiplied and then both requantised (a round of groups took 2.3 k clocks for 1.15 k of matrix work).
template <bool PIPE>
__global__ __launch_bounds__(512, 1) void conv_chain_kernel(const uint8_t *x, const uint8_t *first_weights, const int H, const int W, const int in_cs, const unsigned shape,
                                                            const int n_tiles, const int tiles_per_img, const unsigned mul_tpi, const int tiles_x,
                                                            const unsigned mul_tx, const unsigned shifts, const ChainArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr unsigned OOB = 0x80000000u;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const wbuf = lds;
    uint8_t *const bufA = lds + 2 * kChainWBytes;
    int32_t *const btab = (int32_t *)(bufA + kChainA + kChainB);      // (the other buffer begins at kChainA)

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = wave & 1;

    // the workgroups of an XCD (dealt round-robin) take a contiguous range of tiles: shared patch borders meet in one L2
    // (what the patch and the first layer's weights need are leading arguments, which are in registers when a wave starts)
    const int t = (int)(blockIdx.x & 7) * ((n_tiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (t >= n_tiles) return;
    const int TH = (int)(shape & 0xff), TW = (int)(shape >> 8 & 0xff), L = (int)(shape >> 16);
    const int n = fast_div_packed(t, mul_tpi, shifts & 0xff, shifts >> 8 & 0xff);
    const int r = t - n * tiles_per_img;
    const int ty = fast_div_packed(r, mul_tx, shifts >> 16 & 0xff, shifts >> 24);
    const int y0 = ty * TH, x0 = (r - ty * tiles_x) * TW;

    auto issue_weights = [&](int l, const uint8_t *wp) {
        const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)wp, 0, kChainWBytes, 0x00020000);
        uint8_t *const dst = wbuf + (l & 1) * kChainWBytes;
#pragma unroll
        for (int i = 0; i < (kChainWBytes / 1024 + 7) / 8; ++i) {
            const int e = wave + 8 * i;
            if (e < kChainWBytes / 1024)            // wave-uniform
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (__attribute__((address_space(3))) void *)(dst + e * 1024), 16,
                                                         (unsigned)(e * 1024 + lane * 16), 0, 0, 0);
        }
    };

    // the first layer's patch: LDS piece q (16 bytes) is slot q % 5 of buffer pixel q / 5; slot 4 is the pixel's padding
    const int ph = TH + 2 * L, pw = TW + 2 * L;
    const int ncopy = (ph * kChainRow + 1023) / 1024;
    constexpr int CPW = (kChainA / 1024 + 7) / 8;
    {
        // (every place inside the tensor lies below 2 GiB, OOB above)
        const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            const int e = wave + 8 * i;
            const int q = e * 64 + lane;
            const int pix = q / 5, slot = q - pix * 5;
            const int py = pix / kChainRP, px = pix - py * kChainRP;
            const int iy = y0 - L + py, ix = x0 - L + px;
            const bool ok = slot < 4 && py < ph && px < pw && (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W;
            const unsigned off = ok ? (unsigned)(((n * H + iy) * W + ix) * in_cs + slot * 16) : OOB;
            if (e < ncopy)                          // wave-uniform
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(bufA + e * 1024), 16, off, 0, 0, 0);
        }
    }
    issue_weights(0, first_weights);
    if (wave < L) {                                 // wave l: layer l's biases (and what inputs up to 255 add to them)
        int b = g.l[wave].bias[lane];
        if (g.l[wave].xin) b += 128 * g.l[wave].wsum[lane];
        btab[wave * 64 + lane] = b;
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);             // vmcnt(0), lgkmcnt(0)
    asm volatile("" ::: "memory");
    if (L > 1) issue_weights(1, g.l[1].wp);
    if (g.l[0].xin) {
        // inputs up to 255: the matrix cores take x - 128 (see ConvArgs::frag_xor); every lane flips the pieces it fetched
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            const int e = wave + 8 * i;
            if (e < ncopy) {
                v4i *p = (v4i *)(bufA + e * 1024 + lane * 16);
                *p = *p ^ (int)g.l[0].xin;
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    v4i w[kChainF];                                 // this wave's fragments of the layer
#pragma unroll
    for (int f = 0; f < kChainF; ++f) w[f] = *(const v4i *)(wbuf + (chunk * kChainF + f) * 1024 + lane * 16);
    asm volatile("" ::: "memory");
    // vmcnt(0), lgkmcnt(0): behind the barrier layer 1's weights are there for every wave, as layer 0's last groups read them
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // One layer.  Nothing of it is an argument of the kernel any more once its groups begin: a scalar load in there is waited for together with the
    // fragments on their way.  LAST: the tile goes to memory, else to the other buffer.
    auto layer = [&](auto last_tag, const int l) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        struct { int mul, shift, lo, hi, rq_fast, mul_hi, rq24, t_hi, rnd, rqh, rq_byte; } a = {g.l[l].mul, g.l[l].shift, g.l[l].lo, g.l[l].hi, g.l[l].rq_fast,
                                                                                     g.l[l].mul_hi, g.l[l].rq24, g.l[l].t_hi, g.l[l].rnd, g.l[l].rqh, 0};
        unsigned inv = g.inv[l], xout = LAST ? 0u : g.l[l + 1].xin;
        asm volatile("" : "+s"(a.lo), "+s"(a.hi), "+s"(a.mul_hi), "+s"(inv), "+s"(xout));
        if (l + 2 < L) issue_weights(l + 2, g.l[l + 2].wp);        // (its place's weights are in every wave's registers since the last barrier)
        auto next_weight = [&](int f) { return *(const v4i *)(wbuf + ((l + 1) & 1) * kChainWBytes + (chunk * kChainF + f) * 1024 + lane * 16); };
        const int src = (l & 1) ? kChainA : 0, dst = (l & 1) ? 0 : kChainA;      // bytes behind bufA
        const v16i bias = bias16(btab + l * 64 + chunk * 32 + half * 16);
        const int border = L - 1 - l;               // this layer's region reaches so far beyond the tile
        const int rw = TW + 2 * border, cnt = rw * (TH + 2 * border);
        const int ng = (cnt + 31) >> 5;
        uint8_t *const out = g.out + g.out_co + chunk * 32 + half * 16;
        const size_t out_cs = (size_t)g.out_cs;

        // pixel of this lane in group gr (idx below 2^9, inv below 2^16)
        auto locate = [&](int gr, int &oy, int &ox) {
            const int idx = min(gr * 32 + col, cnt - 1);
            oy = (int)(__umul24((unsigned)idx, inv) >> 16);
            ox = idx - __mul24(oy, rw);
        };
        constexpr int RING = 6;
        v4i bf[RING];
        const uint8_t *p = bufA;
        auto fetch = [&](const uint8_t *from, auto f_tag, auto slot_tag) __attribute__((always_inline)) {
            constexpr int f = decltype(f_tag)::value, T = f / 2;
            bf[decltype(slot_tag)::value % RING] = *(const v4i *)(from + (T / 3) * kChainRow + (T % 3) * kChainPix + (f & 1) * 32);
        };
        auto at = [&](int oy, int ox) { return (const uint8_t *)bufA + (src + half * 16 + __mul24(oy, kChainRow) + __mul24(ox, kChainPix)); };
        auto store = [&](int gr, int oy, int ox, v4i o) __attribute__((always_inline)) {
            const int iy = y0 - border + oy, ix = x0 - border + ox;
            const bool valid = (unsigned)(gr * 32 + col) < (unsigned)cnt;
            const bool inside = ((unsigned)iy < (unsigned)H) & ((unsigned)ix < (unsigned)W);
            if constexpr (LAST) {
                if (valid & inside) *(v4i *)(out + (size_t)((n * H + iy) * W + ix) * out_cs) = o;
            } else {
                if (!inside) o = v4i{0, 0, 0, 0};
                if (valid) *(v4i *)(bufA + (dst + chunk * 32 + half * 16 + __mul24(oy, kChainRow) + __mul24(ox, kChainPix))) = o ^ (int)xout;
            }
        };
        const SkipMul none = {0, 0, 0};
        auto finish = [&](int gr, int oy, int ox, v16i &acc) __attribute__((always_inline)) {
            mfma_drain(acc);
            if constexpr (PIPE) {
                store(gr, oy, ox, epilogue_hi16<0>(a, none, acc, v4i{0, 0, 0, 0}));
            } else {
                int tv[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) tv[q] = acc[q];
                store(gr, oy, ox, requant16_any(a, tv));
            }
        };
        // Multiplies group gr, whose first fragments are on their way, into acc.  Behind its matrix instructions: the fragments to come, in the end those of
        // the group after it, at (oy, ox) then (behind the last group: read and not used); PIPE: the requantisation of group gr - 4, whose sums are in old,
        // and its store.
        auto step = [&](auto reload_tag, int gr, int &oy, int &ox, v16i &acc, v16i &old, int old_y, int old_x) __attribute__((always_inline)) {
            constexpr bool RELOAD = decltype(reload_tag)::value;
            [[maybe_unused]] int ow[4] = {0, 0, 0, 0};
            const uint8_t *next = p;
            static_for<kChainF>([&](auto f_tag) __attribute__((always_inline)) {
                constexpr int f = decltype(f_tag)::value, g5 = f + RING - 1;
                if constexpr (f == 0) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[f], bf[f % RING], bias, 0, 0, 0);
                else acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[f], bf[f % RING], acc, 0, 0, 0);
                asm volatile("" : "+v"(acc));      // here, not wherever the sums are needed
                if constexpr (RELOAD) w[f] = next_weight(f);
                if constexpr (g5 < kChainF) fetch(p, std::integral_constant<int, g5>{}, std::integral_constant<int, g5>{});
                else fetch(next, std::integral_constant<int, g5 - kChainF>{}, std::integral_constant<int, g5>{});
                if constexpr (PIPE && f == 1) mfma_drain(old);
                if constexpr (PIPE && f >= 2 && f < 10) epilogue_hi_slice<0, 2 * (f - 2), 2>(a, none, old, v4i{0, 0, 0, 0}, ow);
                if constexpr (PIPE && f == 10) store(gr - 4, old_y, old_x, v4i{ow[0], ow[1], ow[2], ow[3]});
                if constexpr (f == 11) {
                    locate(gr + 4, oy, ox);
                    next = at(oy, ox);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            p = next;
        };
        static_assert(kChainF % RING == 0, "the next group's fragments take the first slots");
        // This wave's groups, the last one apart: it takes the next layer's weights behind its products.  (A wave without any goes through one whose pixels are
        // none; the first group's predecessor is none either.  One body in a loop and one behind it: with more of them the weights move between registers.)
        int gr = wave >> 1, oy, ox, py = 0, px = 0;
        locate(gr, oy, ox);
        p = at(oy, ox);
        static_for<RING - 1>([&](auto f_tag) __attribute__((always_inline)) { fetch(p, f_tag, f_tag); });
        v16i acc, old = bias;
        for (; gr + 4 < ng; gr += 4) {
            const int cy = oy, cx = ox;
            step(std::false_type{}, gr, oy, ox, acc, old, py, px);
            if constexpr (PIPE) old = acc;
            else finish(gr, cy, cx, acc);
            py = cy; px = cx;
        }
        const int cy = oy, cx = ox;
        step(std::integral_constant<bool, !LAST>{}, gr, oy, ox, acc, old, py, px);
        finish(gr, cy, cx, acc);
        if constexpr (!LAST) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0x0070);     // the weights of the layer after the next have landed; this wave's pixels are in LDS
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    };
    for (int l = 0; l + 1 < L; ++l) layer(std::false_type{}, l);
    layer(std::true_type{}, L - 1);
#endif
}

// ------------------------------------------------------------------ dispatch
// Estimated microseconds of a launch of L layers on TH x TW tiles: the launch itself, then per round of workgroups (one per
// compute unit) a prologue (from the second round on it waits for memory that other workgroups are using) and, per layer, rounds of four
// pixel groups and what a layer costs whatever its size (barrier, latencies, a last epilogue).  Measured / estimated, launches of 2 to 6 layers on
// uniform random bytes: one round of workgroups 256 x 256 8.9 / 8.2, 12.3 / 11.3 and 16.1 / 14.5 for 2 to 4 layers (inputs up to 255 add 5 %), 64 x 64 6.3 / 6.4,
// 8.5 / 8.4, 10.9 / 10.3, 13.5 / 11.7, 15.0 / 13.6; several rounds 480 x 640 28.1 / 30.2, 47.2 / 50.5, 65.0 / 69.9; from 0.81 to 1.18 over all sizes tried (64 x 64
// to 1600 x 2560, one to 16 pictures), low for five and six layers in one round, high for two in many.
static double chain_cost(long long tiles, int L, int th, int tw)
{
    double per_tile = 1.7;
    for (int b = 0; b < L; ++b) {
        const int ng = ((th + 2 * b) * (tw + 2 * b) + 31) / 32;
        per_tile += 0.6 * ((ng + 3) / 4) + 0.75;
    }
    const double rounds = (double)((tiles + 255) / 256);
    return 2.0 + per_tile * rounds + 2.1 * (rounds - 1);
}

// Microseconds of one layer by itself, in the kernel that iconv2d_brelu takes for it; full: inputs up to 255.  Measured / estimated:
// 64 x 64 3.7 / 3.4 (inputs up to 255: 3.7 / 3.4), two of them 4.1 / 4.2 (4.8 / 4.2), 96 x 96 4.2 / 7.5 (7.0 / 7.5), 128 x 128 4.4 / 7.5
// (7.1 / 7.5), 256 x 256 6.0 / 6.0 (9.6 / 9.7), 480 x 640 15.4 / 15.0 (26.8 / 26.8), 720 x 1280 34.2 / 35.7 (64.8 / 70.4).  (What stands at 7.5 goes to
// conv_flat.hip with inputs up to 127; chains are ahead there by more: 128 x 128 48 us for 18 layers, 75 one by one.)
static double layer_cost(int N, int H, int W, bool full)
{
    const long long pixels = (long long)N * H * W;
    if (pixels <= 8192) return pixels <= 4096 ? 3.4 : 4.2;           // conv_lat.hip, one or two work units per compute unit
    const double plane = full ? 0 : conv_plane_cost(N, H, W);
    if (plane > 0) return plane;
    const double tiles = 5.0 + 7.1e-5 * (double)pixels;              // the tile kernels
    return tiles > 7.5 ? tiles : 7.5;
}

// best tile for L layers
static double chain_tile(int N, int H, int W, int L, int &th, int &tw)
{
    const int most = kChainRP - 2 * L;
    double best = 1e300;
    for (int ny = (H + most - 1) / most, iy = 0; iy < 6 && ny <= H; ++ny, ++iy)
        for (int nx = (W + most - 1) / most, ix = 0; ix < 6 && nx <= W; ++nx, ++ix) {
            const int h = (H + ny - 1) / ny, w = (W + nx - 1) / nx;
            const double c = chain_cost((long long)N * ny * nx, L, h, w);
            if (c < best) { best = c; th = h; tw = w; }
        }
    return best;
}

// Cuts n layers into launches of len[0], len[1], ... layers (at most n entries); returns their number.  A piece of one layer is not a chain:
// iconv2d_brelu computes it.  full[i]: layer i's inputs go up to 255.
// 18 layers as cut here / one by one: 64 x 64 42 / 62 us, 256 x 256 71 / 103, 384 x 384 142 / 183; 720 x 1280 one by one 612, in nine chains of two 695;
// with inputs up to 255: 256 x 256 74 / 170, 256 x 384 128 / 204, 720 x 1280 741 / 1169.  Against the best split by the pieces' own times, 22 sizes of 64 x 64
// to 1600 x 2560 in both kinds: within 2 %, but for 480 x 640 with inputs up to 127, which goes one by one (273) where chains of two take 250: each is
// 28.1 us, two layers by themselves 30.8, estimated at 30.2 and 30.0.
int conv_chain_split(int N, int H, int W, int n, const bool *full, int *len)
{
    double cost[kChainMaxLayers + 1];
    int th, tw;
    const double single[2] = {layer_cost(N, H, W, false), layer_cost(N, H, W, true)};
    for (int L = 2; L <= kChainMaxLayers; ++L) cost[L] = chain_tile(N, H, W, L, th, tw);
    // shortest path over the number of layers done
    double best[257];
    int from[257];
    best[0] = 0;
    for (int i = 1; i <= n; ++i) {
        best[i] = 1e300;
        for (int L = 1; L <= kChainMaxLayers && L <= i; ++L) {
            const double c = best[i - L] + (L == 1 ? single[full[i - 1]] : cost[L]);
            // (at equal cost the shorter pieces come first: 256 x 256 in 2, 4, 4, 4, 4 layers takes 0.4 us less than in 4, 4, 4, 4, 2)
            if (c < best[i] + 1e-6) { best[i] = c; from[i] = L; }
        }
    }
    int k = 0;
    for (int i = n; i > 0; i -= from[i]) ++k;
    for (int i = n, j = k; i > 0; i -= from[i]) len[--j] = from[i];
    return k;
}

hipError_t launch_conv_chain(ChainArgs &g, hipStream_t st)
{
    struct Plan { int N, H, W, L, th, tw; };
    static thread_local Plan plan = {0, 0, 0, 0, 0, 0};     // host arithmetic only: the last tile choice of this thread
    if (plan.N != g.N || plan.H != g.H || plan.W != g.W || plan.L != g.L) {
        plan = {g.N, g.H, g.W, g.L, 1, 1};
        chain_tile(g.N, g.H, g.W, g.L, plan.th, plan.tw);
    }
    g.TH = plan.th;
    g.TW = plan.tw;
    if (g.L < 1 || g.L > kChainMaxLayers || g.TH < 1 || g.TW < 1 || g.TH + 2 * g.L > kChainRP || g.TW + 2 * g.L > kChainRP)
        return hipErrorInvalidValue;
    g.tiles_x = (g.W + g.TW - 1) / g.TW;
    g.tiles_per_img = g.tiles_x * ((g.H + g.TH - 1) / g.TH);
    const long long tiles = (long long)g.tiles_per_img * g.N;
    if (tiles < 1 || tiles > 0x7ffffff0LL / 8) return hipErrorInvalidValue;
    g.n_tiles = (int)tiles;
    g.per_xcd = (int)((tiles + 7) / 8);
    g.div_tpi = make_fast_div((unsigned)g.tiles_per_img);
    g.div_tx = make_fast_div((unsigned)g.tiles_x);
    for (int l = 0; l < g.L; ++l) {
        const unsigned rw = (unsigned)(g.TW + 2 * (g.L - 1 - l));
        g.inv[l] = (65536 + rw - 1) / rw;           // idx * inv >> 16 = idx / rw: idx < 22 * 22 and inv * rw - 65536 < 24
    }
    bool pipe = true;
    for (int l = 0; l < g.L; ++l) pipe = pipe && g.l[l].rq_fast;
    const auto kernel = pipe ? conv_chain_kernel<true> : conv_chain_kernel<false>;
    const hipError_t e = allow_large_lds((const void *)kernel);
    if (e != hipSuccess) return e;
    const FastDiv &tpi = g.div_tpi, &tx = g.div_tx;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * g.per_xcd)), dim3(512), kChainLds, st, g.x, g.l[0].wp, g.H, g.W, g.in_cs,
                       (unsigned)g.TH | (unsigned)g.TW << 8 | (unsigned)g.L << 16, g.n_tiles, g.tiles_per_img, tpi.mul, g.tiles_x, tx.mul,
                       tpi.s1 | tpi.s2 << 8 | tx.s1 << 16 | tx.s2 << 24, g);
    return hipGetLastError();
}

}  // namespace icnn
