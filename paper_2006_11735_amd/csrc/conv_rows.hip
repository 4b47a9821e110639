// The two-branch layer of the restoration network on large pictures: a 5x5 layer of 64 channels and, in the same launch, the 3x3 layer
// of the same input (at most 32 output channels each, stride 1, "same" padding, unsigned bytes by one 32-bit or 24-bit product each).
//
// conv_plane.hip runs it with two waves per SIMD that own two tile rows each: 51 % of the matrix cores' rate, because every
// product needs a fresh fragment from LDS (1.34 MB per tile, 7.5 k clocks of LDS against 8.7 k of matrix work), and because the barrier
// per tile keeps the two waves in step, so that both multiply and then both requantise.  Here a SIMD has ONE wave with all of its registers:
//
//   tile     16 rows x 32 columns; wave w owns rows 4 w .. 4 w + 3 (a pixel group of 32 = one tile row), for both layers: eight
//            accumulator tiles
//   K loop   outermost the kernel column and the channel half (ten steps), then the eight input rows under the wave's four output rows:
//            one activation fragment of an input row is multiplied into every output row it reaches (up to five, and three of the
//            twin), with the step's five (+ three) weight fragments in registers.  0.6 KiB of LDS per matrix instruction instead of 1.2.
//   epilogue of the tile before, dealt out between this tile's matrix instructions (two sets of accumulators, used in turn)
//   patch, weights, copies, tile walk: as in conv_plane.hip (conv_patch.h)
//
// Straight-line code for a tile: 248 matrix instructions per wave (272 where the twin has more than 16 channels) and 960 others in their shadow.
// Measured on 2560 x 1600, 64 -> 32 + 16, inside the network: 240 us in the form with two waves per SIMD, 210 us with one wave and 272, 195 us
// here (59 and 53 us on 720 x 1280).  A tile takes 6.1 us = 37 clocks per matrix instruction at the 1.5 GHz that the card's power
// leaves the matrix units when all of them multiply random bytes: what helps is fewer products.
#include "conv_patch.h"

namespace icnn {

constexpr int kRowsTW = 32, kRowsTH = 16;

// The products of input row r of a wave's eight, at kernel column dx: one of the 5x5 layer for each output row that r reaches, and where dx is
// the twin's too one of the twin for each of its rows (PAIR: pairs of rows) that r reaches.
template <bool PAIR>
struct RowsProducts {
    static constexpr int UNITS = PAIR ? 2 : 4, EACH = PAIR ? 2 : 1, SPAN = PAIR ? 4 : 3;     // the twin's accumulators, output rows and input rows of one
    static constexpr bool row(int r, int dy) { return r - dy >= 0 && r - dy < 4; }
    static constexpr bool twin(int r, int dx, int d) { return dx >= 1 && dx <= 3 && r - 1 - d >= 0 && (r - 1 - d) % EACH == 0 && (r - 1 - d) / EACH < UNITS; }
    // matrix instructions of a tile before those of fragment i (step i / 8, input row i % 8), of it before number dy of the layer, number d of the twin
    static constexpr int before(int i, int dy, int d)
    {
        int m = 0;
        for (int f = 0; f <= i; ++f) {
            for (int k = 0; k < (f < i ? 5 : dy); ++k) m += row(f % 8, k);
            for (int k = 0; k < (f < i ? SPAN : d); ++k) m += twin(f % 8, f / 16, k);
        }
        return m;
    }
    static constexpr int ALL = before(80, 0, 0);
    static constexpr int OUTPUTS = (4 + UNITS) * 16;       // of a lane
};
static_assert(RowsProducts<false>::ALL == 4 * (50 + 18) && RowsProducts<true>::ALL == 4 * 50 + 2 * 24, "products of four rows");

// FORM: both layers requantise by that form of requant16: 1 a product's high word (ConvArgs::rq_fast); 3 or 4 where that does not apply to both, at ratios
// of one half and more or a shift of 33 (2560 x 1600, 64 -> 32 + 16, one layer by itself: ratio 1 235 us here, 267 with two-dimensional tiles; shift 33
// 234 and 288; 238 in form 1).  PAIR: the twin has 16 channels; an accumulator tile of it holds two
// output rows, the second in the lanes and weight rows that the channels 16 to 31 would have: 248 products of four rows instead of 272.
template <bool PAIR, int FORM>
__global__ __launch_bounds__(256, 1) void conv_rows_twin_kernel(const ConvArgs a, const ConvArgs b, const TileWalk g)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr int KS = 5, KSB = 3, CIN = 64, RPW = 4;
    using Patch = TilePatch<KS, CIN, kRowsTH, kRowsTW, 4>;
    constexpr int ROWB = Patch::ROWB, CPW = Patch::CPW, PATCH = Patch::BYTES;
    constexpr int F = KS * KS * 2, FB = KSB * KSB * 2;                   // weight fragments of 32 k-values
    constexpr int WBYTES = F * 1024, WBYTESB = FB * 1024;
    static_assert(WBYTES + WBYTESB + 2 * PATCH <= 160 * 1024, "LDS");

    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint8_t *const wbuf = lds;
    uint8_t *const wbufB = lds + WBYTES;
    uint8_t *const pbuf = lds + WBYTES + WBYTESB;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.x_bytes, 0x00020000);

    Patch patch;
    patch.locate(a, wave, lane);
    auto issue_copy = [&](auto i_tag, int base, int y0, int x0, int buf) {
        patch.template issue<decltype(i_tag)::value>(rs_x, a, pbuf + buf * PATCH, wave, base, y0, x0);
    };

    const int v0 = blockIdx.x;
    if (!g.valid(v0)) return;                          // (the whole workgroup: it has no tile at all)
    {
        int n, y0, x0;
        g.template origin<kRowsTH, kRowsTW>(v0, n, y0, x0);
        const int base = Patch::base(a, n, y0, x0);
        static_for<CPW>([&](auto i_tag) { issue_copy(i_tag, base, y0, x0, 0); });
        copy_packed_weights<4, WBYTES, false>(a.wp, a.wp_bytes, wbuf, wave, lane);
        copy_packed_weights<4, WBYTESB, false>(b.wp, b.wp_bytes, wbufB, wave, lane);
    }
    v16i bias[1], biasB[1];
    load_bias_rows<1>(a, 0, half, bias);
    load_bias_rows<1>(b, 0, PAIR ? 0 : half, biasB);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0), lgkmcnt(0): the first patch and the weights are in LDS
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    const uint8_t *const wlane = wbuf + lane * 16, *const wlaneB = wbufB + lane * 16;
    // PAIR: weight row m of a fragment belongs to the tile's first output row, its kernel row is the distance d of the input row from that; or
    // (m & 4: the rows of channels 16 to 31, zeros in memory) to the second, its kernel row is d - 1.  Distance 0 is a fragment as packed; distance
    // 3 is kernel row 2 with the two kinds of rows exchanged; between, a lane reads the fragment of its own kernel row.
    constexpr int KROWB = KSB * 2 * 1024;
    const uint8_t *const wpair = wbufB + (lane & ~4) * 16 - (lane & 4 ? KROWB : 0), *const wlast = wbufB + (lane ^ 4) * 16 - KROWB;
    int ex[KS][2];                                   // this lane's offset in the wave's first patch row, per kernel column and channel half
#pragma unroll
    for (int dx = 0; dx < KS; ++dx)
#pragma unroll
        for (int k = 0; k < 2; ++k) ex[dx][k] = (RPW * wave) * ROWB + (col + dx) * 64 + (((2 * k + half) ^ (((col + dx) >> 2) & 3)) << 4);
    const bool storeA = half * 16 < a.Cout, storeB = PAIR || half * 16 < b.Cout;

    struct Done {                                    // where a finished tile's outputs go
        int pix;                                     // this lane's pixel in the wave's first row
        int rows;                                    // rows of it inside the picture (0: this lane's column is outside)
    };
    // one tile: multiplies into acc / accB; the tile before (sums in old / oldB, place in was) is requantised and stored meanwhile
    using Products = RowsProducts<PAIR>;
    constexpr int UNITS = Products::UNITS, SPANB = Products::SPAN;
    auto tile = [&](auto prev_tag, int v, int buf, v16i (&acc)[RPW], v16i (&accB)[UNITS], const v16i (&old)[RPW], const v16i (&oldB)[UNITS], const Done &was, Done &now) {
        constexpr bool PREV = decltype(prev_tag)::value;
        int n, y0, x0;
        g.template origin<kRowsTH, kRowsTW>(v, n, y0, x0);
        now.pix = (n * a.H + y0 + RPW * wave) * a.W + x0 + col;
        now.rows = x0 + col < a.W ? min(RPW, a.H - y0 - RPW * wave) : 0;
        const bool more = g.valid(v + (int)gridDim.x);
        int nn = 0, ny0 = 0, nx0 = 0;
        if (more) g.template origin<kRowsTH, kRowsTW>(v + (int)gridDim.x, nn, ny0, nx0);
        const int nbase = Patch::base(a, nn, ny0, nx0);
        const uint8_t *const P = pbuf + buf * PATCH;

        constexpr int ROWS = RPW + KS - 1;           // input rows under the wave's output rows
        constexpr int STEPS = KS * 2;
        constexpr int RING = 4;
        v4i A[2][KS], AB[2][SPANB], B[RING];
        [[maybe_unused]] int wd[4] = {0, 0, 0, 0};
        auto fetch_a = [&](auto s_tag, auto q_tag) {             // weight fragment q of step s (q >= KS: the twin's)
            constexpr int s = decltype(s_tag)::value, q = decltype(q_tag)::value, DX = s >> 1, KK = s & 1;
            if constexpr (q < KS) A[s & 1][q] = *(const v4i *)(wlane + ((q * KS + DX) * 2 + KK) * 1024);
            else if constexpr (q < KS + SPANB && DX >= 1 && DX <= KSB) {
                constexpr int d = q - KS;
                const uint8_t *const from = !PAIR || d == 0 ? wlaneB : d < KSB ? wpair : wlast;
                AB[s & 1][d] = *(const v4i *)(from + ((d * KSB + DX - 1) * 2 + KK) * 1024);
            }
        };
        auto fetch_b = [&](auto i_tag) {                         // activation fragment i = step * ROWS + input row
            constexpr int i = decltype(i_tag)::value, s = i / ROWS, r = i % ROWS;
            B[i % RING] = *(const v4i *)(P + ex[s >> 1][s & 1] + r * ROWB);
        };
        // the part of the tile before that goes behind matrix instruction m of this one
        auto deal = [&](auto m_tag) {
            constexpr int m = decltype(m_tag)::value;
            if constexpr (PREV) {
                // pairs of outputs [LO, HI): sixteen outputs of each row of a unit of the twin, then sixteen of that, then the next unit's
                constexpr int LO = m * (Products::OUTPUTS / 2) / Products::ALL, HI = (m + 1) * (Products::OUTPUTS / 2) / Products::ALL;
                static_for<HI - LO>([&](auto q_tag) {
                    constexpr int o = (LO + decltype(q_tag)::value) * 2, k = o % 16, group = Products::EACH + 1, u = o / 16 / group, t = o / 16 % group;
                    constexpr bool twin = t == Products::EACH;
                    constexpr int j = twin ? u : u * Products::EACH + t;
                    const v16i &sums = twin ? oldB[twin ? j : 0] : old[twin ? 0 : j];
                    if constexpr (FORM == 1) epilogue_hi_slice<0, k, 2>(twin ? b : a, SkipMul{0, 0, 0}, sums, v4i{0, 0, 0, 0}, wd);
                    else epilogue_rq24_slice<0, k, 2, FORM>(twin ? b : a, sums, v4i{0, 0, 0, 0}, wd);
                    if constexpr (k == 14) {
                        const ConvArgs &c = twin ? b : a;
                        const int row = PAIR && twin ? 2 * j + half : j, co = PAIR && twin ? 0 : half * 16;
                        if (row < was.rows && (twin ? storeB : storeA))
                            *(v4i *)((uint8_t *)c.out + (size_t)(was.pix + row * a.W) * c.out_cs + c.out_co + co) = v4i{wd[0], wd[1], wd[2], wd[3]};
                    }
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        static_for<KS + SPANB>([&](auto q_tag) { fetch_a(std::integral_constant<int, 0>{}, q_tag); });
        static_for<RING - 1>([&](auto i_tag) { fetch_b(i_tag); });
        static_for<STEPS * ROWS>([&](auto i_tag) {
            constexpr int i = decltype(i_tag)::value, s = i / ROWS, r = i % ROWS, DX = s >> 1;
            if constexpr (i + RING - 1 < STEPS * ROWS) fetch_b(std::integral_constant<int, i + RING - 1>{});
            if constexpr (s + 1 < STEPS) {
                fetch_a(std::integral_constant<int, s + 1>{}, std::integral_constant<int, r>{});
                if constexpr (r == ROWS - 1 && ROWS < KS + SPANB) fetch_a(std::integral_constant<int, s + 1>{}, std::integral_constant<int, ROWS>{});
            }
            constexpr int EVERY = STEPS * ROWS / CPW;            // a copy of the next patch every so many fragments
            if constexpr (i % EVERY == 0 && i / EVERY < CPW) {
                if (more) issue_copy(std::integral_constant<int, i / EVERY>{}, nbase, ny0, nx0, buf ^ 1);
            }
            // this fragment's products, each followed by its share of the tile before: outputs are dealt out evenly over the matrix
            // instructions (between two of them there is room for seven vector instructions)
            static_for<KS>([&](auto dy_tag) {
                constexpr int dy = decltype(dy_tag)::value, j = r - dy, d = dy - 1;
                if constexpr (Products::row(r, dy)) {
                    if constexpr (s == 0 && dy == 0) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[0][0], B[i % RING], bias[0], 0, 0, 0);
                    else acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[s & 1][dy], B[i % RING], acc[j], 0, 0, 0);
                    deal(std::integral_constant<int, Products::before(i, dy, d < 0 ? 0 : d)>{});
                }
                if constexpr (d >= 0 && d < SPANB && Products::twin(r, DX, d)) {
                    constexpr int u = (r - 1 - d) / Products::EACH;
                    if constexpr (s == 2 && d == 0) accB[u] = __builtin_amdgcn_mfma_i32_32x32x32_i8(AB[0][0], B[i % RING], biasB[0], 0, 0, 0);
                    else accB[u] = __builtin_amdgcn_mfma_i32_32x32x32_i8(AB[s & 1][d], B[i % RING], accB[u], 0, 0, 0);
                    deal(std::integral_constant<int, Products::before(i, dy + 1, d)>{});
                }
            });
        });
        mfma_drain(acc);
        mfma_drain(accB);
        asm volatile("" ::: "memory");
        ICNN_WAIT_VMCNT(0);                          // the next tile's patch has landed (this wave's copies of it)
        __builtin_amdgcn_s_waitcnt(0xC07F);          // and this wave has read the last of this tile's patch
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto finish = [&](const v16i (&acc)[RPW], const v16i (&accB)[UNITS], const Done &was) {
        static_for<RPW>([&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
            if (j >= was.rows || !storeA) return;
            *(v4i *)((uint8_t *)a.out + (size_t)(was.pix + j * a.W) * a.out_cs + a.out_co + half * 16) = epilogue_bytes16<0, FORM>(a, acc[j], v4i{0, 0, 0, 0});
        });
        static_for<UNITS>([&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
            const int row = PAIR ? 2 * j + half : j;
            if (row >= was.rows || !storeB) return;
            *(v4i *)((uint8_t *)b.out + (size_t)(was.pix + row * a.W) * b.out_cs + b.out_co + (PAIR ? 0 : half * 16)) = epilogue_bytes16<0, FORM>(b, accB[j], v4i{0, 0, 0, 0});
        });
    };

    v16i acc0[RPW], acc1[RPW], accB0[UNITS], accB1[UNITS];
#pragma unroll
    for (int j = 0; j < RPW; ++j) acc0[j] = acc1[j] = bias[0];
#pragma unroll
    for (int j = 0; j < UNITS; ++j) accB0[j] = accB1[j] = biasB[0];
    Done d0 = {0, 0}, d1 = {0, 0};
    int v = v0;
    tile(std::false_type{}, v, 0, acc0, accB0, acc1, accB1, d1, d0);
    for (;;) {
        v += gridDim.x;
        if (!g.valid(v)) { finish(acc0, accB0, d0); break; }
        tile(std::true_type{}, v, 1, acc1, accB1, acc0, accB0, d0, d1);
        v += gridDim.x;
        if (!g.valid(v)) { finish(acc1, accB1, d1); break; }
        tile(std::true_type{}, v, 0, acc0, accB0, acc1, accB1, d1, d0);
    }
#endif
}

// ------------------------------------------------------------------ dispatch
// what the kernel assumes of a layer beyond its shape (conv_plane_twin_ok)
static bool rows_layer_ok(const ConvArgs &a)
{
    return a.epi_vec && a.out_mode <= 1 && a.res_mode == 0 && (a.Cout & 15) == 0 && a.Cout <= 32;
}
// the cheapest form of the kernel that both layers' parameters allow; 0: none
static int rows_form(const ConvArgs &a, const ConvArgs &b)
{
    return a.rq_fast && b.rq_fast ? 1 : a.rq24 && b.rq24 ? 3 : a.rqh && b.rqh ? 4 : 0;
}
bool conv_rows_twin_applies(const ConvArgs &a, const ConvArgs &b)
{
    return a.KH == 5 && a.Cin == 64 && rows_layer_ok(a) && rows_layer_ok(b) && rows_form(a, b) != 0 && !g_tuning.plane_no_pipe;
}

hipError_t launch_conv_rows_twin(const ConvArgs &a, const ConvArgs &b, hipStream_t st)
{
    TileWalk g;
    if (!tile_walk(g, a.N, a.H, a.W, kRowsTH, kRowsTW)) return hipErrorInvalidValue;
    constexpr size_t lds_bytes = (50 + 18) * 1024 + 2 * (size_t)TilePatch<5, 64, kRowsTH, kRowsTW, 4>::BYTES;
    auto go = [&](auto kernel) -> hipError_t {
        const hipError_t e = allow_large_lds((const void *)kernel);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * g.per_xcd < 256 ? 8 * g.per_xcd : 256)), dim3(256), lds_bytes, st, a, b, g);
        return hipGetLastError();
    };
    const bool pair = b.Cout == 16;
    switch (rows_form(a, b)) {
    case 1: return pair ? go(conv_rows_twin_kernel<true, 1>) : go(conv_rows_twin_kernel<false, 1>);
    case 3: return pair ? go(conv_rows_twin_kernel<true, 3>) : go(conv_rows_twin_kernel<false, 3>);
    case 4: return pair ? go(conv_rows_twin_kernel<true, 4>) : go(conv_rows_twin_kernel<false, 4>);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace icnn
