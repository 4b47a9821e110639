// Convolutions on few pixels (a small batch in the deep stages of a residual network): latency, not throughput.
//
// Such a layer has a few tiles of the tile kernels, each of which walks the whole K axis alone through LDS with a barrier
// per step: 10 us and more for work that is a fraction of a microsecond spread over the chip.  Here a workgroup owns 32
// output channels x 32 pixels and its eight waves split the K axis: every wave requests ALL its weight and
// activation fragments (up to a batch of nine) straight from global memory into registers, so that a layer costs one
// memory latency, multiplies, and the eight partial tiles meet in LDS.  Then every thread finishes two neighbouring
// channels of one pixel, whose bias, skip operand and per-channel parameters have travelled with the
// fragments: the epilogue is spread over all waves too.
//
//   weights      the packed order is the fragment order: 1 KiB of consecutive bytes per wave and fragment
//   activations  a lane's fragment is 16 consecutive channels of its pixel's tap; borders and the K tail of a wave come as
//                zeros from the buffer descriptors' range checks
//   measured     33 of the 42 launches of one image through the 50-layer network, 5.6 us each (kernel trace), of which the matrix cores work
//                1 %: launch, one latency of the memory side (weights from beyond L2), the meeting in LDS
//   order        work units are dealt channel-major to the XCDs, so that each L2 fetches an eighth of the weights
//
// DUAL: a residual block's last layer with its projection (see conv_dual.hip): both contractions have accumulators and
// partial tiles of their own, and the projection's sum is rescaled when the tiles have met.
#include "conv_common.h"

#include <type_traits>

namespace icnn {

constexpr int kLatWaves = 8;
[[maybe_unused]] constexpr int kLatPix = 36 * 4;                      // bytes of one pixel's 32 sums in LDS, with padding against bank conflicts
[[maybe_unused]] constexpr int kLatTile = 32 * kLatPix;               // one wave's partial tile of 32 pixels

struct LatOperand {
    const uint8_t *x, *wp;
    unsigned x_bytes;
    int H, W, in_cs, KW, sh, sw, ph, pw;
    int frags;                                       // K / 32
    int fpt;                                         // fragments per tap: cin / 32
    FastDiv div_fpt, div_kw;
    int chunk_bytes;                                 // packed weights of 32 output channels
};
struct LatArgs {
    LatOperand m, p;                                 // the layer; its projection (DUAL)
    int n_pt, units, per_xcd;                        // pixel tiles, channel chunks x pixel tiles
    FastDiv div_pt, div_howo, div_wo;
    const int32_t *pbias;
    int pres_mul, pres_shift;                        // rescale of the projection's sums
    int pair_out, pair_res;                          // two neighbouring channels can be stored / loaded as one access
};

template <bool DUAL, bool U8>
__global__ __launch_bounds__(64 * kLatWaves, 4) void conv_lat_kernel(const ConvArgs a, const LatArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr unsigned OOB = 0x80000000u;
    constexpr int BATCH = 9;                         // fragments in flight per wave
    __shared__ __attribute__((aligned(16))) uint8_t part[(DUAL ? 2 : 1) * kLatWaves * kLatTile];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = (int)(blockIdx.x & 7) * g.per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= g.per_xcd || u >= g.units) return;
    const int chunk = fast_div(u, g.div_pt), pt = u - chunk * g.n_pt;

    // ---- what this thread finishes: channels co, co + 1 of pixel p
    const int co = chunk * 32 + 2 * (tid & 15), p = pt * 32 + (tid >> 4);
    const bool mine = p < a.M && co < a.Cout, c1 = co + 1 < a.Cout;
    int bias2[2] = {0, 0}, pbias2[2] = {0, 0}, res2[2] = {0, 0};
    const int32_t *const gp = a.pc ? a.pc + (size_t)(min(co, ((a.Cout + 15) & ~15) - 2) >> 4) * kPcGroupInts + (co & 15) : nullptr;
    if (mine) {
        bias2[0] = a.bias[co] + (U8 ? 128 * a.wsum[co] : 0);
        if (c1) bias2[1] = a.bias[co + 1] + (U8 ? 128 * a.wsum[co + 1] : 0);
        if (DUAL) {
            pbias2[0] = g.pbias[co];
            if (c1) pbias2[1] = g.pbias[co + 1];
        }
        if (a.res_mode != 0) {
            const size_t ro = (size_t)p * a.res_cs + co;
            if (g.pair_res) {
                const int v = *(const uint16_t *)((const uint8_t *)a.res + ro);
                res2[0] = v & 0xff;
                res2[1] = v >> 8;
            } else {
                res2[0] = load_elem(a.res, ro, a.res_dtype);
                if (c1) res2[1] = load_elem(a.res, ro + 1, a.res_dtype);
            }
        }
    }

    // ---- this lane's pixel as MFMA column
    const int mp = pt * 32 + col;
    const bool pok = mp < a.M;
    const int pn = fast_div(pok ? mp : 0, g.div_howo);
    const int pr = (pok ? mp : 0) - pn * (a.Ho * a.Wo);
    const int py = fast_div(pr, g.div_wo), px = pr - py * a.Wo;

    // A chip full of such waves is bound by the instructions it issues, so a fragment's requests cost none but themselves: the weights'
    // place is a scalar offset, and a pixel's place under the kernel window is worked out once per tap.
    auto contract = [&](const LatOperand &o, v16i &acc) {
        // wave w takes fragments [f0, f1)
        const int f0 = wave * o.frags / kLatWaves, f1 = (wave + 1) * o.frags / kLatWaves;
        // (the descriptor ends behind this wave's last fragment: what a batch requests beyond it comes as zeros)
        const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)(o.wp + (size_t)chunk * o.chunk_bytes), 0, f1 * 1024, 0x00020000);
        const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)o.x, 0, o.x_bytes, 0x00020000);
        const int iy0 = py * o.sh - o.ph, ix0 = px * o.sw - o.pw;
        const int base = ((pn * o.H + iy0) * o.W + ix0) * o.in_cs + half * 16;
        int tap = fast_div(f0, o.div_fpt), kk = f0 - tap * o.fpt;
        int kh = fast_div(tap, o.div_kw), kw = tap - kh * o.KW;
        auto place = [&] {                           // this lane's byte offset at the current tap
            const bool in = pok && (unsigned)(iy0 + kh) < (unsigned)o.H && (unsigned)(ix0 + kw) < (unsigned)o.W;
            return in ? (unsigned)(base + (kh * o.W + kw) * o.in_cs) : OOB;
        };
        unsigned off = place();
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0;
        for (int fb = f0; fb < f1; fb += BATCH) {
            v4i fa[BATCH], fx[BATCH];
#pragma unroll
            for (int q = 0; q < BATCH; ++q)
                fa[q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_w, (unsigned)(lane * 16 + q * 1024), fb * 1024, 0));
#pragma unroll
            for (int q = 0; q < BATCH; ++q) {
                if (fb + q < f1) fx[q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off, kk * 32, 0));
                else fx[q] = v4i{0, 0, 0, 0};
                if (++kk == o.fpt) {
                    kk = 0;
                    if (++kw == o.KW) { kw = 0; ++kh; }
                    off = place();
                }
            }
            __builtin_amdgcn_sched_barrier(0);       // all requests go out before the first use
#pragma unroll
            for (int q = 0; q < BATCH; ++q) {
                if (U8) fx[q] ^= (int)0x80808080;
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[q], fx[q], acc, 0, 0, 0);
            }
        }
        mfma_drain(acc);
    };
    auto spill = [&](const v16i &acc, int which) {
        uint8_t *d = part + (which * kLatWaves + wave) * kLatTile + col * kLatPix + half * 64;
#pragma unroll
        for (int q = 0; q < 4; ++q) *(v4i *)(d + q * 16) = v4i{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    };
    {
        v16i acc;
        if (DUAL) {
            contract(g.p, acc);
            spill(acc, 1);
        }
        contract(g.m, acc);
        spill(acc, 0);
    }
    __syncthreads();

    if (!mine) return;
    auto total = [&](int which, int (&s)[2]) {
        typedef int v2i __attribute__((ext_vector_type(2)));
        const uint8_t *d = part + which * kLatWaves * kLatTile + (tid >> 4) * kLatPix + (tid & 15) * 8;
#pragma unroll
        for (int w = 0; w < kLatWaves; ++w) {
            const v2i v = *(const v2i *)(d + w * kLatTile);
            s[0] += v.x;
            s[1] += v.y;
        }
    };
    total(0, bias2);
    if (DUAL) {
        // (the host has proved that the merged sum stays inside int32)
        total(1, pbias2);
#pragma unroll
        for (int e = 0; e < 2; ++e)
            bias2[e] += (int)rsr64((int64_t)pbias2[e] * (gp ? gp[kPcResMul + e] : g.pres_mul), gp ? gp[kPcResShift + e] & 63 : g.pres_shift);
    }
    const size_t oo = (size_t)p * a.out_cs + a.out_co + co;
    int q2[2];
    if (a.rq24 && !a.pc && (a.res_mode == 0 || (a.res_mode == 1 && a.res_fast))) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int t = bias2[e];
            if (a.res_mode != 0)
                t = __builtin_elementwise_add_sat(t, (int)((__umul24((uint32_t)res2[e], (uint32_t)a.res_mul) + (uint32_t)((1 << a.res_shift) >> 1)) >> a.res_shift));
            q2[e] = (int)((__umul24((uint32_t)med3_v0s(t, a.t_hi), (uint32_t)a.mul) + (uint32_t)a.rnd) >> a.shift);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int mul = a.mul, sh = a.shift, rm = a.res_mul, rs = a.res_shift;
            if (gp) {
                mul = gp[kPcMul + e]; sh = gp[kPcShift + e] & 63;
                rm = gp[kPcResMul + e]; rs = gp[kPcResShift + e] & 63;
            }
            int64_t t = bias2[e];
            const int64_t skip = a.res_mode != 0 ? rsr64((int64_t)res2[e] * rm, rs) : 0;
            if (a.res_mode == 1) t += skip;
            const int ti = sat32(t);
            if (a.out_mode == 3) {
                q2[e] = ti;
            } else {
                int64_t q = rsr64((int64_t)ti * mul, sh);
                if (a.res_mode == 2) q += skip;
                q2[e] = clampi64(q, a.lo, a.hi);
            }
        }
    }
    if (a.out_mode == 3) {
        ((int32_t *)a.out)[oo] = q2[0];
        if (c1) ((int32_t *)a.out)[oo + 1] = q2[1];
    } else if (g.pair_out) {
        *(uint16_t *)((uint8_t *)a.out + oo) = (uint16_t)((q2[0] & 0xff) | (q2[1] << 8));
    } else {
        ((uint8_t *)a.out)[oo] = (uint8_t)q2[0];
        if (c1) ((uint8_t *)a.out)[oo + 1] = (uint8_t)q2[1];
    }
#endif
}

// ------------------------------------------------------------------ dispatch
static void lat_operand(LatOperand &o, const uint8_t *x, const uint8_t *wp, unsigned x_bytes, int H, int W, int Cin, int in_cs, int KH, int KW,
                        int sh, int sw, int ph, int pw, int ksteps)
{
    o.x = x; o.wp = wp; o.x_bytes = x_bytes;
    o.H = H; o.W = W; o.in_cs = in_cs; o.KW = KW; o.sh = sh; o.sw = sw; o.ph = ph; o.pw = pw;
    o.fpt = Cin / 32;
    o.frags = KH * KW * o.fpt;
    o.div_fpt = make_fast_div((unsigned)o.fpt);
    o.div_kw = make_fast_div((unsigned)KW);
    o.chunk_bytes = ksteps * kChunkBytes;
}

static bool lat_shape_ok(const ConvArgs &a)
{
    return a.Cin % 32 == 0 && a.in_cs % 16 == 0 && !((uintptr_t)a.x & 15) && a.in_xor == 0 && a.x_bytes < 0x7fffff00u && a.KH * a.KW <= 1024 &&
           a.ksteps == (a.KH * a.KW * a.Cin + 63) / 64;
}

// Worth it while all work units (32 channels x 32 pixels) are on the chip at once: two workgroups of eight waves fit a compute unit, and a
// launch costs by whole units per compute unit.  Microseconds here / in the tile kernels, over layers of residual networks at 1 to 24
// images: 3x3 of 256 channels on 14 x 14, 248 units 6.1 / 9.4, 448 units 8.2 / 9.4, 496 units 8.3 / 9.5, 544 units 10.8 / 9.5;
// 1024 -> 256 there, 496 units 6.8 / 7.4, 544 units 8.7 / 7.3; 3x3 / 2 of 512 channels, 496 units 14.3 / 18.4, 592 units 19.0 / 18.4;
// 512 -> 2048 on 7 x 7, 448 units 5.6 / 6.0, 512 units 5.9 / 5.9, 640 units 7.3 / 6.2.
// The kernel whose waves split K over a patch in LDS (conv_deep.hip) is nearer where it applies: two units per compute unit lose to it
// with 144 fragments of K (3x3 of 512 channels on 7 x 7: 256 units 8.2 / 11.4, 272 units 12.0 / 11.5) and win with 72 (the first line).
// With a projection: 12 fragments, 400 units 6.8 / 6.5 on its own and 1 % of a one-image step the other way; 24, 416 units 7.9 / 7.9, 608
// units 10.4 / 7.8; 48, 512 units 9.0 / 9.9, 640 units 11.8 / 10.1.
constexpr int kLatOnePerCu = 256, kLatTwoPerCu = 512;
static bool lat_worth(int M, int Cout, int frags, int most_units)
{
    const long long units = (long long)((Cout + 31) / 32) * ((M + 31) / 32);
    return frags >= 4 && units <= most_units;
}

bool conv_lat_applies(const ConvArgs &a)
{
    if (!lat_shape_ok(a) || g_tuning.no_lat) return false;
    if (g_tuning.no_fc && a.KH == 1 && a.KW == 1 && a.sh == 1 && a.sw == 1 && a.M <= 64 && a.Cin >= 512) return false;
    const bool forced = g_tuning.tile >= 0 || g_tuning.ksplit || g_tuning.deep_always || g_tuning.halo_always || g_tuning.halo_tile || g_tuning.plane_always;
    const int frags = a.KH * a.KW * a.Cin / 32;
    const bool nearer = frags > 96 && !g_tuning.no_deep && conv_deep_applies(a);
    return g_tuning.lat || (!forced && lat_worth(a.M, a.Cout, frags, nearer ? kLatOnePerCu : kLatTwoPerCu));
}

static hipError_t launch_lat(const ConvArgs &a, const ProjArgs *q, hipStream_t st)
{
    LatArgs g;
    lat_operand(g.m, a.x, a.wp, a.x_bytes, a.H, a.W, a.Cin, a.in_cs, a.KH, a.KW, a.sh, a.sw, a.ph, a.pw, a.ksteps);
    g.p = g.m;
    g.pbias = nullptr;
    g.pres_mul = 1;
    g.pres_shift = 0;
    if (q) {
        lat_operand(g.p, q->x, q->wp, q->x_bytes, q->H, q->W, q->Cin, q->in_cs, 1, 1, q->sh, q->sw, 0, 0, q->ksteps);
        g.pbias = q->bias;
        g.pres_mul = q->res_mul;
        g.pres_shift = q->res_shift;
    }
    const int chunks = (a.Cout + 31) / 32;
    g.n_pt = (a.M + 31) / 32;
    const long long units = (long long)chunks * g.n_pt;
    if (units < 1 || units > (1 << 28)) return hipErrorInvalidValue;
    g.units = (int)units;
    g.per_xcd = (g.units + 7) / 8;
    g.div_pt = make_fast_div((unsigned)g.n_pt);
    g.div_howo = make_fast_div((unsigned)(a.Ho * a.Wo));
    g.div_wo = make_fast_div((unsigned)a.Wo);
    g.pair_out = a.out_mode != 3 && !((uintptr_t)a.out & 1) && a.out_cs % 2 == 0 && a.out_co % 2 == 0 && a.Cout % 2 == 0;
    g.pair_res = a.res_mode != 0 && a.res_dtype == 0 && !((uintptr_t)a.res & 1) && a.res_cs % 2 == 0 && a.Cout % 2 == 0;
    const dim3 grid((unsigned)(8 * g.per_xcd)), block(64 * kLatWaves);
    if (q) hipLaunchKernelGGL((conv_lat_kernel<true, false>), grid, block, 0, st, a, g);
    else if (a.frag_xor) hipLaunchKernelGGL((conv_lat_kernel<false, true>), grid, block, 0, st, a, g);
    else hipLaunchKernelGGL((conv_lat_kernel<false, false>), grid, block, 0, st, a, g);
    return hipGetLastError();
}

hipError_t launch_conv_lat(const ConvArgs &a, hipStream_t st)
{
    return launch_lat(a, nullptr, st);
}

bool conv_lat_dual_applies(const ConvArgs &a, const ProjArgs &q)
{
    if (!lat_shape_ok(a) || g_tuning.no_lat || q.Cin % 32 || q.in_cs % 16 || ((uintptr_t)q.x & 15) || a.frag_xor) return false;
    return g_tuning.lat || lat_worth(a.M, a.Cout, (a.Cin + q.Cin) / 32, kLatTwoPerCu);
}
hipError_t launch_conv_lat_dual(const ConvArgs &a, const ProjArgs &q, hipStream_t st)
{
    return launch_lat(a, &q, st);
}

}  // namespace icnn
