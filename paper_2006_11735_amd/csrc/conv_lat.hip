// Convolutions on few pixels (a small batch in the deep stages of a residual network): latency, not throughput.
//
// Such a layer has a few tiles of the tile kernels, each of which walks the whole K axis alone through LDS with a barrier
// per step: 10 us and more for work that is a fraction of a microsecond spread over the chip.  Here a workgroup owns 16 or 32
// output channels x 16 or 32 pixels and its eight waves split the K axis: every wave requests ALL its weight and
// activation fragments (up to NS steps of 64) straight from global memory into registers, so that a layer costs one
// memory latency, multiplies, and the eight partial tiles meet in LDS.  Then every thread finishes one or two outputs, whose bias,
// skip operand and per-channel parameters have travelled with the fragments.
//
//   order        what bounds these launches is the time before the last request is out and the chain behind the data, so the weights'
//                requests come first and need the fewest instructions, then the activations', then what the epilogue reads; no load's
//                result is looked at before all of them are out, and which steps a wave takes stands in a table the host has made
//   weights      packed for fragments of 32 x 32: the four K quarters of a step's 64, 16 consecutive rows of each (256 bytes: whole cache lines),
//                are a fragment of 16 x 64
//   activations  a lane's fragment is 16 consecutive channels of its pixel's tap; borders come as zeros from the buffer descriptors' range
//                checks, a wave's missing steps from the weights' one
//   tile         the smaller, the fewer bytes pass a unit's memory path (64 B/clk) and the more compute units take part (lat_tile)
//   measured     one image through the 50-layer network, clocks from a wave's start (the kernel before, which asked for its skip operand and bias first
//                / this one): 1024 -> 256 on 14 x 14 weights requested 3600 / 480, data there 4600 / 2300, stored 7700 / 3300; 3x3 of 256 channels 4400 / 820,
//                6000 / 4080, 10100 / 5100; the launch 4.7 / 2.9 and 5.9 / 3.9 us, 1.1 of them between launches; the network 224 / 169 us
//   order        work units are dealt channel-major to the XCDs, so that each L2 fetches an eighth of the weights
//
// DUAL: a residual block's last layer with its projection (see conv_dual.hip): some of the waves take the projection's K axis, the others the
// layer's own; the partial tiles are summed apart and the projection's sum is rescaled when they have met.
#include "conv_common.h"

namespace icnn {

constexpr int kLatWaves = 8;

struct LatOperand {
    int H, W, KW, sh, sw, ph, pw;
    int per_tap;                                     // steps of 64 per tap; TAPS == 2: 16-byte pieces
    unsigned mul_tap, mul_kw;                        // TAPS == 1: division by per_tap and KW, as mul_div has it
};
// What the first requests need is passed as single arguments: the command processor puts these into registers before a wave starts, the others
// arrive by scalar loads some 1000 clocks later.
struct LatFirst {
    const uint8_t *wp, *x;
    int ksteps, units, n_pt;                         // TAPS == 3: ksteps | n_pt << 16, units, the division by steps per tap as mul_div has it
    unsigned div_pt;                                 // unit / n_pt, as mul_div has it
    int in_cs, M;
    unsigned mul_howo, mul_wo, howo_wo, hw;          // TAPS == 3: as mul_div has them; two halves each
};
struct LatArgs {
    LatOperand op;
    unsigned mul_howo, mul_wo;                       // TAPS == 1, as mul_div has them
    int howo, wo, Cout;
    const int32_t *bias, *wsum, *pc;
    const void *res;
    void *out;
    int out_cs, out_co, mul, shift, lo, hi, out_mode;
    int res_mode, res_dtype, res_cs, res_mul, res_shift;   // with a projection: the rescale of its sums
    int fast, t_hi, rnd;                             // per layer: the 32-bit form of ConvArgs::rq24 (and res_fast) does
};
struct LatLanes {                                    // TAPS == 2
    int pieces;                                      // 16-byte pieces of K
    FastDiv div_tap, div_kw, div_howo, div_wo;
};
struct LatProj {                                     // DUAL
    const uint8_t *wp, *x;
    int ksteps, in_cs;
    const int32_t *bias;
    LatOperand op;
    LatLanes l;
    int split;                                       // waves from here on take the projection
    struct { int s0, n; } wave[kLatWaves];           // a wave's steps of 64 within its operand
};
template <bool DUAL, int TAPS>
struct LatMore {};                                   // the arguments that only some forms have
template <>
struct LatMore<false, 2> { LatLanes l; };
template <int TAPS>
struct LatMore<true, TAPS> {
    LatLanes l;
    LatProj p;
};

__device__ __forceinline__ int half_div(int n, unsigned mul)      // see mul_div
{
    return (int)__umulhi(2u * (unsigned)n, mul);
}

__device__ __forceinline__ void lat_drain(v4i &acc)
{
    asm volatile(ICNN_DRAIN_NOPS : "+v"(acc));
}

// CH, PX: 16-channel and 16-pixel groups of a tile.  NS: steps a wave has in flight; LOOP: it may have more of them.
// TAPS: 0 pointwise at stride 1; 1 any window, steps of 64 within a tap (input channels a multiple of 64), 2 any multiple of 16; 3 as 1, 3x3 at padding 1
// and one stride of 1 or 2.
template <int CH, int PX, int NS, bool LOOP, int TAPS, bool DUAL, bool U8>
__global__ __launch_bounds__(64 * kLatWaves, 4) void conv_lat_kernel(const uint8_t *wp, const uint8_t *x, int ksteps, int units, int n_pt, unsigned div_pt,
                                                               int in_cs, int M, unsigned k_mul_howo, unsigned k_mul_wo, unsigned k_howo_wo, unsigned k_hw, const LatArgs g,
                                                               const LatMore<DUAL, TAPS> m)
{
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    constexpr unsigned OOB = 0x80000000u;
    constexpr int PITCH = 16 * CH + 4;               // ints of one pixel's sums in LDS, with padding against bank conflicts
    constexpr int TILE = 16 * PX * PITCH;            // one wave's partial tile
    constexpr int COLS = 16 * CH, ROWS = 64 * kLatWaves / COLS, PER = (16 * PX + ROWS - 1) / ROWS;
    __shared__ __attribute__((aligned(16))) int part[kLatWaves * TILE];
    const int tid = threadIdx.x, lane = tid & 63, kq = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned k_mul_tap = (unsigned)n_pt;
    if (TAPS == 3) {
        n_pt = (int)((unsigned)ksteps >> 16);
        ksteps &= 0xffff;
    }
    const int u = (int)(blockIdx.x & 7) * ((units + 7) >> 3) + (int)(blockIdx.x >> 3);
    const bool mine = u < units;
    const int ct = half_div(u, div_pt), pt = u - ct * n_pt;
    int s0 = (int)((unsigned)(wave * ksteps) / kLatWaves), n = (int)((unsigned)(wave * ksteps + ksteps) / kLatWaves) - s0;
    LatOperand o = g.op;
    LatLanes ln = {};
    if constexpr (DUAL || TAPS == 2) ln = m.l;
    if constexpr (DUAL) {
        s0 = m.p.wave[wave].s0;
        n = m.p.wave[wave].n;
        if (wave >= m.p.split) {
            o = m.p.op; ln = m.p.l;
            wp = m.p.wp; x = m.p.x; ksteps = m.p.ksteps; in_cs = m.p.in_cs;
        }
    }
    n = mine ? n : 0;
    if (TAPS == 3) {
        // (the stride stands in the unused high bit of the image width's half)
        o.H = k_hw & 0xffff; o.W = k_hw >> 16 & 0x7fff; o.KW = 3;
        o.sh = o.sw = 1 + (int)(k_hw >> 31);
        o.ph = o.pw = 1;
        o.per_tap = (int)((unsigned)ksteps / 9u);
        o.mul_tap = k_mul_tap;
    }

    // ---- the other arguments are asked for here and waited for behind the weights' requests
    const unsigned mul_howo = TAPS == 3 ? k_mul_howo : g.mul_howo, mul_wo = TAPS == 3 ? k_mul_wo : g.mul_wo;
    const int howo = TAPS == 3 ? k_howo_wo & 0xffff : g.howo, wo = TAPS == 3 ? k_howo_wo >> 16 : g.wo, Cout = g.Cout, res_mode = g.res_mode, res_dtype = g.res_dtype, res_cs = g.res_cs;
    const int a_mul = g.mul, a_shift = g.shift, a_rm = g.res_mul, a_rs = g.res_shift;
    const int32_t *const bias = g.bias, *const pc = g.pc, *const wsums = g.wsum;
    const int32_t *pbias = nullptr;
    int split = kLatWaves;
    if constexpr (DUAL) { pbias = m.p.bias; split = m.p.split; }
    const void *const gres = g.res;
    void *const out = g.out;
    const int out_cs = g.out_cs, out_co = g.out_co, lo = g.lo, hi = g.hi, out_mode = g.out_mode, fast = g.fast, t_hi = g.t_hi, rnd = g.rnd;
    __builtin_amdgcn_sched_barrier(0);

    // ---- this lane's pixels as MFMA columns (the first one's place here, the second's relative to no other: they may be pictures apart)
    int iy0[PX], ix0[PX];
    unsigned base[PX];
    bool pok[PX];
    v4i fa[NS][CH], fx[NS][PX];
    v4i acc[CH][PX];
#pragma unroll
    for (int i = 0; i < CH; ++i)
#pragma unroll
        for (int j = 0; j < PX; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // (the descriptor ends behind this wave's last step: what it requests beyond comes as zeros)
    const int odd = CH == 1 ? (ct & 1) * 256 : 0;
    const unsigned woff = (unsigned)((kq >> 1) * 1024 + ((kq & 1) * 32 + l16) * 16);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(wp + ((unsigned)((CH == 1 ? ct >> 1 : ct) * ksteps + s0) * (unsigned)kChunkBytes + (unsigned)odd)), 0, max(n * kChunkBytes - odd, 0), 0x00020000);
    // (every place inside the tensor lies below 2 GiB, OOB above)
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);
    auto request_w = [&](int sb) {
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int i = 0; i < CH; ++i)
                fa[q][i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_w, woff + (unsigned)((sb + q) * kChunkBytes + i * 256), 0, 0));
    };
    unsigned off[PX];
    // TAPS == 1 and 3: lane i has the tap of the wave's step i of a batch and its distance from a pixel's first tap in bytes (an instruction costs such a
    // wave some 9 clocks, and per step in scalar registers this takes 19)
    int tap_h = 0, tap_w = 0, delta = 0;
    auto steps_to_lanes = [&](int sb) {
        const int sl = s0 + sb + lane, tap = half_div(sl, o.mul_tap);
        tap_h = TAPS == 3 ? tap * 11 >> 5 : half_div(tap, o.mul_kw);
        tap_w = tap - tap_h * o.KW;
        delta = (tap_h * o.W + tap_w) * in_cs + (sl - tap * o.per_tap) * 64;
    };
    auto request_x = [&](int sb) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int s = sb + q;
            if (TAPS == 0) {
                const int at = max(s0 + min(s, n - 1), 0) * 64;
#pragma unroll
                for (int j = 0; j < PX; ++j) fx[q][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off[j], at, 0));
            } else if (TAPS != 2) {
                const int kh = __builtin_amdgcn_readlane(tap_h, q), kw = __builtin_amdgcn_readlane(tap_w, q), to = __builtin_amdgcn_readlane(delta, q);
#pragma unroll
                for (int j = 0; j < PX; ++j) {
                    const bool in = ((unsigned)(iy0[j] + kh) < (unsigned)o.H) & ((unsigned)(ix0[j] + kw) < (unsigned)o.W);
                    fx[q][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_x, in ? base[j] + (unsigned)to : OOB, 0, 0));
                }
            } else {
                const int piece = 4 * (s0 + s) + kq;
                const int tap = fast_div(piece, ln.div_tap), c = piece - tap * o.per_tap;
                const int th = fast_div(tap, ln.div_kw), tw = tap - th * o.KW;
#pragma unroll
                for (int j = 0; j < PX; ++j) {
                    const bool in = s < n && piece < ln.pieces && (unsigned)(iy0[j] + th) < (unsigned)o.H && (unsigned)(ix0[j] + tw) < (unsigned)o.W;
                    fx[q][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                        rs_x, in ? base[j] + (unsigned)((th * o.W + tw) * in_cs + c * 16) : OOB, 0, 0));
                }
            }
        }
    };
    request_w(0);
    __builtin_amdgcn_sched_barrier(0);
    if (TAPS == 1 || TAPS == 3) {
        if (TAPS == 1)
            in_registers(mul_howo, mul_wo, howo, wo, o.H, o.W, o.KW, o.sh, o.sw, o.ph, o.pw, o.per_tap, o.mul_tap, o.mul_kw);
        steps_to_lanes(0);
    }
    if (TAPS == 2) in_registers(howo, wo, o.H, o.W, o.KW, o.sh, o.sw, o.ph, o.pw, o.per_tap);
#pragma unroll
    for (int j = 0; j < PX; ++j) {
        const int mp = pt * (16 * PX) + j * 16 + l16;
        pok[j] = mp < M;
        if (TAPS == 0) {
            off[j] = pok[j] ? (unsigned)(mp * in_cs + kq * 16) : OOB;
            continue;
        }
        const int mc = pok[j] ? mp : 0;
        const int pn = TAPS != 2 ? half_div(mc, mul_howo) : fast_div(mc, ln.div_howo);
        const int pr = mc - pn * howo;
        const int py = TAPS != 2 ? half_div(pr, mul_wo) : fast_div(pr, ln.div_wo), px = pr - py * wo;
        // (a pixel that is none lies outside every picture)
        iy0[j] = pok[j] ? py * o.sh - o.ph : -0x40000000;
        ix0[j] = px * o.sw - o.pw;
        base[j] = (unsigned)(((pn * o.H + py * o.sh - o.ph) * o.W + ix0[j]) * in_cs + (TAPS != 2 ? kq * 16 : 0));
    }
    request_x(0);
    __builtin_amdgcn_sched_barrier(0);
    in_registers(Cout, res_mode, res_dtype, res_cs, a_mul, a_shift, a_rm, a_rs, bias, pc, gres, out, out_cs, out_co, lo, hi, out_mode, fast, t_hi, rnd);
    if (U8) in_registers(wsums);
    if (DUAL) in_registers(pbias);
__builtin_amdgcn_sched_barrier(0);

    // ---- what this thread finishes: channel co of pixels p0, p0 + ROWS, ...
    // (of a chunk of 32 the matrix rows 16 i .. 16 i + 15 are channels 8 i .. 8 i + 7 and 16 more each)
    const int col = CH == 1 ? (tid & 7) + (tid & 8) * 2 + (ct & 1) * 8 : tid & 31, co = (CH == 1 ? ct >> 1 : ct) * 32 + col;
    const int at = (CH == 1 ? 0 : (col & 8) * 2) + (col & 3) + (col & 4) * 2 + (col >> 4) * 4;
    const int row = tid / COLS, p0 = pt * (16 * PX) + row;
    const bool cok = mine && co < Cout && row < 16 * PX;
    int b = 0, wsum = 0, pb = 0, res[PER], mul = a_mul, sh = a_shift, rm = a_rm, rs = a_rs;
    if (cok) {
        b = bias[co];
        if (U8) wsum = wsums[co];
        if (DUAL) pb = pbias[co];
        if (pc) {
            const int32_t *const gp = pc + (size_t)(co >> 4) * kPcGroupInts + (co & 15);
            mul = gp[kPcMul]; sh = gp[kPcShift];
            rm = gp[kPcResMul]; rs = gp[kPcResShift];
        }
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        res[e] = 0;
        if (!DUAL && res_mode != 0 && cok && p0 + e * ROWS < M) res[e] = load_elem(gres, (size_t)(p0 + e * ROWS) * res_cs + co, res_dtype);
    }
    __builtin_amdgcn_sched_barrier(0);               // all requests go out before the first use

    for (int sb = 0;;) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
#pragma unroll
            for (int j = 0; j < PX; ++j)
                if (U8) fx[q][j] ^= (int)0x80808080;
#pragma unroll
            for (int i = 0; i < CH; ++i)
#pragma unroll
                for (int j = 0; j < PX; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[q][i], fx[q][j], acc[i][j], 0, 0, 0);
        }
        sb += NS;
        if (!LOOP || sb >= n) break;
        request_w(sb);
        if (TAPS == 1 || TAPS == 3) steps_to_lanes(sb);
        request_x(sb);
    }
#pragma unroll
    for (int i = 0; i < CH; ++i)
#pragma unroll
        for (int j = 0; j < PX; ++j) lat_drain(acc[i][j]);
#pragma unroll
    for (int i = 0; i < CH; ++i)
#pragma unroll
        for (int j = 0; j < PX; ++j) *(v4i *)(part + wave * TILE + (j * 16 + l16) * PITCH + i * 16 + kq * 4) = acc[i][j];
    __syncthreads();

    if (!cok) return;
    if (U8) b += 128 * wsum;
    sh &= 63;
    rs &= 63;
    int sum[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int *const d = part + (row + e * ROWS) * PITCH + at;
        int psum = pb;
        sum[e] = b;
#pragma unroll
        for (int w = 0; w < kLatWaves; ++w) {
            const int v = d[w * TILE];
            const int own = DUAL ? (w < split ? -1 : 0) : -1;
            sum[e] += v & own;
            if (DUAL) psum += v & ~own;
        }
        // (with a projection the host has proved that the merged sum stays inside int32)
        if (DUAL) sum[e] += (int)rsr64((int64_t)psum * rm, rs);
    }
    const size_t oo = (size_t)p0 * out_cs + out_co + co;
    if (out_mode == 3 || !fast) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            if (p0 + e * ROWS >= M) break;
            int64_t t = sum[e];
            const int64_t skip = !DUAL && res_mode != 0 ? rsr64((int64_t)res[e] * rm, rs) : 0;
            if (!DUAL && res_mode == 1) t += skip;
            const int q = sat32(t);
            const size_t to = oo + (size_t)(e * ROWS) * out_cs;
            if (out_mode == 3) {
                ((int32_t *)out)[to] = q;
            } else {
                int64_t v = rsr64((int64_t)q * mul, sh);
                if (!DUAL && res_mode == 2) v += skip;
                ((uint8_t *)out)[to] = (uint8_t)clampi64(v, lo, hi);
            }
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        int t = sum[e];
        if (!DUAL && res_mode != 0)
            t = __builtin_elementwise_add_sat(t, (int)((__umul24((uint32_t)res[e], (uint32_t)rm) + (uint32_t)((1 << rs) >> 1)) >> rs));
        sum[e] = (int)((__umul24((uint32_t)med3_v0s(t, t_hi), (uint32_t)mul) + (uint32_t)rnd) >> sh);
    }
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (p0 + e * ROWS < M) ((uint8_t *)out)[oo + (size_t)(e * ROWS) * out_cs] = (uint8_t)sum[e];
#endif
}

// ------------------------------------------------------------------ dispatch
// n / d = high word of 2 n * ceil(2^31 / d) for n * d < 2^31: the factor's excess over 2^31 / d adds less than n / 2^31 < 1 / d
static unsigned mul_div(int d)
{
    return (unsigned)(((1ull << 31) + (unsigned)d - 1) / (unsigned)d);
}

// (with steps within taps: fewer than 2^15 of them)
static LatOperand lat_operand(int H, int W, int Cin, int KW, int sh, int sw, int ph, int pw, int taps)
{
    LatOperand o;
    o.H = H; o.W = W; o.KW = KW; o.sh = sh; o.sw = sw; o.ph = ph; o.pw = pw;
    o.per_tap = Cin / (taps == 2 ? 16 : 64);
    o.mul_tap = o.mul_kw = 0;
    if (taps == 1 || taps == 3) {
        o.mul_tap = mul_div(o.per_tap);
        o.mul_kw = mul_div(KW);
    }
    return o;
}

static LatLanes lat_lanes(const LatOperand &o, int KH, int howo, int wo)
{
    return LatLanes{KH * o.KW * o.per_tap, make_fast_div((unsigned)o.per_tap), make_fast_div((unsigned)o.KW), make_fast_div((unsigned)howo),
                    make_fast_div((unsigned)wo)};
}

// A block's last layer with its projection: the waves go to the two K axes in proportion to their steps
static int lat_split(const ConvArgs &a, const ProjArgs &q)
{
    const int all = a.ksteps + q.ksteps, main = (int)(((long long)kLatWaves * a.ksteps + all / 2) / all);
    return main < 1 ? 1 : (main > kLatWaves - 1 ? kLatWaves - 1 : main);
}
struct LatShare {
    int s0, n;
};
static LatShare lat_share(int main_steps, int proj_steps, int split, int w)
{
    const bool first = w < split;
    const long long k = first ? main_steps : proj_steps, n = first ? split : kLatWaves - split, i = first ? w : w - split;
    const int s0 = (int)(k * i / n);
    return LatShare{s0, (int)(k * (i + 1) / n) - s0};
}

static bool lat_shape_ok(const ConvArgs &a)
{
    return a.Cin % 16 == 0 && a.in_cs % 16 == 0 && !((uintptr_t)a.x & 15) && a.in_xor == 0 && a.x_bytes < 0x7fffff00u && a.KH * a.KW <= 1024 &&
           a.ksteps == (a.KH * a.KW * a.Cin + 63) / 64 && (a.Cout + 31LL) / 32 * 2 * ((a.M + 15LL) / 16) * ((a.M + 15LL) / 16) < 0x7fffffffLL && a.wp_bytes < 0x7fffff00u;
}

// The tile, and what a launch costs with it: rounds of one unit per compute unit times what a unit moves through its memory path (16 x 16,
// 32 x 16 and 32 x 32 move 2 : 3 : 4 parts; the last has half the waves' requests behind one another and counts 6).  Microseconds over layers of
// residual networks, replayed as a graph over 16 sets of weights (16 x 16 / 32 x 16 / 32 x 32; costs): 3x3 of 256 channels on 14 x 14, one image
// 3.1 / 3.4 / 4.6 (2, 3, 6), two 4.4 / 3.5 / 4.7 (4, 3, 6), four 6.7 / 5.1 / 4.8 (8, 6, 6), ten 12.2 / 8.3 / 7.5 (16, 12, 12); 512 -> 2048 on 7 x 7, one
// 2.6 / 2.4 / 3.1 (4, 3, 6), two 3.1 / 2.7 / 3.2 (8, 6, 6); 3x3 of 512 channels, two 4.5 / 5.3 / 7.6 (2, 3, 6), four 6.7 / 5.3 / 7.6 (4, 3, 6).  At equal cost
// the smaller tile with fewer than 16 steps of K, the larger one from there on.
struct LatTile {
    int ch, px;
    long long cost;
};
constexpr long long kLatCus = 256;
static LatTile lat_tile(long long M, long long Cout, int ksteps)
{
    const long long chunks = (Cout + 31) / 32, narrow = (M + 15) / 16, wide = (M + 31) / 32;
    auto rounds = [](long long units) { return (units + kLatCus - 1) / kLatCus; };
    LatTile t = {2, 1, 3 * rounds(chunks * narrow)};
    const long long small = 2 * rounds(2 * chunks * narrow), large = 6 * rounds(chunks * wide);
    if (small < t.cost) t = LatTile{1, 1, small};
    if (large < t.cost || (large == t.cost && ksteps >= 16)) t = LatTile{2, 2, large};
    return t;
}

// Against the tile kernels: while all units of 32 channels x 32 pixels are on the chip at once, two workgroups of eight waves to a compute unit.
// Against the kernel whose waves split K over a patch in LDS (conv_deep.hip), which is nearer with 144 fragments of K: one unit per compute unit
// (3x3 of 512 channels on 7 x 7: 256 units 7.8 / 8.7, 320 units 12.7 / 8.7).
constexpr int kLatOnePerCu = 256, kLatTwoPerCu = 512;
static bool lat_worth(int M, int Cout, int frags, int most_units)
{
    const long long units = (long long)((Cout + 31) / 32) * ((M + 31) / 32);
    return frags >= 4 && units <= most_units;
}

// Against the kernel with weights straight into registers (conv_flat.hip), which has one workgroup per 128 channels x 64 pixels: here up to cost 6, and up
// to 9 where that kernel's few workgroups have long K loops to themselves (at 12 the two are level, and between other layers this one loses: nine images in
// the 50-layer network, 3x3 of 256 channels at stride 2 9.0 / 8.2, 1024 -> 256 5.5 / 5.2).  Microseconds here / there, costs in brackets: 3x3 of 256 channels on
// 14 x 14 (6) 4.8 / 6.2, (9) 6.6 / 6.3; of 128 on 28 x 28 (6) 3.9 / 4.4, (9) 4.9 / 4.4; of 64 on 56 x 56 (6) 2.8 / 3.8, (12) 3.5 / 3.8, (18) 4.2 / 3.9;
// stride 2, 256 channels on 28 x 28 (9) 6.7 / 7.7, (12) 7.5 / 7.7, (15) 10.3 / 7.8; 512 channels on 14 x 14 (6) 8.0 / 11.5, (9) 11.5 / 11.3;
// 1024 -> 256 (9) 3.9 / 4.9, (12) 4.4 / 4.9, (15) 5.5 / 5.0; 2048 -> 512 (6) 5.2 / 7.3, (9) 7.0 / 7.3; 512 -> 2048 (9) 3.2 / 3.8, (12) 3.4 / 3.8, (15) 4.2 / 3.9;
// 512 -> 128 (12) 3.3 / 3.5, (15) 4.1 / 3.6; 256 -> 1024 (6) 2.5 / 2.9, (12) 3.1 / 2.9; 128 -> 512 (12) 3.1 / 2.6.
bool conv_lat_before_flat(const ConvArgs &a)
{
    if (!lat_shape_ok(a) || g_tuning.no_lat) return false;
    const long long cost = lat_tile(a.M, a.Cout, a.ksteps).cost;
    const bool longer = a.KH == 1 && a.sh == 1 ? a.ksteps >= 8 : (a.sh == 2 ? a.ksteps <= 36 : a.ksteps <= 9) && a.KH == 3;
    return cost <= (longer ? 9 : 6);
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

namespace {
struct LatPlan {
    const ConvArgs &a;
    const ProjArgs *q;
    int ch, px, steps;                               // tile; most steps of one wave
    int taps;
    LatFirst f;
};

template <int CH, int PX, int NS, bool LOOP, int TAPS>
hipError_t go_lat(const LatPlan &p, const LatArgs &g, hipStream_t st)
{
    const dim3 grid((unsigned)(8 * ((p.f.units + 7) / 8))), block(64 * kLatWaves);
    const LatFirst &f = p.f;
    auto launch = [&](auto kernel, const auto &more) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, f.wp, f.x, f.ksteps, f.units, f.n_pt, f.div_pt, f.in_cs, f.M, f.mul_howo, f.mul_wo,
                           f.howo_wo, f.hw, g, more);
        return hipGetLastError();
    };
    const ConvArgs &a = p.a;
    if (p.q) {
        if constexpr (TAPS == 1 || TAPS == 2) {
            const ProjArgs &q = *p.q;
            LatMore<true, TAPS> m;
            m.l = TAPS == 2 ? lat_lanes(g.op, a.KH, g.howo, g.wo) : LatLanes{};
            m.p.wp = q.wp; m.p.x = q.x; m.p.ksteps = q.ksteps; m.p.in_cs = q.in_cs;
            m.p.bias = q.bias;
            m.p.op = lat_operand(q.H, q.W, q.Cin, 1, q.sh, q.sw, 0, 0, TAPS);
            m.p.l = TAPS == 2 ? lat_lanes(m.p.op, 1, g.howo, g.wo) : LatLanes{};
            m.p.split = lat_split(a, q);
            for (int w = 0; w < kLatWaves; ++w) {
                const LatShare s = lat_share(a.ksteps, q.ksteps, m.p.split, w);
                m.p.wave[w].s0 = s.s0;
                m.p.wave[w].n = s.n;
            }
            return launch(conv_lat_kernel<CH, PX, NS, LOOP, TAPS, true, false>, m);
        }
        return hipErrorInvalidValue;
    }
    LatMore<false, TAPS> m;
    if constexpr (TAPS == 2) m.l = lat_lanes(g.op, a.KH, g.howo, g.wo);
    if (a.frag_xor) return launch(conv_lat_kernel<CH, PX, NS, LOOP, TAPS, false, true>, m);
    return launch(conv_lat_kernel<CH, PX, NS, LOOP, TAPS, false, false>, m);
}
template <int CH, int PX, int NS, bool LOOP>
hipError_t pick_taps(const LatPlan &p, const LatArgs &g, hipStream_t st)
{
    if (p.taps == 0) return go_lat<CH, PX, NS, LOOP, 0>(p, g, st);
    if (p.taps == 3) return go_lat<CH, PX, NS, LOOP, 3>(p, g, st);
    return p.taps == 1 ? go_lat<CH, PX, NS, LOOP, 1>(p, g, st) : go_lat<CH, PX, NS, LOOP, 2>(p, g, st);
}
}  // namespace

static hipError_t launch_lat(const ConvArgs &a, const ProjArgs *q, hipStream_t st)
{
    LatArgs g;
    LatPlan p = {a, q, 2, 2, 0, 0, {}};
    // (what mul_div does not reach is placed lane by lane)
    const bool lanes = a.Cin % 64 != 0 || (q && q->Cin % 64 != 0) || a.ksteps > 0x7fff || (q && q->ksteps > 0x7fff) || a.M > 0x7fff;
    if (!q && a.Cin % 64 == 0 && a.KH == 1 && a.KW == 1 && a.sh == 1 && a.sw == 1 && a.ph == 0 && a.pw == 0) p.taps = 0;
    else if (lanes) p.taps = 2;
    else if (!q && a.KH == 3 && a.KW == 3 && a.sh == a.sw && a.sh <= 2 && a.ph == 1 && a.pw == 1 && a.H <= 0x7fff && a.W <= 0x7fff) p.taps = 3;
    else p.taps = 1;
    g.op = lat_operand(a.H, a.W, a.Cin, a.KW, a.sh, a.sw, a.ph, a.pw, p.taps);
    p.steps = (a.ksteps + kLatWaves - 1) / kLatWaves;
    if (q) {
        p.steps = 0;
        for (int w = 0, split = lat_split(a, *q); w < kLatWaves; ++w) {
            const int n = lat_share(a.ksteps, q->ksteps, split, w).n;
            p.steps = n > p.steps ? n : p.steps;
        }
    }
    const LatTile tile = lat_tile(a.M, a.Cout, a.ksteps + (q ? q->ksteps : 0));
    p.ch = g_tuning.lat > 1 ? (g_tuning.lat == 2 ? 1 : 2) : tile.ch;
    p.px = g_tuning.lat > 1 ? (g_tuning.lat == 4 ? 2 : 1) : tile.px;
    const int cts = (a.Cout + 31) / 32 * (p.ch == 1 ? 2 : 1), n_pt = (a.M + 16 * p.px - 1) / (16 * p.px);
    const long long units = (long long)cts * n_pt;
    if (units < 1 || units * n_pt >= 0x7fffffffLL) return hipErrorInvalidValue;
    g.howo = a.Ho * a.Wo; g.wo = a.Wo; g.Cout = a.Cout;
    g.mul_howo = g.mul_wo = 0;
    if (p.taps == 1 || p.taps == 3) {
        g.mul_howo = mul_div(g.howo);
        g.mul_wo = mul_div(g.wo);
    }
    p.f = LatFirst{a.wp, a.x, a.ksteps, (int)units, n_pt, mul_div(n_pt), a.in_cs, a.M, g.mul_howo, g.mul_wo, 0, 0};
    if (p.taps == 3) {
        p.f.ksteps = (int)((unsigned)a.ksteps | (unsigned)n_pt << 16);
        p.f.n_pt = (int)g.op.mul_tap;
        p.f.howo_wo = (unsigned)g.howo | (unsigned)g.wo << 16;
        p.f.hw = (unsigned)a.H | (unsigned)a.W << 16 | (unsigned)(a.sh - 1) << 31;
    }
    g.bias = a.bias; g.wsum = a.wsum; g.pc = a.pc; g.res = a.res; g.out = a.out;
    g.out_cs = a.out_cs; g.out_co = a.out_co; g.mul = a.mul; g.shift = a.shift; g.lo = a.lo; g.hi = a.hi; g.out_mode = a.out_mode;
    g.res_mode = a.res_mode; g.res_dtype = a.res_dtype; g.res_cs = a.res_cs;
    g.res_mul = q ? q->res_mul : a.res_mul;
    g.res_shift = q ? q->res_shift : a.res_shift;
    g.fast = a.rq24 && !a.pc && (a.res_mode == 0 || (a.res_mode == 1 && a.res_fast));
    g.t_hi = a.t_hi; g.rnd = a.rnd;
    // As many loads in flight as the waves have steps: a missing one is still requested and multiplied.  One image, its layers replayed as a graph over 16 sets
    // of weights, us with the next larger number / as here, 16 x 16, 32 x 16 and 32 x 32: one step (256 -> 1024) 4.2 / 3.2, 3.5 / 2.9, 3.6 / 3.1; two (1024 -> 256)
    // 2.9 / 2.7, 3.1 / 2.8, 3.9 / 3.4; three (3x3 of 128 channels) 4.8 / 3.8, 3.9 / 3.3, 5.1 / 4.0.  Nine steps (3x3 of 512) at once where they have the registers, in
    // 16 x 16: 4.8 / 4.6 against rounds of five.
    if (p.ch == 1) {
        if (p.steps <= 1) return pick_taps<1, 1, 1, false>(p, g, st);
        if (p.steps <= 2) return pick_taps<1, 1, 2, false>(p, g, st);
        if (p.steps <= 3) return pick_taps<1, 1, 3, false>(p, g, st);
        if (p.steps <= 5) return pick_taps<1, 1, 5, false>(p, g, st);
        return pick_taps<1, 1, 9, true>(p, g, st);
    }
    if (p.px == 1) {
        if (p.steps <= 1) return pick_taps<2, 1, 1, false>(p, g, st);
        if (p.steps <= 2) return pick_taps<2, 1, 2, false>(p, g, st);
        if (p.steps <= 3) return pick_taps<2, 1, 3, false>(p, g, st);
        return pick_taps<2, 1, 5, true>(p, g, st);
    }
    if (p.steps <= 1) return pick_taps<2, 2, 1, false>(p, g, st);
    if (p.steps <= 2) return pick_taps<2, 2, 2, false>(p, g, st);
    if (p.steps <= 3) return pick_taps<2, 2, 3, false>(p, g, st);
    return pick_taps<2, 2, 5, true>(p, g, st);
}

hipError_t launch_conv_lat(const ConvArgs &a, hipStream_t st)
{
    return launch_lat(a, nullptr, st);
}

bool conv_lat_dual_applies(const ConvArgs &a, const ProjArgs &q)
{
    if (!lat_shape_ok(a) || g_tuning.no_lat || q.Cin % 16 || q.in_cs % 16 || ((uintptr_t)q.x & 15) || a.frag_xor || q.wp_bytes >= 0x7fffff00u) return false;
    return g_tuning.lat || lat_worth(a.M, a.Cout, (a.Cin + q.Cin) / 32, kLatTwoPerCu);
}
hipError_t launch_conv_lat_dual(const ConvArgs &a, const ProjArgs &q, hipStream_t st)
{
    return launch_lat(a, &q, st);
}

}  // namespace icnn
