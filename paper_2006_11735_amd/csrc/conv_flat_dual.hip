// A block's closing 1x1 layer with the projection of its skip operand (conv_dual.hip has the arithmetic) where the projection reads twice the
// closing layer's channels: as conv_flat.hip, each wave's weights straight into its registers.
//
//   tile     64 consecutive output pixels x 128 channels, a wave per 32 channels
//   input    segments of CH channels, 128 or 256: the projection's at their strided pixels, the closing layer's.  Two LDS
//            buffers: one is filled while the other is multiplied.  Rows padded by 16 bytes
//   weights  a group for every segment, fetched eight K steps ahead, across the segments
//
// Two to four workgroups share a compute unit, whose memory path (64 to 72 bytes a clock) is what bounds it: 98 KB of weights and 48 KB of input for
// 6144 clocks of matrix instructions at 256 + 512 channels, 18.1 us for 64 images of 14 x 14 -> 1024 channels where both operands through LDS
// take 23.7.  Segments of 256 channels rather than of all 512 leave room for a third workgroup (128 images of 7 x 7: 30.3 us against 33.1).
#include "conv_common.h"

#include <type_traits>

namespace icnn {

// The leading arguments are in registers when a wave starts (as in conv_flat.hip): a workgroup's place, where a pixel lies in the projection's input (image, row,
// pixel: bytes from one to the next); the others arrive while the first copies are requested.  (64 images, 128 + 256 -> 512 channels on 28 x 28: 22.6 -> 21.9 us.)
// PS segments of the projection, MS of the closing layer, G steps of 64 each.  FORM: 1 requantisation as a product's high word (rq_fast), 8-bit output; 3 as 1, to bytes (requant_fits_byte); 0 any form of one
// pair per layer; 2 per output channel.
template <int G, int PS, int MS, int FORM>
__global__ __launch_bounds__(256, 2) void conv_flat_dual_kernel(const uint8_t *proj_x, const int M, const unsigned div_mul, const unsigned tiles, const int howo,
                                                                const int wo, const unsigned mul_howo, const unsigned mul_wo, const unsigned shifts,
                                                                const unsigned image, const unsigned row, const unsigned pixel, const ConvArgs a,
                                                                const ProjArgs q)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    constexpr int CH = 64 * G, AP = CH + 16, PIECES = AP / 16, PX = 64, NS = 8 / G, ALL = PS + MS;
    constexpr int BUF = PX * AP;                       // a whole number of KiB: 64 rows of PIECES pieces

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    // LDS: two buffers | the projection's biases | the closing layer's | where each pixel is in the projection's input | FORM 2: rescale factors, shifts, factors
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    int32_t *const tab = (int32_t *)(lds + 2 * BUF);
    unsigned *const rtab = (unsigned *)(tab + 256);
    int32_t *const rescale = tab + 256 + PX, *const factors = rescale + 256 + wave * 32;

    const int n_ct = (int)(tiles & 0xffff), n_pt = (int)(((unsigned)M + PX - 1) / PX), n_tiles = n_ct * n_pt;
    const int logical = (int)(blockIdx.x & 7) * ((n_tiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (logical >= n_tiles) return;
    const bool by_pt = tiles >> 30 & 1;
    const int major = fast_div_packed(logical, div_mul, tiles >> 16 & 0xff, tiles >> 24 & 0x3f), minor = logical - major * (by_pt ? n_pt : n_ct);
    const int ct = by_pt ? major : minor, pt = by_pt ? minor : major;
    const int p0 = pt * PX, co_tile = ct * 128, co_wave = co_tile + wave * 32;

    // ---- weights: group k of this wave's chunks, the projection's first, in slot k % NS of the ring
    const uint8_t *const wpp = q.wp + (size_t)(co_wave >> 5) * (PS * G * kChunkBytes);
    const uint8_t *const wpm = a.wp + (size_t)(co_wave >> 5) * (MS * G * kChunkBytes);
    v4i ring[NS][2 * G];
    const int lane16 = lane * 16;
    auto load_frag = [&](auto k_tag, auto f_tag) __attribute__((always_inline)) {
        constexpr int k = decltype(k_tag)::value, f = decltype(f_tag)::value;
        if constexpr (k < ALL) {
            const uint8_t *const from = k < PS ? wpp + k * (G * kChunkBytes) : wpm + (k - PS) * (G * kChunkBytes);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)from, 0, G * kChunkBytes, 0x00020000);
            ring[k % NS][f] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane16 + (f & 1) * 1024, (f >> 1) * kChunkBytes, 0);
        }
    };
    [[maybe_unused]] bool one_product = false;
    // ---- prologue: where the pixels are, then the projection's segments, the tables and the ring's first groups in flight together
    if (tid < PX) {
        const int p = p0 + tid;
        unsigned off = OOB;
        if (p < M) {
            const int n = fast_div_packed(p, mul_howo, shifts & 0xff, shifts >> 8 & 0xff), at = p - n * howo;
            const int y = fast_div_packed(at, mul_wo, shifts >> 16 & 0xff, shifts >> 24);
            off = n * image + y * row + (at - y * wo) * pixel;
        }
        rtab[tid] = off;
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rs_p = __builtin_amdgcn_make_buffer_rsrc((void *)proj_x, 0, 0x7fffff00, 0x00020000);    // (every place inside the tensor lies below 2 GiB, OOB above)
    const __amdgpu_buffer_rsrc_t rs_m = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.x_bytes, 0x00020000);
    // 16-byte piece i of a buffer is piece i % PIECES of row i / PIECES, the last of a row padding
    auto copy = [&](int seg) __attribute__((always_inline)) {
        uint8_t *const to = lds + (seg & 1) * BUF;
        for (int c = wave; c < PIECES; c += 4) {
            const unsigned i = c * 64 + lane, r = i / PIECES, piece = i - r * PIECES;
            if (seg < PS) {
                const unsigned off = piece < PIECES - 1 ? rtab[r] + piece * 16 : OOB;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_p, (__attribute__((address_space(3))) void *)(to + c * 1024), 16, off, seg * CH, 0, 0);
            } else {
                const unsigned off = piece < PIECES - 1 && p0 + (int)r < M ? (p0 + r) * (unsigned)a.in_cs + piece * 16 : OOB;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_m, (__attribute__((address_space(3))) void *)(to + c * 1024), 16, off, (seg - PS) * CH, 0, 0);
            }
        }
    };
    copy(0);
    copy(1);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    in_registers(q.bias, a.bias, q.wp, a.wp, a.x, a.x_bytes, a.in_cs, q.res_mul, q.res_shift, a.out, a.out_cs, a.out_co, a.lo, a.hi);
    if constexpr (FORM == 1 || FORM == 3) in_registers(a.mul_hi);
    {
        const int co = co_tile + (tid & 127);
        tab[tid] = tid < 128 ? q.bias[co] : a.bias[co];
        if constexpr (FORM == 2) rescale[tid] = a.pc[(co >> 4) * kPcGroupInts + (tid < 128 ? kPcResMul : kPcResShift) + (co & 15)];
        if constexpr (FORM == 2) {
            int factor, none, position;
            const bool ok = pc_hi_channel(a.pc, co_wave + col, false, factor, none, position);
            one_product = a.pc_fast_ok && __builtin_amdgcn_ballot_w64(!ok) == 0;
            if (half == 0) factors[col] = factor;
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    constexpr int FIRST = NS < ALL ? NS : ALL;
    static_for<FIRST * 2 * G>([&](auto i_tag) __attribute__((always_inline)) {
        constexpr int i = decltype(i_tag)::value;
        load_frag(std::integral_constant<int, i / (2 * G)>{}, std::integral_constant<int, i % (2 * G)>{});
    });
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    ICNN_WAIT_VMCNT(2 * G * FIRST);                    // this wave's copies have landed: the ring's loads are younger
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();                      // ... everybody's
    asm volatile("" ::: "memory");

    v16i acc[1][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[0][j] = bias16(tab + wave * 32 + half * 16);

    constexpr int NB = 2 * G < 4 ? 2 * G : 4, AHEAD = NB - 1, T = 2 * G;      // fragments in flight; half steps of a segment
    const int row0 = col * AP + half * 16;
    auto segment = [&](auto seg_tag) __attribute__((always_inline)) {
        constexpr int seg = decltype(seg_tag)::value;
        const uint8_t *const from = lds + (seg & 1) * BUF + row0;
        v4i bf[NB][2];
#pragma unroll
        for (int h = 0; h < AHEAD; ++h)
#pragma unroll
            for (int j = 0; j < 2; ++j) bf[h][j] = *(const v4i *)(from + j * (32 * AP) + h * 32);
        static_for<T>([&](auto h_tag) __attribute__((always_inline)) {
            constexpr int h = decltype(h_tag)::value, hn = h + AHEAD;
            static_for<2>([&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                acc[0][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[seg % NS][h], bf[h % NB][j], acc[0][j], 0, 0, 0);
                asm volatile("" : "+v"(acc[0][j]));        // here, not wherever the sums are needed
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (hn < T) bf[hn % NB][j] = *(const v4i *)(from + j * (32 * AP) + hn * 32);
                if constexpr (j == 1) load_frag(std::integral_constant<int, seg + NS>{}, h_tag);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // ---- the projection's sums at the closing layer's ratio, on its biases
    auto rescale_sums = [&]() __attribute__((always_inline)) {
        mfma_drain(acc);
        const int32_t *const bias = tab + 128 + wave * 32 + half * 16, *const rm = rescale + wave * 32 + half * 16;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const v4i b = *(const v4i *)(bias + 4 * q4);
            v4i mu, sf;
            if constexpr (FORM == 2) {
                mu = *(const v4i *)(rm + 4 * q4);
                sf = *(const v4i *)(rm + 128 + 4 * q4);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t s = acc[0][j][4 * q4 + e];
                    acc[0][j][4 * q4 + e] = (int)(FORM == 2 ? rsr64(s * mu[e], sf[e] & 63) : rsr64(s * q.res_mul, q.res_shift)) + b[e];
                }
        }
    };
    static_for<ALL>([&](auto s_tag) __attribute__((always_inline)) {
        constexpr int seg = decltype(s_tag)::value;
        if constexpr (seg > 1) {
            // this segment's copies have landed: younger than they are the ring's loads of the segment before
            asm volatile("" ::: "memory");
            ICNN_WAIT_VMCNT((seg - 1 + NS < ALL ? 2 * G : 0));
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        segment(s_tag);
        if constexpr (seg + 2 < ALL) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();              // everybody has read the buffer
            asm volatile("" ::: "memory");
            copy(seg + 2);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (seg == PS - 1) rescale_sums();
    });

    mfma_drain(acc);
    const int pw = p0;
    if (FORM == 1 || FORM == 3 || (FORM == 2 && one_product)) {
        const SkipMul none = {0, 0, 0};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = pw + 32 * j + col;
            v4i w;
            if constexpr (FORM == 2) w = epilogue_pc_hi16<0>(a, factors + half * 16, factors, nullptr, acc[0][j], v4i{0, 0, 0, 0});
            else w = epilogue_hi16<0, FORM == 3>(a, none, acc[0][j], v4i{0, 0, 0, 0});
            if (p < M) *(v4i *)((uint8_t *)a.out + (size_t)p * a.out_cs + a.out_co + co_wave + half * 16) = w;
        }
    } else {
        const v4i none[1][2] = {{v4i{0, 0, 0, 0}, v4i{0, 0, 0, 0}}};           // the layer's arguments carry no skip operand here
        if constexpr (FORM == 2) epilogue_pc_tiles<1, 2>(a, acc, co_wave, pw, lane, none, a.pc, 0);
        else epilogue_tiles<1, 2>(a, acc, co_wave, pw, lane, none);
    }
#endif
}

bool conv_flat_dual_applies(const ConvArgs &a, const ProjArgs &q)
{
    if (g_tuning.flat == 2) return false;
    return a.KH == 1 && a.KW == 1 && a.sh == 1 && a.sw == 1 && a.ph == 0 && a.pw == 0 && (a.Cin == 128 || a.Cin == 256 || a.Cin == 512) && q.Cin == 2 * a.Cin && a.Cout % 128 == 0 &&
           a.vec_bias && q.vec_bias && !a.frag_xor && !a.in_xor && a.M <= 0x7fffffff - 64 && a.Cout / 128 <= 0xffff && q.x_bytes < 0x7fffff00u;
}

hipError_t launch_conv_flat_dual(const ConvArgs &args, const ProjArgs &q, hipStream_t st)
{
    ConvArgs a = args;
    if (!conv_flat_dual_applies(a, q) || !finish_args(a, 128, 64)) return hipErrorInvalidValue;
    a.div_howo = make_fast_div((unsigned)(a.Ho * a.Wo));
    a.div_wo = make_fast_div((unsigned)a.Wo);
    const double wt = (double)a.wp_bytes + q.wp_bytes, in = (double)a.x_bytes + (double)a.M * q.Cin;       // as in conv_flat.hip
    const bool by_pt = a.n_ct > 1 && wt * 8 + in > wt * (a.n_ct < 8 ? 8 / a.n_ct : 1) + in * (a.n_ct < 8 ? a.n_ct : 8);
    const FastDiv by = make_fast_div((unsigned)(by_pt ? a.n_tiles / a.n_ct : a.n_ct)), dh = a.div_howo, dw = a.div_wo;
    const unsigned tiles = (unsigned)a.n_ct | by.s1 << 16 | by.s2 << 24 | (by_pt ? 1u << 30 : 0u), shifts = dh.s1 | dh.s2 << 8 | dw.s1 << 16 | dw.s2 << 24;
    const size_t lds_bytes = 2 * 64 * ((a.Cin == 128 ? 128 : 256) + 16) + (256 + 64 + (a.pc ? 384 : 0)) * 4;
    auto go = [&](auto kernel) -> hipError_t {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * a.per_xcd)), dim3(256), lds_bytes, st, q.x, a.M, by.mul, tiles, a.Ho * a.Wo, a.Wo, dh.mul, dw.mul, shifts,
                           (unsigned)q.H * q.W * q.in_cs, (unsigned)q.sh * q.W * q.in_cs, (unsigned)q.sw * q.in_cs, a, q);
        return hipGetLastError();
    };
#define ICNN_FLAT_DUAL(G, PS, MS) \
    (a.pc ? go(conv_flat_dual_kernel<G, PS, MS, 2>) : a.rq_fast && a.epi_vec ? requant_fits_byte(a) ? go(conv_flat_dual_kernel<G, PS, MS, 3>) : go(conv_flat_dual_kernel<G, PS, MS, 1>) : go(conv_flat_dual_kernel<G, PS, MS, 0>))
    return a.Cin == 128 ? ICNN_FLAT_DUAL(2, 2, 1) : a.Cin == 256 ? ICNN_FLAT_DUAL(4, 2, 1) : ICNN_FLAT_DUAL(4, 4, 2);
#undef ICNN_FLAT_DUAL
}

}  // namespace icnn
