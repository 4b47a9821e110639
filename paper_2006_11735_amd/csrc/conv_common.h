// Device and host helpers shared by the convolution kernels (tile layout, epilogue,
// bias rows, fast division, counted waits).  Internal; not installed.
#pragma once
#include "icnn_device.h"

#include <type_traits>

namespace icnn {

typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load, dword aligned

// LDS tile layout of one K step (both kernels):
//   A (weights): BM*64 bytes in packed-fragment order, i.e. a straight copy of
//      BM/32 consecutive 2 KiB chunks of the packed weights.
//   B (activations): BP rows of 64 bytes (one output pixel each); the 16-byte slot
//      s of row r lives at slot s ^ ((r >> 2) & 3), which makes both the row-wise
//      fill and the column-wise fragment reads free of bank conflicts.
__device__ __forceinline__ int b_slot_offset(int row, int slot)
{
    return row * 64 + ((slot ^ ((row >> 2) & 3)) << 4);
}

// ---------------------------------------------------------------- epilogue
// Every call handles channels co0..co0+15 (co0 a multiple of 16) of output pixel p,
// held in one lane's accumulator registers, which were initialised with the bias
// (so they hold Y = U + b).  Then (Section 4.1)
// the rescaled skip operand, then (Section 3.2.1) requantisation and the clamp.

// any alignment, any tail: one element at a time, 64-bit arithmetic throughout
__device__ __forceinline__ void epilogue_slow(const ConvArgs &a, const v16i &acc, int p, int co0, int nv)
{
    const size_t ro = (size_t)p * a.res_cs + co0;
    const size_t oo = (size_t)p * a.out_cs + a.out_co + co0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (r >= nv) break;
        int64_t t = acc[r];
        int64_t skip = 0;
        if (a.res_mode != 0) skip = rsr64((int64_t)load_elem(a.res, ro + r, a.res_dtype) * a.res_mul, a.res_shift);
        if (a.res_mode == 1) t += skip;
        const int ti = sat32(t);
        if (a.out_mode == 3) {
            ((int32_t *)a.out)[oo + r] = ti;
        } else {
            int64_t q = rsr64((int64_t)ti * a.mul, a.shift);
            if (a.res_mode == 2) q += skip;
            ((uint8_t *)a.out)[oo + r] = (uint8_t)clampi64(q, a.lo, a.hi);
        }
    }
}

// One output: y = accumulator with the bias in it, resraw = its skip operand as loaded (any kind), oo = its element index
// in the output.  quick32 (wave-uniform; the caller checked a.out_mode != raw, a.rq_fast, and a.res_fast where there is a
// skip operand): the same arithmetic in 32 bits.
__device__ __forceinline__ void epilogue_one(const ConvArgs &a, int y, int resraw, size_t oo, bool quick32)
{
    if (quick32) {
        int skip = 0;
        if (a.res_mode != 0) skip = (int)(((uint32_t)resraw * (uint32_t)a.res_mul + (uint32_t)((1 << a.res_shift) >> 1)) >> a.res_shift);
        const int ti = a.res_mode == 1 ? __builtin_elementwise_add_sat(y, skip) : y;
        int q = (int)(((int64_t)ti * a.mul_hi + 0x80000000LL) >> 32);
        if (a.res_mode == 2) q = __builtin_elementwise_add_sat(q, skip);       // the clamp below makes the saturation exact
        ((uint8_t *)a.out)[oo] = (uint8_t)min(max(q, a.lo), a.hi);
        return;
    }
    int64_t t = y;
    int64_t skip = 0;
    if (a.res_mode != 0) skip = rsr64((int64_t)resraw * a.res_mul, a.res_shift);
    if (a.res_mode == 1) t += skip;
    const int ti = sat32(t);
    if (a.out_mode == 3) {
        ((int32_t *)a.out)[oo] = ti;
    } else {
        int64_t q = rsr64((int64_t)ti * a.mul, a.shift);
        if (a.res_mode == 2) q += skip;
        ((uint8_t *)a.out)[oo] = (uint8_t)clampi64(q, a.lo, a.hi);
    }
}

// min(max(x, lo), hi) as one instruction (the compiler only fuses the pair when it can prove lo <= hi);
// at most one of the three operands may live in a scalar register
__device__ __forceinline__ int med3_v0s(int x, int hi_s)
{
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi_s));
    return r;
}
__device__ __forceinline__ int med3_vvs(int x, int lo_v, int hi_s)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo_v), "s"(hi_s));
    return r;
}
// the low bytes of four values as one word (three byte-permutes)
__device__ __forceinline__ int pack_low_bytes(int v0, int v1, int v2, int v3)
{
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)v1, (uint32_t)v0, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)v3, (uint32_t)v2, 0x0c0c0400u);
    return (int)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// t clamped to [0, t_hi], times m, the high 32 bits of it: t_hi and m (scalars) below 2^24.  Plain arithmetic that the compiler turns
// into two clamps and v_mul_hi_u32_u24: around hand-written instructions it puts wait states.
__device__ __forceinline__ uint32_t clamp_mul_hi_u24(int t, int t_hi, int m)
{
    const uint32_t x = (uint32_t)min(max(t, 0), t_hi & 0xffffff);
    return (uint32_t)(((uint64_t)(x & 0xffffff) * (uint64_t)((uint32_t)m & 0xffffff)) >> 32);
}

// byte `pos` (1..3) of w = low byte of x >> sh; the other bytes of w are kept
__device__ __forceinline__ void shift_into_byte(int &w, uint32_t x, int sh_v, int pos)
{
    if (pos == 1)
        asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
            : "+v"(w) : "v"(sh_v), "v"(x));
    else if (pos == 2)
        asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
            : "+v"(w) : "v"(sh_v), "v"(x));
    else
        asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD"
            : "+v"(w) : "v"(sh_v), "v"(x));
}

// Sixteen values t (bias and skip operand already in) -> sixteen requantised, clamped bytes as four words
// (Section 3.2.1).  RQ as in epilogue_vec: 1 one 32x32->64 multiply-add whose high word is the result;
// 2 general 64-bit multiply, add, shift; 3 in 32 bits after clamping t to [0, t_hi] (see ConvArgs::rq24); 4 likewise with the
// high half of a 24-bit product (see ConvArgs::rqh).  (Form 4 in place of form 1 in every kernel measured slower, the nine-image
// network 341 -> 354 us; it serves kernels that deal an epilogue out between matrix instructions, where form 1's word pairs do not fit.)  5 bytes
// (requant_fits_byte), as in epilogue_hi_slice.
// (P: ConvArgs, or any struct with the same requantisation fields)
template <int RQ, class P>
__device__ __forceinline__ v4i requant16(const P &a, const int (&t)[16])
{
    if (RQ == 3) {
        // clamp, multiply-add, then the shift writes its byte of the output word: three instructions per value
        int w[4];
        const int sh_v = a.shift;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t tc = (uint32_t)med3_v0s(t[r], a.t_hi);
            const uint32_t x = __umul24(tc, (uint32_t)a.mul) + (uint32_t)a.rnd;
            if ((r & 3) == 0) w[r >> 2] = (int)(x >> a.shift);
            else shift_into_byte(w[r >> 2], x, sh_v, r & 3);
        }
        return v4i{w[0], w[1], w[2], w[3]};
    }
    if (RQ == 4) {
        int w[4];
        const int one_v = 1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t x = clamp_mul_hi_u24(t[r], a.t_hi, a.rqh) + 1u;
            if ((r & 3) == 0) w[r >> 2] = (int)(x >> 1);
            else shift_into_byte(w[r >> 2], x, one_v, r & 3);
        }
        return v4i{w[0], w[1], w[2], w[3]};
    }
    if (RQ == 5) {
        typedef short i16x2 __attribute__((ext_vector_type(2)));
        const int m = a.mul_hi << 8;
        uint32_t two[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2)
            two[r / 2] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, __builtin_amdgcn_cvt_pk_i16((int)(((int64_t)t[r] * m + 0x8000000000LL) >> 32),
                                                                                    (int)(((int64_t)t[r + 1] * m + 0x8000000000LL) >> 32))), i16x2{0, 0}));
        v4i w;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (int)__builtin_amdgcn_perm(two[2 * q + 1], two[2 * q], 0x07050301u);
        return w;
    }
    int v[16];
    const int lo_v = a.lo;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (RQ == 1) {
            // [t * mul / 2^shift] = high word of t * (mul << (32 - shift)) + 2^31   (1 <= shift <= 32)
            const int q = (int)(((int64_t)t[r] * a.mul_hi + 0x80000000LL) >> 32);
            v[r] = med3_vvs(q, lo_v, a.hi);
        } else {
            v[r] = clampi64(rsr64((int64_t)t[r] * a.mul, a.shift), a.lo, a.hi);
        }
    }
    return v4i{pack_low_bytes(v[0], v[1], v[2], v[3]), pack_low_bytes(v[4], v[5], v[6], v[7]),
               pack_low_bytes(v[8], v[9], v[10], v[11]), pack_low_bytes(v[12], v[13], v[14], v[15])};
}
// the cheapest exact form the layer's parameters allow (wave-uniform choice)
template <class P>
__device__ __forceinline__ v4i requant16_any(const P &a, const int (&t)[16])
{
    if (a.rq_byte) return requant16<5>(a, t);
    if (a.rq24) return requant16<3>(a, t);
    if (a.rq_fast) return requant16<1>(a, t);
    return requant16<2>(a, t);
}

// vector path: all 16 channels valid, 16-byte aligned skip operand and output.
// RES: 0 no skip operand; 1 unsigned 8-bit operand joined before requantisation with a rescale
//      that fits 32 bits; 2 anything else (signed or int32 operand, wide multiplier, join after).
// RQ:  0 raw int32 output; 1 requantisation as one 32x32->64 multiply-add whose high
//      word is the result; 2 general 64-bit multiply, add, shift; 3 in 32 bits after clamping
//      t to [0, t_hi] (see ConvArgs::rq24; never with RES 2).
template <int RES, int RQ>
__device__ __forceinline__ void epilogue_vec(const ConvArgs &a, const v16i &acc, int p, int co0, const v4i &res8)
{
    int t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = acc[r];
    int rv[16];
    if (RES != 0) {
        if (RES == 2 && a.res_dtype == 2) {
            const v4i *rp = (const v4i *)((const int32_t *)a.res + ((size_t)p * a.res_cs + co0));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i v = rp[q];
                rv[4 * q] = v.x; rv[4 * q + 1] = v.y; rv[4 * q + 2] = v.z; rv[4 * q + 3] = v.w;
            }
        } else {
            const int wd[4] = {res8.x, res8.y, res8.z, res8.w};
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int b8 = (int)(((uint32_t)wd[r >> 2] >> ((r & 3) * 8)) & 0xffu);
                rv[r] = RES == 2 && a.res_dtype == 1 ? (int)(int8_t)b8 : b8;
            }
        }
    }
    if (RES == 1) {
        const int half = (1 << a.res_shift) >> 1;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            // unsigned operand and 255 * res_mul + half < 2^31 (the host's gate), so res_mul < 2^24: an unsigned
            // 24-bit multiply (the signed one would read multipliers from 2^23 on as negative)
            t[r] = __builtin_elementwise_add_sat(t[r], (int)((__umul24((uint32_t)rv[r], (uint32_t)a.res_mul) + (uint32_t)half) >> a.res_shift));
    }
    if (RES == 2 && a.res_mode == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) t[r] = sat32((int64_t)t[r] + rsr64((int64_t)rv[r] * a.res_mul, a.res_shift));
    }
    const size_t oo = (size_t)p * a.out_cs + a.out_co + co0;
    if (RQ == 0) {
        v4i *op = (v4i *)((int32_t *)a.out + oo);
#pragma unroll
        for (int q = 0; q < 4; ++q) op[q] = v4i{t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]};
        return;
    }
    if (RQ == 3 || (RQ == 1 && RES != 2)) {
        *(v4i *)((uint8_t *)a.out + oo) = requant16<RQ>(a, t);
        return;
    }
    int v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        int64_t q = RQ == 1 ? (((int64_t)t[r] * a.mul_hi + 0x80000000LL) >> 32) : rsr64((int64_t)t[r] * a.mul, a.shift);
        if (RES == 2 && a.res_mode == 2) q += rsr64((int64_t)rv[r] * a.res_mul, a.res_shift);
        v[r] = clampi64(q, a.lo, a.hi);
    }
    *(v4i *)((uint8_t *)a.out + oo) = v4i{pack_low_bytes(v[0], v[1], v[2], v[3]), pack_low_bytes(v[4], v[5], v[6], v[7]),
                                          pack_low_bytes(v[8], v[9], v[10], v[11]), pack_low_bytes(v[12], v[13], v[14], v[15])};
}

// True when the call's skip operand is 8-bit and the vector epilogue handles it: then the operands of
// a wave's tiles can be fetched ahead of the K loop (prefetch_res8) and handed to epilogue_tiles.
__device__ __forceinline__ bool res8_applies(const ConvArgs &a)
{
    return a.epi_vec && !(a.Cout & 15) && a.res_mode != 0 && a.res_dtype != 2;
}

// ---- per-output-channel parameters (Section 3.4.3: one weight step per output channel leaves
// every channel its own ratio): channel c is requantised with (pc_mul[c], pc_shift[c]) and its
// skip operand rescaled with (pc_res_mul[c], pc_res_shift[c]).
// General form for one pixel's 16 channels (nv of them valid): any parameters, any alignment, any
// tail; 64-bit arithmetic, four channels at a time.  g: the group's packed parameters.
__device__ __forceinline__ void epilogue_pc_slow(const ConvArgs &a, const v16i &acc, int p, int co0, int nv,
                                                 const int32_t *g)
{
    const bool vec = a.epi_vec && nv == 16;
    const size_t ro = (size_t)p * a.res_cs + co0;
    const size_t oo = (size_t)p * a.out_cs + a.out_co + co0;
    const bool requant = a.out_mode != 3;
    uint32_t wd[4] = {0, 0, 0, 0};
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        const v4i mu = *(const v4i *)(g + kPcMul + 4 * q4), sf = *(const v4i *)(g + kPcShift + 4 * q4);
        const v4i rmu = *(const v4i *)(g + kPcResMul + 4 * q4), rsf = *(const v4i *)(g + kPcResShift + 4 * q4);
        int rv[4] = {0, 0, 0, 0};
        if (a.res_mode != 0) {
            if (vec && a.res_dtype == 2) {
                const v4i v = *(const v4i *)((const int32_t *)a.res + ro + 4 * q4);
                rv[0] = v.x; rv[1] = v.y; rv[2] = v.z; rv[3] = v.w;
            } else if (vec) {
                const int w4 = *(const int *)((const uint8_t *)a.res + ro + 4 * q4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int b8 = (w4 >> (8 * e)) & 0xff;
                    rv[e] = a.res_dtype == 1 ? (int)(int8_t)b8 : b8;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * q4 + e < nv) rv[e] = load_elem(a.res, ro + 4 * q4 + e, a.res_dtype);
            }
        }
        int ti[4];
        int qv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int64_t t = acc[4 * q4 + e];
            const int64_t skip = a.res_mode != 0 ? rsr64((int64_t)rv[e] * rmu[e], rsf[e] & 63) : 0;
            if (a.res_mode == 1) t += skip;
            ti[e] = sat32(t);
            int64_t q = rsr64((int64_t)ti[e] * mu[e], sf[e] & 63);
            if (a.res_mode == 2) q += skip;
            qv[e] = clampi64(q, a.lo, a.hi);
            wd[q4] |= (uint32_t)(qv[e] & 0xff) << (8 * e);
        }
        if (!requant) {
            if (vec) {
                *(v4i *)((int32_t *)a.out + oo + 4 * q4) = v4i{ti[0], ti[1], ti[2], ti[3]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * q4 + e < nv) ((int32_t *)a.out)[oo + 4 * q4 + e] = ti[e];
            }
        } else if (!vec) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * q4 + e < nv) ((uint8_t *)a.out)[oo + 4 * q4 + e] = (uint8_t)qv[e];
        }
    }
    if (requant && vec) *(v4i *)((uint8_t *)a.out + oo) = v4i{(int)wd[0], (int)wd[1], (int)wd[2], (int)wd[3]};
}

// One row of a wave's tiles (16 channels per lane, TP pixels) in the single-multiply form of
// pc_prepack_kernel.  skip: an 8-bit skip operand joins before requantisation and its rescale fits 32
// bits.  plain: no channel of the wave's groups needs the clamp, the pre-shift or the post-shift.  Both
// are wave-uniform.  Parameters are fetched four channels at a time and used for all TP pixels before
// the next four (registers are scarce here); the arithmetic variants branch inside that loop.
template <int TP>
__device__ __forceinline__ void epilogue_pc_row(const ConvArgs &a, const v16i (&acc)[TP], int co0, int pix_wave, int lane,
                                                const int32_t *g, const v4i (&rw)[TP], bool skip, bool plain)
{
    uint32_t wd[TP][4];
    const int lo_v = a.lo;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        const v4i A = *(const v4i *)(g + kPcA + 4 * q4);
        v4i L = {0, 0, 0, 0}, T = {0, 0, 0, 0}, C = {0, 0, 0, 0}, rmu = {1, 1, 1, 1}, rsf = {0, 0, 0, 0};
        if (!plain) {
            L = *(const v4i *)(g + kPcL + 4 * q4);
            T = *(const v4i *)(g + kPcT + 4 * q4);
            C = *(const v4i *)(g + kPcC + 4 * q4);
        }
        if (skip) { rmu = *(const v4i *)(g + kPcResMul + 4 * q4); rsf = *(const v4i *)(g + kPcResShift + 4 * q4); }
        auto body = [&](auto res_tag, auto plain_tag) {
            constexpr bool RES = decltype(res_tag)::value;
            constexpr bool PLAIN = decltype(plain_tag)::value;
#pragma unroll
            for (int j = 0; j < TP; ++j) {
                const uint32_t w4 = (uint32_t)rw[j][q4];
                int v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int t = acc[j][4 * q4 + e];
                    if (RES) {
                        // unsigned operands only (a.pc_fast_ok) and 255 * rmu + half < 2^31 (group flag bit 0): an
                        // unsigned 24-bit multiply whose sum stays below 2^31
                        const uint32_t rv = (w4 >> (8 * e)) & 0xffu;
                        t = __builtin_elementwise_add_sat(t, (int)((__umul24(rv, (uint32_t)rmu[e]) + ((1u << rsf[e]) >> 1)) >> rsf[e]));
                    }
                    int q;
                    if (PLAIN) {
                        q = (int)(((int64_t)t * A[e] + 0x80000000LL) >> 32);
                    } else {
                        const int tc = min(max(t, ~T[e]), T[e]) << L[e];
                        q = (int)(((int64_t)tc * A[e] + ((int64_t)1 << (31 + C[e]))) >> 32) >> C[e];
                    }
                    v[e] = med3_vvs(q, lo_v, a.hi);
                }
                wd[j][q4] = (uint32_t)pack_low_bytes(v[0], v[1], v[2], v[3]);
            }
        };
        if (skip) {
            if (plain) body(std::true_type{}, std::true_type{});
            else body(std::true_type{}, std::false_type{});
        } else {
            if (plain) body(std::false_type{}, std::true_type{});
            else body(std::false_type{}, std::false_type{});
        }
        __builtin_amdgcn_sched_barrier(0);     // keep the four parameter fetches apart
    }
#pragma unroll
    for (int j = 0; j < TP; ++j) {
        const int p = pix_wave + j * 32 + (lane & 31);
        if (p < a.M)
            *(v4i *)((uint8_t *)a.out + ((size_t)p * a.out_cs + a.out_co + co0)) =
                v4i{(int)wd[j][0], (int)wd[j][1], (int)wd[j][2], (int)wd[j][3]};
    }
}

// Epilogue of a wave's tiles with per-channel parameters.  The single-multiply form is used when the
// call allows it (8-bit output, 16-byte accesses, no skip operand or an 8-bit one joined before
// requantisation: a.pc_fast_ok), the lane's 16 channels are all valid and the skip rescale of its group
// fits 32 bits; the decision is taken for the whole wave, so each form is straight-line code.
// res8: the 8-bit skip operands fetched by prefetch_res8 for the same tile when res8_applies(a).
// groups: packed parameters of the channel group that starts at channel co_base (a multiple of 16),
// followed by those of the next groups (global memory or a copy in LDS).
template <int TM, int TP>
__device__ __forceinline__ void epilogue_pc_tiles(const ConvArgs &a, const v16i (&acc)[TM][TP], int co_wave, int pix_wave,
                                                  int lane, const v4i (&res8)[TM][TP], const int32_t *groups, int co_base)
{
    const bool skip = a.res_mode != 0;
    const bool have_res8 = res8_applies(a);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int co0 = co_wave + i * 32 + (lane >> 5) * 16;
        const int nv = min(16, a.Cout - co0);          // <= 0: this half of the wave has no channels here
        const int32_t *g = groups + ((co0 - co_base) >> 4) * kPcGroupInts;
        const int flags = nv > 0 ? g[kPcFlags] : 3;
        const bool fast = nv <= 0 || (a.pc_fast_ok && nv == 16 && (!skip || (flags & 1)));
        const bool wave_fast = __builtin_amdgcn_ballot_w64(!fast) == 0;
        const bool wave_plain = __builtin_amdgcn_ballot_w64(!(flags & 2)) == 0;
        if (!wave_fast) {
#pragma unroll
            for (int j = 0; j < TP; ++j) {
                const int p = pix_wave + j * 32 + (lane & 31);
                if (nv > 0 && p < a.M) epilogue_pc_slow(a, acc[i][j], p, co0, nv, g);
            }
            continue;
        }
        if (nv <= 0) continue;
        v4i rw[TP];
#pragma unroll
        for (int j = 0; j < TP; ++j) {
            const int p = pix_wave + j * 32 + (lane & 31);
            rw[j] = have_res8 ? res8[i][j] : v4i{0, 0, 0, 0};
            if (skip && !have_res8 && p < a.M) rw[j] = *(const v4i *)((const uint8_t *)a.res + ((size_t)p * a.res_cs + co0));
        }
        epilogue_pc_row<TP>(a, acc[i], co0, pix_wave, lane, g, rw, skip, wave_plain);
    }
}
template <int TM, int TP>
__device__ __forceinline__ void prefetch_res8(const ConvArgs &a, int co_wave, int pix_wave, int lane, v4i (&res8)[TM][TP])
{
    if (!res8_applies(a)) return;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int co0 = co_wave + i * 32 + (lane >> 5) * 16;
#pragma unroll
        for (int j = 0; j < TP; ++j) {
            const int p = pix_wave + j * 32 + (lane & 31);
            if (co0 < a.Cout && p < a.M)
                res8[i][j] = *(const v4i *)((const uint8_t *)a.res + ((size_t)p * a.res_cs + co0));
        }
    }
}
// res8: the 8-bit skip operands fetched by prefetch_res8 for the same tile (ignored otherwise)
template <int TM, int TP>
__device__ __forceinline__ void epilogue_tiles(const ConvArgs &a, const v16i (&acc)[TM][TP], int co_wave, int pix_wave,
                                               int lane, const v4i (&res8)[TM][TP])
{
    const int half = lane >> 5;
    auto for_tiles = [&](auto fn) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int co0 = co_wave + i * 32 + half * 16;
#pragma unroll
            for (int j = 0; j < TP; ++j) {
                const int p = pix_wave + j * 32 + (lane & 31);
                if (co0 < a.Cout && p < a.M) fn(acc[i][j], p, co0, i, j);
            }
        }
    };
    // Unaligned tensors take the element-wise path for the whole call, and so do channel tails (cout % 16 != 0)
    // together with a skip operand (prefetch_res8 does not serve them); otherwise only the last, partial group
    // of 16 channels does.
    const bool all_slow = !a.epi_vec || ((a.Cout & 15) && a.res_mode != 0);
    if (!all_slow) {
        switch (a.epi_mode) {
#define ICNN_EPI_CASE(RES, RQ)                                                                      \
    case RES * 4 + RQ:                                                                              \
        for_tiles([&](const v16i &c, int p, int co0, int i, int j) {                                \
            if (co0 + 16 <= a.Cout) epilogue_vec<RES, RQ>(a, c, p, co0, res8[i][j]);                \
        });                                                                                         \
        break;
            ICNN_EPI_CASE(0, 0) ICNN_EPI_CASE(0, 1) ICNN_EPI_CASE(0, 2) ICNN_EPI_CASE(0, 3)
            ICNN_EPI_CASE(1, 0) ICNN_EPI_CASE(1, 1) ICNN_EPI_CASE(1, 2) ICNN_EPI_CASE(1, 3)
            ICNN_EPI_CASE(2, 0) ICNN_EPI_CASE(2, 1) ICNN_EPI_CASE(2, 2)
#undef ICNN_EPI_CASE
        default: break;
        }
    }
    if (all_slow || (a.Cout & 15)) {
        for_tiles([&](const v16i &c, int p, int co0, int, int) {
            if (all_slow || co0 + 16 > a.Cout) epilogue_slow(a, c, p, co0, min(16, a.Cout - co0));
        });
    }
}
// One pixel's 16 channels co0..co0+15 (all valid; the call allows 16-byte accesses: a.epi_vec) in the form the
// host chose (a.epi_mode).  res8: the 8-bit skip operand's 16 bytes, when there is one.
__device__ __forceinline__ void epilogue_px16(const ConvArgs &a, const v16i &acc, int p, int co0, const v4i &res8)
{
    switch (a.epi_mode) {
#define ICNN_EPI_CASE(RES, RQ) case RES * 4 + RQ: epilogue_vec<RES, RQ>(a, acc, p, co0, res8); break;
        ICNN_EPI_CASE(0, 0) ICNN_EPI_CASE(0, 1) ICNN_EPI_CASE(0, 2) ICNN_EPI_CASE(0, 3)
        ICNN_EPI_CASE(1, 0) ICNN_EPI_CASE(1, 1) ICNN_EPI_CASE(1, 2) ICNN_EPI_CASE(1, 3)
        ICNN_EPI_CASE(2, 0) ICNN_EPI_CASE(2, 1) ICNN_EPI_CASE(2, 2)
#undef ICNN_EPI_CASE
    default: break;
    }
}
// The same arithmetic as epilogue_px16 for a layer that stores unsigned bytes and whose skip operand, if any, is
// the unsigned 8-bit kind joined before requantisation (RES 0 or 1, RQ 1, 2 or 3): the sixteen bytes are returned,
// for callers that keep the result on chip as well.
// RQ: 0 the requantisation form is chosen at run time (wave-uniform branch); 1, 2, 3 that form of requant16, for
// callers that need the epilogue to be straight-line code.
template <int RES, int RQ = 0>
__device__ __forceinline__ v4i epilogue_bytes16(const ConvArgs &a, const v16i &acc, const v4i &res8)
{
    int t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = acc[r];
    if (RES == 1) {
        const int wd[4] = {res8.x, res8.y, res8.z, res8.w};
        const int half = (1 << a.res_shift) >> 1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t b8 = ((uint32_t)wd[r >> 2] >> ((r & 3) * 8)) & 0xffu;
            t[r] = __builtin_elementwise_add_sat(t[r], (int)((__umul24(b8, (uint32_t)a.res_mul) + (uint32_t)half) >> a.res_shift));
        }
    }
    if constexpr (RQ == 0) return requant16_any(a, t);
    else return requant16<RQ>(a, t);
}
// epilogue_bytes16 with per-channel parameters (g: those of the lane's group of 16, see kPcGroupInts; in LDS, the lanes of a half read the same
// ones): unsigned bytes, skip operand as there.  The forms are those of epilogue_pc_row and, where a skip rescale does not fit 32 bits,
// of epilogue_pc_slow; which one is decided for the whole wave.
template <int RES>
__device__ __forceinline__ v4i epilogue_pc_bytes16(const ConvArgs &a, const v16i &acc, const v4i &res8, const int32_t *g)
{
    const int flags = g[kPcFlags];
    const bool plain = __builtin_amdgcn_ballot_w64(!(flags & 2)) == 0;
    const bool res32 = RES == 0 || __builtin_amdgcn_ballot_w64(!(flags & 1)) == 0;
    const int lo_v = a.lo;
    v4i w;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        int t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = acc[4 * q4 + e];
        if (RES == 1) {
            const v4i rmu = *(const v4i *)(g + kPcResMul + 4 * q4), rsf = *(const v4i *)(g + kPcResShift + 4 * q4);
            const uint32_t w4 = (uint32_t)res8[q4];
            if (res32) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    t[e] = __builtin_elementwise_add_sat(t[e], (int)((__umul24((w4 >> (8 * e)) & 0xffu, (uint32_t)rmu[e]) + ((1u << rsf[e]) >> 1)) >> rsf[e]));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = sat32((int64_t)t[e] + rsr64((int64_t)((w4 >> (8 * e)) & 0xffu) * rmu[e], rsf[e] & 63));
            }
        }
        const v4i A = *(const v4i *)(g + kPcA + 4 * q4);
        int v[4];
        if (plain) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = med3_vvs((int)(((int64_t)t[e] * A[e] + 0x80000000LL) >> 32), lo_v, a.hi);
        } else {
            const v4i L = *(const v4i *)(g + kPcL + 4 * q4), T = *(const v4i *)(g + kPcT + 4 * q4), C = *(const v4i *)(g + kPcC + 4 * q4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tc = min(max(t[e], ~T[e]), T[e]) << L[e];
                v[e] = med3_vvs((int)(((int64_t)tc * A[e] + ((int64_t)1 << (31 + C[e]))) >> 32) >> C[e], lo_v, a.hi);
            }
        }
        w[q4] = pack_low_bytes(v[0], v[1], v[2], v[3]);
    }
    return w;
}
// The parameters of n_groups groups from memory to LDS (16-byte pieces, dealt over the workgroup's threads)
template <int THREADS>
__device__ __forceinline__ void copy_pc_groups(int32_t *dst, const int32_t *src, int n_groups, int tid)
{
    for (int i = tid; i < n_groups * (kPcGroupInts / 4); i += THREADS) ((v4i *)dst)[i] = ((const v4i *)src)[i];
}
// Sixteen outputs of a layer with rq_fast that joins an int32 skip operand before requantisation, where skip_s32_fits below holds: 32 bits of
// (r * res_mul + half + t * 2^shift) >> shift are the rescaled operand r and the sum t together, two multiply-adds, and an overflow is kept at
// int32's ends by its high word alone: what is left below that is too little to leave the output's range.  Six and three quarter
// instructions per output, some 25 in the general form.
__device__ __forceinline__ v4i epilogue_skip_s32(const ConvArgs &a, const v16i &acc, const v4i (&res)[4])
{
    int t[16];
    const int sh = a.res_shift, ends = 1 << (sh - 1);
    const int lowest = -ends;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t sum = (int64_t)acc[r] * (1 << sh) + ((int64_t)res[r >> 2][r & 3] * a.res_mul + ends);
        const int high = med3_vvs((int)(sum >> 32), lowest, ends - 1);
        t[r] = (int)__builtin_amdgcn_alignbit((uint32_t)high, (uint32_t)sum, (uint32_t)sh);
    }
    return requant16<1>(a, t);
}
static inline bool skip_s32_fits(const ConvArgs &a)
{
    if (a.res_mode != 1 || a.res_dtype != 2 || !a.rq_fast || !a.epi_vec || a.res_shift < 2 || a.res_shift > 30) return false;
    const long long left = 1LL << (32 - a.res_shift);        // an overflow ends up to this much (less one) inside int32's ends
    auto out = [&](long long v) { return (v * a.mul_hi + 0x80000000LL) >> 32; };
    return out(0x7fffffffLL + 1 - left) >= a.hi && out(-0x80000000LL + left - 1) <= a.lo;
}
// Outputs R0 .. R0 + N - 1 of epilogue_bytes16<RES, 3> (the 32-bit requantisation form, a.rq24): their bytes go into
// the words w[R0 / 4 ..], which the caller collects over the sixteen outputs.  For callers that deal the epilogue out
// in slices between matrix instructions.  R0 and N are multiples of... any; a word is started by its output 4 q.
// FORM: 3 (a.rq24) or 4 (a.rqh), as in requant16.
template <int RES, int R0, int N, int FORM = 3, class P>
__device__ __forceinline__ void epilogue_rq24_slice(const P &a, const v16i &acc, const v4i &res8, int (&w)[4])
{
    const int wd[4] = {res8.x, res8.y, res8.z, res8.w};
    const int sh_v = a.shift;
#pragma unroll
    for (int r = R0; r < R0 + N; ++r) {
        int t = acc[r];
        if constexpr (RES == 1) {
            const int half = (1 << a.res_shift) >> 1;
            const uint32_t b8 = ((uint32_t)wd[r >> 2] >> ((r & 3) * 8)) & 0xffu;
            t = __builtin_elementwise_add_sat(t, (int)((__umul24(b8, (uint32_t)a.res_mul) + (uint32_t)half) >> a.res_shift));
        }
        const uint32_t x = FORM == 4 ? clamp_mul_hi_u24(t, a.t_hi, a.rqh) + 1u : __umul24((uint32_t)med3_v0s(t, a.t_hi), (uint32_t)a.mul) + (uint32_t)a.rnd;
        if ((r & 3) == 0) w[r >> 2] = (int)(x >> (FORM == 4 ? 1 : a.shift));
        else shift_into_byte(w[r >> 2], x, FORM == 4 ? 1 : sh_v, r & 3);
    }
}
// Outputs R0 .. R0 + N - 1 (N even) of epilogue_bytes16<RES, 1>: a layer with a.rq_fast whose skip operand's rescale, if any, is sk.  Five and
// three quarter instructions per output, two and three quarters without the operand (the 32-bit form takes seven and three): every one of
// them issues in the same four to five clocks on this chip, wide multiplies included (v_mad_i64_i32 4.6, v_mul_hi_u32 4.8, v_mad_u32_u24
// 4.8 with two waves per SIMD and matrix instructions between them), so a product whose high word is the result wants no shift behind it.
// Step by step for the N values together, so that none waits for the instruction just before it.
// w: the words of the sixteen bytes, which the caller collects over its slices; a word's lower half is kept in it until the upper one comes.
// BYTE (requant_fits_byte): bytes from 0 to 127 by a multiplier below 2^23.  The product is taken 2^8 times as large, so that the saturating conversion to 16 bits is
// the upper clamp, one packed maximum the lower one of two outputs, and the result the upper byte: two and a quarter instructions in place of
// two and three quarters.
template <int RES, int R0, int N, bool BYTE = false, class P>
__device__ __forceinline__ void epilogue_hi_slice(const P &a, const SkipMul &sk, const v16i &acc, const v4i &res8, int (&w)[4])
{
    static_assert(N % 2 == 0 && R0 % 2 == 0, "whole pairs");
    int t[N];
    [[maybe_unused]] const int lo_v = a.lo;
    if constexpr (RES == 1) {
        uint32_t x[N];
        // byte in the top bits, the rounding constant below it
#pragma unroll
        for (int e = 0; e < N; ++e)
            x[e] = __builtin_amdgcn_perm((uint32_t)res8[(R0 + e) >> 2], sk.rnd, 0x00020100u | (uint32_t)(4 + ((R0 + e) & 3)) << 24);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < N; ++e) x[e] = __umulhi(x[e], sk.k);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < N; ++e) t[e] = __builtin_elementwise_add_sat(acc[R0 + e], (int)x[e]);
        __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) t[e] = acc[R0 + e];
    }
    if constexpr (BYTE) {
        typedef short i16x2 __attribute__((ext_vector_type(2)));
        const int m = a.mul_hi << 8;
#pragma unroll
        for (int e = 0; e < N; ++e) t[e] = (int)(((int64_t)t[e] * m + 0x8000000000LL) >> 32);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t two[N / 2];
#pragma unroll
        for (int e = 0; e < N; e += 2) two[e / 2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_i16(t[e], t[e + 1]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < N; e += 2) two[e / 2] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, two[e / 2]), i16x2{0, 0}));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < N; e += 2) {
            if (((R0 + e) & 2) == 0) w[(R0 + e) >> 2] = (int)two[e / 2];
            else w[(R0 + e) >> 2] = (int)__builtin_amdgcn_perm(two[e / 2], (uint32_t)w[(R0 + e) >> 2], 0x07050301u);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = (int)(((int64_t)t[e] * a.mul_hi + 0x80000000LL) >> 32);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = med3_vvs(t[e], lo_v, a.hi);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < N; e += 2) {
        const uint32_t two = __builtin_amdgcn_perm((uint32_t)t[e + 1], (uint32_t)t[e], 0x0c0c0400u);
        if (((R0 + e) & 2) == 0) w[(R0 + e) >> 2] = (int)two;
        else w[(R0 + e) >> 2] = (int)__builtin_amdgcn_perm(two, (uint32_t)w[(R0 + e) >> 2], 0x05040100u);
    }
}
template <int RES, bool BYTE = false, class P>
__device__ __forceinline__ v4i epilogue_hi16(const P &a, const SkipMul &sk, const v16i &acc, const v4i &res8)
{
    int w[4];
    epilogue_hi_slice<RES, 0, 8, BYTE>(a, sk, acc, res8, w);
    __builtin_amdgcn_sched_barrier(0);
    epilogue_hi_slice<RES, 8, 8, BYTE>(a, sk, acc, res8, w);
    return v4i{w[0], w[1], w[2], w[3]};
}
// The same per output channel, from tables of a factor (pc_prepack_kernel's A) and of the skip rescale's multiplier and byte position (pc_hi_channel):
// five and three quarter instructions per output, two and three quarters without the operand.  A, K: those of outputs R0, R0 + 1; P: the positions
// of the four outputs that R0 is among, a byte each.
typedef int v2i __attribute__((ext_vector_type(2)));
template <int RES, int R0>
__device__ __forceinline__ void epilogue_pc_hi_pair(const ConvArgs &a, v2i A, v2i K, uint32_t P, const v16i &acc, const v4i &res8, int (&w)[4])
{
    int t[2];
    const int lo_v = a.lo;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        t[e] = acc[R0 + e];
        if constexpr (RES == 1) {
            // [x * mul / 2^shift] = high 32 bits of (x << (32 - shift)) * mul + 2^31
            const int byte = 8 * ((R0 + e) & 3);
            const uint32_t x = (((uint32_t)res8[(R0 + e) >> 2] >> byte) & 0xffu) << ((P >> byte) & 0xffu);
            t[e] = __builtin_elementwise_add_sat(t[e], (int)(((uint64_t)x * (uint32_t)K[e] + 0x80000000ull) >> 32));
        }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) t[e] = med3_vvs((int)(((int64_t)t[e] * A[e] + 0x80000000LL) >> 32), lo_v, a.hi);
    const uint32_t two = __builtin_amdgcn_perm((uint32_t)t[1], (uint32_t)t[0], 0x0c0c0400u);
    if constexpr ((R0 & 2) == 0) w[R0 >> 2] = (int)two;
    else w[R0 >> 2] = (int)__builtin_amdgcn_perm(two, (uint32_t)w[R0 >> 2], 0x05040100u);
}
// sixteen of them, tables in LDS
template <int RES>
__device__ __forceinline__ v4i epilogue_pc_hi16(const ConvArgs &a, const int32_t *A, const int32_t *K, const uint8_t *P, const v16i &acc, const v4i &res8)
{
    int w[4];
    static_for<8>([&](auto h_tag) __attribute__((always_inline)) {
        constexpr int R0 = 2 * decltype(h_tag)::value;
        epilogue_pc_hi_pair<RES, R0>(a, *(const v2i *)(A + R0), RES ? *(const v2i *)(K + R0) : v2i{0, 0}, RES ? *(const uint32_t *)(P + (R0 & ~3)) : 0u, acc, res8, w);
    });
    return v4i{w[0], w[1], w[2], w[3]};
}
// A channel's table entries from the packed parameters; returns whether that form is exact for it (the factor needs no shift or clamp around
// it, the rescale of an unsigned byte stays in int32).  skip: the layer has such an operand.
__device__ __forceinline__ bool pc_hi_channel(const int32_t *pc, int channel, bool skip, int &A, int &K, int &P)
{
    const int32_t *const g = pc + (channel >> 4) * kPcGroupInts;
    const int r = channel & 15, flags = g[kPcFlags], rm = g[kPcResMul + r], rs = g[kPcResShift + r];
    A = g[kPcA + r];
    // (flag bit 0: shifts of 0 to 30, 255 * rm below 2^31; with a shift below 8 the byte goes to the top and the multiplier up by the rest)
    P = 32 - max(rs & 31, 8);
    K = skip ? rm << max(8 - (rs & 31), 0) : 0;
    return (flags & 2) && (!skip || (flags & 1));
}
// Between the last v_mfma of an accumulation and the first instruction that reads the accumulator.  The compiler's
// hazard recogniser does not always keep the two apart (seen in a kernel whose epilogue starts two instructions after
// the last MFMA, behind a branch: the reads returned the sums without the last product, now and then), and the
// hardware does not hold the reader back.  Twenty wait states, more than the compiler itself takes where it sees the reader (twelve behind the 32x32x32
// product of eight passes, eight behind the 16x16x64 one of four); the empty
// statements before and after tie every accumulator tile to the wait, so neither an MFMA nor a reader can cross it.
#ifdef ICNN_NO_DRAIN            // measurement only: what the wait states and the register pinning cost
#define ICNN_DRAIN_NOPS ""
#else
#define ICNN_DRAIN_NOPS "s_nop 15\n\ts_nop 3"
#endif
__device__ __forceinline__ void mfma_drain(v16i &acc)
{
    asm volatile(ICNN_DRAIN_NOPS : "+v"(acc));
}
template <int N>
__device__ __forceinline__ void mfma_drain(v16i (&acc)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(acc[i]));
    asm volatile(ICNN_DRAIN_NOPS);
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(acc[i]));
}
template <int M, int N>
__device__ __forceinline__ void mfma_drain(v16i (&acc)[M][N])
{
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("" : "+v"(acc[i][j]));
    asm volatile(ICNN_DRAIN_NOPS);
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("" : "+v"(acc[i][j]));
}

// fn(integral_constant<int, 0>) ... fn(integral_constant<int, N - 1>): a loop the compiler cannot leave rolled
// (register arrays indexed inside it stay in registers)
template <int N, class F>
__device__ __forceinline__ void static_for(F &&fn)
{
    if constexpr (N > 0) {
        static_for<N - 1>(fn);
        fn(std::integral_constant<int, N - 1>{});
    }
}

// sixteen consecutive int32 of the bias table in LDS
__device__ __forceinline__ v16i bias16(const int32_t *tab)
{
    const v4i *bp = (const v4i *)tab;
    v16i b;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4i v = bp[q];
        b[4 * q] = v.x; b[4 * q + 1] = v.y; b[4 * q + 2] = v.z; b[4 * q + 3] = v.w;
    }
    return b;
}

// for callers without a K loop to hide the fetch behind: fetch, then finish
template <int TM, int TP>
__device__ __forceinline__ void epilogue_tiles(const ConvArgs &a, const v16i (&acc)[TM][TP], int co_wave, int pix_wave,
                                               int lane)
{
    v4i res8[TM][TP];
    prefetch_res8<TM, TP>(a, co_wave, pix_wave, lane, res8);
    epilogue_tiles<TM, TP>(a, acc, co_wave, pix_wave, lane, res8);
}

// Scalars that have to be in registers here.  The compiler asks for a kernel argument where it is first used, one round of scalar loads after
// the other, some 1000 clocks for the first and 200 to 500 for each of the others (six of them before the last request of conv_lat.hip was out).
__device__ __forceinline__ void in_registers() {}
template <class T, class... R>
__device__ __forceinline__ void in_registers(T v, R... rest)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::"s"(v));
#endif
    in_registers(rest...);
}

// A kernel's argument that is read here and not where the compiler would have it, which is at the kernel's start: there it holds registers through phases
// that do not use it, and where they run out it is waited for at once to be put aside.  at: its place among the kernel's arguments (their
// order in a struct of the same members, which the kernel's file checks with parameters_of).
template <class T>
__device__ __forceinline__ T late_argument(unsigned at)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using Args = const __attribute__((address_space(4))) char *;
    Args p = (Args)__builtin_amdgcn_kernarg_segment_ptr() + at;
    asm volatile("" : "+s"(p));
    return *(const T *)p;
#else
    (void)at;
    return T{};
#endif
}
template <class... T>
struct Types {};
template <class... T>
Types<T...> parameters_of(void (*)(T...));

// fast_div with its parts as they come in scalar arguments
__device__ __forceinline__ int fast_div_packed(int n, unsigned mul, unsigned s1, unsigned s2)
{
    const unsigned t = __umulhi((unsigned)n, mul);
    return (int)((t + (((unsigned)n - t) >> s1)) >> s2);
}

// Maps the hardware workgroup id to a tile.  Workgroups are dealt round-robin to the
// 8 XCDs (each with its own L2); giving XCD x the contiguous tile range
// [x*per_xcd, (x+1)*per_xcd) keeps the cout tiles of one pixel tile, and neighbouring
// pixel tiles (shared halo rows), in one L2.  Returns false for padding workgroups.
__device__ __forceinline__ bool tile_of_block(const ConvArgs &a, int &ct, int &pt)
{
    const int xcd = blockIdx.x & 7;
    const int idx = blockIdx.x >> 3;
    const int logical = xcd * a.per_xcd + idx;
    if (logical >= a.n_tiles) return false;
    ct = logical % a.n_ct;
    pt = logical / a.n_ct;
    return true;
}

// Bias of the channels a lane owns: register r of a lane in half h of tile row i holds
// channel co_base + 32*i + 16*h + r.  Accumulators start at these values.
template <int TM>
__device__ __forceinline__ void load_bias_rows(const ConvArgs &a, int co_base, int half, v16i (&b)[TM])
{
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int co0 = co_base + i * 32 + half * 16;
        if (a.vec_bias) {
            const v4i *bp = (const v4i *)(a.bias + max(0, min(co0, a.Cout - 16)));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i v = bp[q];
                b[i][4 * q] = v.x; b[i][4 * q + 1] = v.y; b[i][4 * q + 2] = v.z; b[i][4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) b[i][r] = a.bias[min(co0 + r, a.Cout - 1)];
        }
        if (a.frag_xor) {
            // unsigned inputs up to 255: the matrix cores see x - 128, so 128 * (sum of the channel's
            // weights) is due (wsum is padded to whole 32-channel chunks and 16-byte aligned)
            const v4i *wp = (const v4i *)(a.wsum + co0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i v = wp[q];
                b[i][4 * q] += 128 * v.x; b[i][4 * q + 1] += 128 * v.y; b[i][4 * q + 2] += 128 * v.z; b[i][4 * q + 3] += 128 * v.w;
            }
        }
    }
}

template <int TM, int TP>
__device__ __forceinline__ void init_acc_with_bias(const ConvArgs &a, int co_base, int half, v16i (&acc)[TM][TP])
{
    v16i b[TM];
    load_bias_rows<TM>(a, co_base, half, b);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j) acc[i][j] = b[i];
}

#define ICNN_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | 0x0F70 | (((n) >> 4) << 14))

// Waits until at most `later` stages' worth of this wave's copies (LPS each) are still in
// flight; the count is an immediate of s_waitcnt (6 bits), hence the switch.
template <int LPS>
__device__ __forceinline__ void wait_stages_in_flight(int later)
{
    constexpr int kMax = 63 / LPS < 7 ? 63 / LPS : 7;
    if (later > kMax) later = kMax;
    switch (later) {
    case 0: ICNN_WAIT_VMCNT(0); break;
    case 1: ICNN_WAIT_VMCNT(LPS); break;
    case 2: ICNN_WAIT_VMCNT(2 * LPS <= 63 ? 2 * LPS : 63); break;
    case 3: ICNN_WAIT_VMCNT(3 * LPS <= 63 ? 3 * LPS : 63); break;
    case 4: ICNN_WAIT_VMCNT(4 * LPS <= 63 ? 4 * LPS : 63); break;
    case 5: ICNN_WAIT_VMCNT(5 * LPS <= 63 ? 5 * LPS : 63); break;
    case 6: ICNN_WAIT_VMCNT(6 * LPS <= 63 ? 6 * LPS : 63); break;
    default: ICNN_WAIT_VMCNT(7 * LPS <= 63 ? 7 * LPS : 63); break;
    }
}

// floor(n / d) for 0 <= n < 2^31 by multiply-high and shifts (Granlund & Montgomery's
// round-up method); the host fills `FastDiv` for d.
__device__ __forceinline__ int fast_div(int n, const FastDiv &d)
{
    const unsigned t = __umulhi((unsigned)n, d.mul);
    return (int)((t + (((unsigned)n - t) >> d.s1)) >> d.s2);
}

static inline bool finish_args(ConvArgs &a, int BM, int BP)
{
    a.n_ct = (a.Cout + BM - 1) / BM;
    const long long tiles = (long long)a.n_ct * ((a.M + BP - 1) / BP);
    if (tiles <= 0 || tiles > 0x7ffffff0LL) return false;
    a.n_tiles = (int)tiles;
    a.per_xcd = (int)((tiles + 7) / 8);
    return true;
}

static inline FastDiv make_fast_div(unsigned d)
{
    // l = ceil(log2 d); mul = floor(2^32 * (2^l - d) / d) + 1; q = (t + ((n - t) >> min(l,1))) >> max(l-1,0)
    FastDiv f;
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    f.mul = (unsigned)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 1 ? l - 1 : 0;
    return f;
}


}  // namespace icnn
