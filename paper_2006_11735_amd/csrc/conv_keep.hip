// 3x3 / stride 1 / padding 1 layers of 64 -> 64 channels on many pixels (the basic blocks of a residual network's first stage), with all the
// layer's weights in the registers of every wave for the workgroup's life.
//
//   work     the flattened N*H*W axis in rounds of 128 consecutive pixels, dealt out evenly: a workgroup takes a run of 6 or 7 of them
//            (64 pictures of 56 x 56) in tiles of at most eight; each of its four waves takes 32 pixels of a round, all 64 channels
//   patch    the picture rows that a tile's pixels lie in and one above and below, W + 2 pixels of 80 bytes each (64 channels and 16 bytes that keep
//            sixteen consecutive pixels on different banks), zeros outside the picture and in a row between two pictures: a tap is a constant
//            distance, without masks.  Two buffers, the next tile's rows are asked for before this one is multiplied
//   weights  36 fragments = 144 registers of a wave that has a SIMD's 512 for itself; they pass through the second buffer's place, so
//            that memory is asked once per workgroup and not once per wave
//   K loop   a pixel fragment (1 KiB of LDS) feeds two matrix instructions; between them the fragments to come are read and the group before is
//            requantised, two outputs at a time, and stored.  No barrier but one per tile
//
// What bounds it, 64 x 56 x 56 pixels in tiles of two and of four rounds, clocks of a workgroup (16400, with a skip operand 17700; 10.7 and 11.1 us a launch, conv_flat.hip
// and conv_plane.hip 13.5 and 16): 3600 until weights and first rows are there, 1900 until the next tile's are asked for (their copies pass the unit's 64 bytes a clock), 1600 a
// round (36 matrix instructions at 32 clocks and what they do not hide; with a skip operand, 100 vector instructions more, 1650), 700 between the tiles, 600 for the last group
// (970).  With a skip operand a round waits for loads that stand behind the next tile's copies, and so for most of those: the first tile's two rounds take 3430
// then, and 4480 at 128 pictures, whose tiles have four rounds' rows to copy.  Taken back: the next tile's copies dealt out between the products (1930 a round
// with a skip operand: the wave issues an instruction every 5 clocks); a pair of outputs behind every second product (1860: a product behind another one waits for
// the unit, and the wave's vector instructions with it); odd tiles that leave their sums where they are, the two sets of registers in turn through all tiles (skip
// operand 11.1 -> 11.4 to 12.7: where ways meet, the compiler waits for more of the loads than it has to).
#include "conv_common.h"

#include <algorithm>
#include <type_traits>

namespace icnn {

constexpr int kKeepPix = 80;                           // bytes of a pixel in LDS
constexpr int kKeepF = 18;                             // K fragments of 32 (9 taps x 64 channels)
constexpr int kKeepWBytes = 2 * kKeepF * 1024;
constexpr int kKeepCopies = 10;                        // KiB of a patch row at most: pictures up to 126 pixels wide
constexpr int kKeepRounds = 8;                         // of a tile at most

struct KeepArgs {
    SkipMul sk;
    unsigned out_bytes, res_bytes;
};

// Products written out: with more registers than a SIMD's 256 vector ones the compiler keeps the sums among the accumulation registers and moves them for every
// product and every vector instruction.  Here the weights are there, which nothing else reads.  The compiler does not know them for products and puts no wait states
// behind them: a round's last two come with the twelve that it gives this product elsewhere, in one statement.  A copy of the compiler's own could still come in front of
// it, so tests/test_keep_waits.py looks for one in the built kernel.  (Two products of one sum have another one between them)
__device__ __forceinline__ void keep_mfma(v16i &sum, const v4i &w, const v4i &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(sum) : "a"(w), "v"(x));
#endif
}
__device__ __forceinline__ void keep_mfma_first(v16i &sum, const v4i &w, const v4i &x, const v16i &start)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %3" : "=&v"(sum) : "a"(w), "v"(x), "v"(start));
#endif
}
__device__ __forceinline__ void keep_mfma_last(v16i (&sum)[2], const v4i &w0, const v4i &w1, const v4i &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %4, %0\n\tv_mfma_i32_32x32x32_i8 %1, %3, %4, %1\n\ts_nop 11" : "+v"(sum[0]), "+v"(sum[1]) : "a"(w0), "a"(w1), "v"(x));
#endif
}

// RES: an unsigned 8-bit skip operand joined before requantisation (g.sk).  The layer requantises as a product's high word (rq_fast); BYTE: to bytes
// (requant_fits_byte).
// hw: H | W << 16; geo: KiB of a patch row | rounds of a tile << 4 | KiB of a buffer << 8 | workgroups / 8 << 16 | rounds of the first tile << 24; share: rounds of a
// workgroup << 8 | workgroups with one more; shifts: of the divisions by W (two) and H (two), a byte each.
template <bool RES, bool BYTE>
__global__ __launch_bounds__(256, 1) void conv_keep_kernel(const uint8_t *x, const uint8_t *wp, const int32_t *bias, const int M, const int in_cs, const unsigned hw,
                                                           const unsigned geo, const unsigned share, const unsigned mul_w, const unsigned mul_h, const unsigned shifts,
                                                           const ConvArgs a, const KeepArgs g)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr unsigned OOB = 0x80000000u;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int H = (int)(hw & 0xffff), W = (int)(hw >> 16);
    const int copies = (int)(geo & 15), most = (int)(geo >> 4 & 15), start = (int)(geo >> 24 & 15), buf_bytes = (int)(geo >> 8 & 0xff) * 1024, pitch = copies * 1024;
    auto by_w = [&](int n) { return fast_div_packed(n, mul_w, shifts & 0xff, shifts >> 8 & 0xff); };
    auto by_h = [&](int n) { return fast_div_packed(n, mul_h, shifts >> 16 & 0xff, shifts >> 24); };
    auto sync = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // this workgroup's rounds; an XCD's workgroups take a contiguous range, so that the rows they share meet in one L2
    const int wg = (int)(blockIdx.x & 7) * (int)(geo >> 16 & 0xff) + (int)(blockIdx.x >> 3);
    const int extra = (int)(share & 0xff), per = (int)(share >> 8);
    const int first = wg * per + min(wg, extra), end = first + per + (wg < extra ? 1 : 0);

    if (first >= end) return;

    // ---- weights and biases, which take the fewest instructions to ask for
    {
        const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)wp, 0, kKeepWBytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < kKeepWBytes / 4096; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (__attribute__((address_space(3))) void *)(lds + buf_bytes + (wave + 4 * i) * 1024), 16,
                                                     (unsigned)((wave + 4 * i) * 1024 + lane * 16), 0, 0, 0);
    }
    v16i b[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) b[c] = bias16(bias + c * 32 + half * 16);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // ---- a tile's patch: its row r is picture row y0 - 1 + r of the pictures one after the other, with a row of zeros before each of them and
    // behind the last.  Copy c of a row brings 16-byte pieces 64 c + lane: piece % 5 of pixel piece / 5, whose first and last are the picture's border
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, 0x7fffff00, 0x00020000);      // (every place inside the tensor lies below 2 GiB, OOB above)
    unsigned piece_at[kKeepCopies];
#pragma unroll
    for (int c = 0; c < kKeepCopies; ++c) {
        if (c >= copies) break;
        const int i = c * 64 + lane, px = (int)(((unsigned)i * 52429u) >> 18), k = i - px * 5;
        piece_at[c] = k < 4 && px >= 1 && px <= W ? (unsigned)((px - 1) * in_cs + k * 16) : OOB;
    }
    struct Tile { int p0, last, v0; };                 // first pixel, last one, place of the patch's first row among the pictures' rows and the rows of zeros
    const int all_rows = by_w(M);
    auto tile_at = [&](int round, int n) {
        Tile t;
        t.p0 = round * 128;
        t.last = min(t.p0 + n * 128, M) - 1;
        const int r = by_w(t.p0);
        t.v0 = r + by_h(r);
        return t;
    };
    // (every fourth row by this wave)
    auto issue_patch = [&](const Tile &t, int b) __attribute__((always_inline)) {
        const int r0 = by_w(t.p0), r1 = by_w(t.last), rows = r1 + by_h(r1) + 3 - t.v0;
        int n = by_h(r0), y = r0 - n * H + wave;       // (y: 0 a row of zeros, else picture row y - 1)
#pragma unroll 1
        for (int r = wave; r < rows; r += 4, y += 4) {
            while (y > H) { y -= H + 1; ++n; }
            const int row = n * H + y - 1;
            const bool ok = y > 0 && row < all_rows;
            const unsigned at = ok ? (unsigned)row * (unsigned)(W * in_cs) : 0u;
#pragma unroll
            for (int c = 0; c < kKeepCopies; ++c)
                if (c < copies)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(lds + b * buf_bytes + r * pitch + c * 1024), 16,
                                                             ok ? piece_at[c] : OOB, at, 0, 0);
        }
        return ((rows - wave + 3) >> 2) * copies;
    };

    int round = first, n = min(start, end - first);    // (a short tile first: its rows are here sooner)
    Tile t = tile_at(round, n);
    const int asked = issue_patch(t, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    in_registers(a.out, a.out_cs, a.out_co, a.lo, a.hi, a.mul_hi, g.out_bytes);
    if constexpr (RES) in_registers(a.res, a.res_cs, g.res_bytes, g.sk.k, g.sk.rnd);
    // the weights have landed where as many younger copies as the patch's are in flight; they are read while those travel
    asm volatile("" ::: "memory");
    if (asked >= 16) ICNN_WAIT_VMCNT(16);
    else if (asked >= 10) ICNN_WAIT_VMCNT(10);
    else if (asked >= 5) ICNN_WAIT_VMCNT(5);
    else ICNN_WAIT_VMCNT(0);
    sync();
    v4i w[2][kKeepF];
#pragma unroll
    for (int f = 0; f < kKeepF; ++f)
#pragma unroll
        for (int c = 0; c < 2; ++c) w[c][f] = *(const v4i *)(lds + buf_bytes + (c * kKeepF + f) * 1024 + lane * 16);
#pragma unroll
    for (int f = 0; f < kKeepF; ++f)
#pragma unroll
        for (int c = 0; c < 2; ++c) asm volatile("" : "+a"(w[c][f]));
    asm volatile("" ::: "memory");
    ICNN_WAIT_VMCNT(0);
    sync();                                            // the first patch is here; every wave has its weights: the next tile's rows may take their place

    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void *)a.out, 0, g.out_bytes, 0x00020000);
    [[maybe_unused]] const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void *)a.res, 0, RES ? g.res_bytes : 0, 0x00020000);

    // a group of this wave: where its taps' rows begin in LDS, what it stores to
    struct Group { int row[3]; unsigned p; };          // p: this lane's pixel, OOB: none
    auto locate = [&](const Tile &t, int b, int j) __attribute__((always_inline)) {
        Group q;
        const int p = t.p0 + j * 128 + wave * 32 + col, pc = min(p, t.last);
        const int r = by_w(pc);
        q.row[0] = b * buf_bytes + (r + by_h(r) - t.v0) * pitch + (pc - r * W) * kKeepPix + half * 16;
        q.row[1] = q.row[0] + pitch;
        q.row[2] = q.row[1] + pitch;
        q.p = p <= t.last ? (unsigned)p : OOB;
        return q;
    };
    constexpr int RING = 6;
    static_assert(kKeepF % RING == 0, "the next group's fragments take the first slots");
    v4i bf[RING];
    auto fetch = [&](const Group &q, auto f_tag, auto slot_tag) __attribute__((always_inline)) {
        constexpr int f = decltype(f_tag)::value, T = f / 2;
        bf[decltype(slot_tag)::value % RING] = *(const v4i *)(lds + q.row[T / 3] + (T % 3) * kKeepPix + (f & 1) * 32);
    };
    auto fetch_first = [&](const Group &q) __attribute__((always_inline)) { static_for<RING - 1>([&](auto f_tag) __attribute__((always_inline)) { fetch(q, f_tag, f_tag); }); };
    struct Sums { v16i s[2]; v4i r8[2]; unsigned p; };
    auto store = [&](unsigned p, int c, const int (&o)[4]) __attribute__((always_inline)) {
        const unsigned at = p == OOB ? OOB : p * (unsigned)a.out_cs + (unsigned)(a.out_co + c * 32 + half * 16);
        __builtin_amdgcn_raw_buffer_store_b128(v4i{o[0], o[1], o[2], o[3]}, rs_y, at, 0, 0);
    };
    auto ask_skip = [&](const Group &q, Sums &s) __attribute__((always_inline)) {
        if constexpr (RES) {
            const unsigned at = q.p == OOB ? OOB : q.p * (unsigned)a.res_cs + (unsigned)(half * 16);
#pragma unroll
            for (int c = 0; c < 2; ++c) s.r8[c] = __builtin_amdgcn_raw_buffer_load_b128(rs_r, at + c * 32, 0, 0);
        }
    };
    auto high = [&](int t) __attribute__((always_inline)) {
        return BYTE ? (int)(((int64_t)t * (a.mul_hi << 8) + 0x8000000000LL) >> 32) : (int)(((int64_t)t * a.mul_hi + 0x80000000LL) >> 32);
    };
    // Multiplies group q, whose first fragments are on their way, into cur.  Between its products: the fragments to come, in the end those of group
    // j (of a tile's last: its own again, not used), and the requantisation and store of the group before, whose place takes group j's skip operand then.
    auto step = [&](const Tile &t, int b_, int j, Group &q, Sums &cur, Sums &old) __attribute__((always_inline)) {
        Group next = q;
        int o[4] = {0, 0, 0, 0}, sum[2] = {0, 0};
        cur.p = q.p;
        __builtin_amdgcn_sched_barrier(0);
        static_for<2 * kKeepF>([&](auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value, f = s / 2, c = s & 1, ahead = f + RING - 1;
            if constexpr (f == 0) keep_mfma_first(cur.s[c], w[c][f], bf[f % RING], b[c]);
            else if constexpr (f < kKeepF - 1) keep_mfma(cur.s[c], w[c][f], bf[f % RING]);
            else if constexpr (c == 1) keep_mfma_last(cur.s, w[0][f], w[1][f], bf[f % RING]);
            __builtin_amdgcn_sched_barrier(0);
            // a pair of the outputs behind two products, in two halves: a product that follows another one at once waits for the matrix unit, and the
            // wave's vector instructions with it
            constexpr int pair = f - 1, oc = pair / 8, R0 = 2 * (pair % 8);
            if constexpr (pair >= 0 && pair < 16 && c == 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    sum[e] = old.s[oc][R0 + e];
                    if constexpr (RES) {
                        const uint32_t x = __builtin_amdgcn_perm((uint32_t)old.r8[oc][(R0 + e) >> 2], g.sk.rnd, 0x00020100u | (uint32_t)(4 + ((R0 + e) & 3)) << 24);
                        sum[e] = __builtin_elementwise_add_sat(sum[e], (int)__umulhi(x, g.sk.k));
                    } else {
                        sum[e] = high(sum[e]);
                    }
                }
            }
            if constexpr (pair >= 0 && pair < 16 && c == 1) {
                if constexpr (RES) {
                    sum[0] = high(sum[0]);
                    sum[1] = high(sum[1]);
                }
                uint32_t two;
                if constexpr (BYTE) {                  // as in epilogue_hi_slice
                    typedef short i16x2 __attribute__((ext_vector_type(2)));
                    two = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, __builtin_amdgcn_cvt_pk_i16(sum[0], sum[1])), i16x2{0, 0}));
                } else {
                    const int lo_v = a.lo;
                    two = __builtin_amdgcn_perm((uint32_t)med3_vvs(sum[1], lo_v, a.hi), (uint32_t)med3_vvs(sum[0], lo_v, a.hi), 0x0c0c0400u);
                }
                if constexpr ((R0 & 2) == 0) o[R0 >> 2] = (int)two;
                else o[R0 >> 2] = (int)__builtin_amdgcn_perm(two, (uint32_t)o[R0 >> 2], BYTE ? 0x07050301u : 0x05040100u);
                if constexpr (pair % 8 == 7) store(old.p, oc, o);
            }
            if constexpr (c == 1) {
                if constexpr (ahead < kKeepF) fetch(q, std::integral_constant<int, ahead>{}, std::integral_constant<int, ahead>{});
                else fetch(next, std::integral_constant<int, ahead - kKeepF>{}, std::integral_constant<int, ahead>{});
            }
            if constexpr (s == 20) {
                next = locate(t, b_, j);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        ask_skip(next, old);
        q = next;
    };

    Sums s0, s1;
    s1.s[0] = b[0]; s1.s[1] = b[1];
    s1.r8[0] = s1.r8[1] = s0.r8[0] = s0.r8[1] = v4i{0, 0, 0, 0};
    s1.p = OOB;
    for (int at = 0;; at ^= 1) {
        const int next_round = round + n, next_n = min(most, end - next_round);
        Tile next = t;
        Group q = locate(t, at, 0);
        fetch_first(q);
        ask_skip(q, s0);
        if (next_n > 0) {
            next = tile_at(next_round, next_n);
            issue_patch(next, at ^ 1);
        }
#pragma unroll 1
        for (int j = 0; j < n; j += 2) {
            step(t, at, min(j + 1, n - 1), q, s0, s1);
            if (j + 1 < n) step(t, at, min(j + 2, n - 1), q, s1, s0);
            else {
                // (not a copy: the compiler makes it in front of the last products, whose sums it then has in s1's place, and without wait states)
                int zero = 0;
                asm volatile("" : "+s"(zero));
#pragma unroll
                for (int c = 0; c < 2; ++c) s1.s[c] = s0.s[c] + zero, s1.r8[c] = s0.r8[c];
                s1.p = s0.p;
            }
        }
        if (next_n <= 0) break;
        // the next tile's rows have landed: younger are two stores a round.  (And with a skip operand loads of it, but not two a round on every way: those that
        // nothing reads are left out.  So they do not count)
        asm volatile("" ::: "memory");
        switch (n) {
        case 1: ICNN_WAIT_VMCNT(2); break;
        case 2: ICNN_WAIT_VMCNT(4); break;
        case 3: ICNN_WAIT_VMCNT(6); break;
        default: ICNN_WAIT_VMCNT(8); break;
        }
        sync();                                        // ... everybody's, and nobody reads this tile's any more
        t = next;
        round = next_round;
        n = next_n;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const v4i o = epilogue_hi16<RES ? 1 : 0, BYTE>(a, g.sk, s1.s[c], s1.r8[c]);
        const int p[4] = {o[0], o[1], o[2], o[3]};
        store(s1.p, c, p);
    }
#endif
}

// ------------------------------------------------------------------ dispatch
namespace {
// LDS bytes of a buffer for tiles of n rounds: the rows that 128 n pixels can lie in, one above and below, and the rows of zeros between pictures
long long keep_buffer(int H, int W, int n)
{
    const long long rows = (128LL * n - 1 + W - 1) / W + 1, pitch = ((W + 2) * kKeepPix + 1023) / 1024 * 1024;
    return std::max<long long>((rows + 2 + (rows - 1 + H - 1) / H) * pitch, kKeepWBytes);
}

bool keep_takes(const ConvArgs &a, bool direct_ok)
{
    if (!direct_ok || a.frag_xor || a.in_xor || a.sh != 1 || a.sw != 1 || a.KH != 3 || a.KW != 3 || a.ph != 1 || a.pw != 1 || a.Cin != 64 || a.Cout != 64) return false;
    if (!a.vec_bias || !a.epi_vec || !a.rq_fast || a.pc || a.out_mode == 3) return false;
    if (a.x_bytes >= 0x7fffff00u || (long long)a.M * a.out_cs >= 0x7fffff00LL || a.M > 0x7fffffff - 2048 || a.H > 0xffff) return false;
    if (a.res_mode != 0 && (a.res_mode != 1 || a.res_dtype != 0 || !make_skip_mul(a.res_mul, a.res_shift).ok || (long long)a.M * a.res_cs >= 0x7fffff00LL)) return false;
    return (a.W + 2) * kKeepPix <= kKeepCopies * 1024 && 2 * keep_buffer(a.H, a.W, 1) <= 160 * 1024;
}
}  // namespace

bool conv_keep_applies(const ConvArgs &a, bool direct_ok)
{
    if (g_tuning.keep == 2) return false;
    if (g_tuning.keep == 1) return keep_takes(a, direct_ok);
    if (g_tuning.tile >= 0 || g_tuning.stages || g_tuning.ksplit || g_tuning.deep_always || g_tuning.halo_always || g_tuning.halo_tile || g_tuning.plane_always ||
        g_tuning.lat || g_tuning.flat == 1)
        return false;
    // Up to 768 tiles of 128 pixels conv_flat.hip has all of them on the chip at once; beyond, this kernel is ahead (us, there / here; 31, 32, 40, 48, 64 and 128
    // images of 56 x 56: 7.0 / 7.5, 8.3 / 7.8, 8.7 / 8.4, 11.7 / 10.1, 12.3 / 11.2, 23.1 / 20.7; with a skip operand 24, 32, 64 and 128: 7.8 / 8.0, 9.9 / 8.8,
    // 16.5 / 14.0, 29.6 / 25.4; 16 images of 112 x 112 13.9 / 12.4 and 16.3 / 14.6).
    return keep_takes(a, direct_ok) && a.M > 768 * 128;
}

hipError_t launch_conv_keep(const ConvArgs &a, hipStream_t st)
{
    if (!keep_takes(a, true) || a.M < 1) return hipErrorInvalidValue;
    const int rounds = (int)((a.M + 127LL) / 128), eighth = std::min(32, (rounds + 7) / 8), wgs = 8 * eighth;
    const int per = rounds / wgs, extra = rounds % wgs, longest = per + (extra ? 1 : 0);
    int most = 1;
    while (most < kKeepRounds && 2 * keep_buffer(a.H, a.W, most + 1) <= 160 * 1024) ++most;
    // a first tile of two rounds, the rest in as few as there are room for, of one length
    const int start = std::min(2, most), rest = std::max(longest - start, 1), tiles = (rest + most - 1) / most;
    most = std::max((rest + tiles - 1) / tiles, start);
    const long long buf = keep_buffer(a.H, a.W, most);
    if (per > 0xffffff || 2 * buf > 160 * 1024) return hipErrorInvalidValue;
    const FastDiv dw = make_fast_div((unsigned)a.W), dh = make_fast_div((unsigned)a.H);
    KeepArgs g;
    g.sk = a.res_mode ? make_skip_mul(a.res_mul, a.res_shift) : SkipMul{0, 0, 0};
    g.out_bytes = (unsigned)(((long long)a.M - 1) * a.out_cs + a.out_co + 64);
    g.res_bytes = a.res_mode ? (unsigned)(((long long)a.M - 1) * a.res_cs + 64) : 0u;
    const bool byte = requant_fits_byte(a);
    const auto kernel = a.res_mode ? byte ? conv_keep_kernel<true, true> : conv_keep_kernel<true, false> : byte ? conv_keep_kernel<false, true> : conv_keep_kernel<false, false>;
    const hipError_t e = allow_large_lds((const void *)kernel);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(256), (size_t)(2 * buf), st, a.x, a.wp, a.bias, a.M, a.in_cs, (unsigned)a.H | (unsigned)a.W << 16,
                       (unsigned)(((a.W + 2) * kKeepPix + 1023) / 1024) | (unsigned)most << 4 | (unsigned)(buf / 1024) << 8 | (unsigned)eighth << 16 | (unsigned)start << 24,
                       (unsigned)per << 8 | (unsigned)extra, dw.mul, dh.mul, dw.s1 | dw.s2 << 8 | dh.s1 << 16 | dh.s2 << 24, a, g);
    return hipGetLastError();
}

}  // namespace icnn
