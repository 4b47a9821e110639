// Two-dimensional tiles of a picture, for the kernels whose persistent workgroups keep a layer's weights in LDS and take one tile after the
// other with the input patch under it in LDS (conv_plane.hip, conv_rows.hip): the walk over the tiles, the patch, the copies.
#pragma once
#include "conv_common.h"

#include <type_traits>

namespace icnn {

// Work slot v (blockIdx.x, + gridDim.x, ...; the grid is a multiple of 8) is tile (v & 7) * per_xcd + (v >> 3): the workgroups of an XCD
// walk a contiguous range of tiles, so the patch borders neighbouring tiles share meet in one L2.
struct TileWalk {
    int tiles_x, tiles_per_img, n_tiles;
    int per_xcd;                // tiles handed to each of the 8 XCDs
    FastDiv div_tpi, div_tx;    // / tiles_per_img, / tiles_x

    __device__ __forceinline__ int tile_of(int v) const { return (v & 7) * per_xcd + (v >> 3); }
    __device__ __forceinline__ bool valid(int v) const { return (v >> 3) < per_xcd && tile_of(v) < n_tiles; }
    // picture and first pixel of slot v's tile of TH x TW pixels
    template <int TH, int TW>
    __device__ __forceinline__ void origin(int v, int &n, int &y0, int &x0) const
    {
        const int t = tile_of(v);
        n = fast_div(t, div_tpi);
        const int r = t - n * tiles_per_img;
        const int ty = fast_div(r, div_tx);
        y0 = ty * TH;
        x0 = (r - ty * tiles_x) * TW;
    }
};

// host: the walk over N pictures of H x W in tiles of th x tw; false where their number does not fit
inline bool tile_walk(TileWalk &g, int N, int H, int W, int th, int tw)
{
    g.tiles_x = (W + tw - 1) / tw;
    g.tiles_per_img = g.tiles_x * ((H + th - 1) / th);
    const long long tiles = (long long)g.tiles_per_img * N;
    if (tiles < 1 || tiles > 0x7ffffff0LL / 8) return false;
    g.n_tiles = (int)tiles;
    g.per_xcd = (int)((tiles + 7) / 8);
    g.div_tpi = make_fast_div((unsigned)g.tiles_per_img);
    g.div_tx = make_fast_div((unsigned)g.tiles_x);
    return true;
}

// Input patch of a "same" KS x KS layer of CIN channels (48 or 64) under a tile of TH x TW pixels, copied by WAVES waves.
// Layout in LDS: pixel (py, px) at (py * PWL + px) * CIN.  64-byte pixels: the 16-byte piece c of a pixel lives in slot
// c ^ ((px >> 2) & 3), so that the fragment reads of 16 consecutive pixels hit every bank once (rows are whole multiples of 256
// bytes, so the row does not enter); 48-byte pixels spread over the banks by themselves.
template <int KS, int CIN, int TH, int TW, int WAVES>
struct TilePatch {
    static constexpr int PAD = KS / 2;
    static constexpr int PH = TH + KS - 1, PW = TW + KS - 1;
    static constexpr int PWL = (PW + 3) & ~3;               // pixels per patch row in LDS: whole groups of four
    static constexpr int PPT = CIN / 16;                    // 16-byte pieces per pixel (= per tap)
    static constexpr int ROWB = PWL * CIN;                  // bytes per patch row
    static constexpr int PIECES = PH * PWL * PPT;
    static constexpr int NCOPY = (PIECES + 63) / 64;        // wave-wide 1 KiB copies per patch
    static constexpr int CPW = (NCOPY + WAVES - 1) / WAVES; // per wave
    static constexpr int BYTES = NCOPY * 1024;
    static_assert(CIN == 48 || CIN == 64, "row layouts exist for 48 and 64 channels");

    // Copy e of a patch covers LDS bytes [1024 e, 1024 e + 1024): what this lane fetches for each of its copies does not depend on the
    // tile but for the origin: the piece's offset from the patch's first pixel, and (py, px) for the check against the
    // picture's borders (a lane beyond the patch gets py = 0x7fff, which never passes it).
    int rel[CPW], yx[CPW];
    __device__ __forceinline__ void locate(const ConvArgs &a, int wave, int lane)
    {
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            const int q = (wave + WAVES * i) * 64 + lane;
            const int pix = q / PPT, slot = q - pix * PPT;
            const int py = pix / PWL, px = pix - py * PWL;
            const int logical = CIN == 64 ? slot ^ ((px >> 2) & 3) : slot;
            const bool in_patch = q < PIECES && px < PW;
            rel[i] = (py * a.W + px) * a.in_cs + logical * 16;
            yx[i] = ((in_patch ? py : 0x7fff) << 16) | px;
        }
    }
    // byte offset of the patch's first pixel, picture pixel (n, y0 - PAD, x0 - PAD) (may be negative: only pixels inside the picture use it)
    static __device__ __forceinline__ int base(const ConvArgs &a, int n, int y0, int x0) { return ((n * a.H + y0 - PAD) * a.W + x0 - PAD) * a.in_cs; }
#if defined(__HIP_DEVICE_COMPILE__)   // the buffer-resource type exists in the device pass only
    // copy I of this wave for that patch, into the buffer at dst
    template <int I>
    __device__ __forceinline__ void issue(const __amdgpu_buffer_rsrc_t &rs_x, const ConvArgs &a, uint8_t *dst, int wave, int from, int y0, int x0) const
    {
        const int e = wave + WAVES * I;
        if (e < NCOPY) {                             // wave-uniform
            const int iy = y0 - PAD + (yx[I] >> 16), ix = x0 - PAD + (yx[I] & 0xffff);
            const bool ok = ((unsigned)iy < (unsigned)a.H) & ((unsigned)ix < (unsigned)a.W);
            const unsigned off = ok ? (unsigned)(from + rel[I]) : 0x80000000u;      // beyond any buffer these kernels accept (< 2 GiB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(dst + e * 1024), 16, off, 0, 0, 0);
        }
    }
#endif
};

#if defined(__HIP_DEVICE_COMPILE__)
// A layer's packed weights (BYTES of them, whole KiB) to LDS as they are, by WAVES waves: direct copies of 1 KiB per wave, all in flight together
// with the first patch.  (Through registers the copy loop waited out one memory latency per 8 KiB, five of them for a 3x3 layer of
// 64 channels, which is most of the kernel's time on a picture with one tile per workgroup.)  UNROLL: not where a wave has many copies and the
// tile loop behind them all the registers: unrolled, the addresses of seventeen copies are held across it.
template <int WAVES, int BYTES, bool UNROLL = true>
__device__ __forceinline__ void copy_packed_weights(const uint8_t *wp, unsigned wp_bytes, uint8_t *dst, int wave, int lane)
{
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)wp, 0, wp_bytes, 0x00020000);
    auto copy = [&](int e) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (__attribute__((address_space(3))) void *)(dst + e * 1024), 16, (unsigned)(e * 1024 + lane * 16), 0, 0, 0);
    };
    if constexpr (UNROLL) {
#pragma unroll
        for (int e0 = 0; e0 < BYTES / 1024; e0 += WAVES)
            if (e0 + wave < BYTES / 1024) copy(e0 + wave);      // wave-uniform
    } else {
        for (int e = wave; e < BYTES / 1024; e += WAVES) copy(e);
    }
}
#endif

}  // namespace icnn
