// Output tiles of the kernels that take a bottleneck block through its three layers.  Plain C++: host code only.
#pragma once

namespace icnn {

// The tile th x tw with th * tw <= pix and (th + 2) * (tw + 2) <= rows that covers an H x W image with the fewest tiles; among
// those the widest, and of its heights the smallest that needs no more tiles.  For a width only the tallest tile can be the best, so
// the widths are walked with that height beside them, which only falls: some 30 to 60 divisions.  (Every pair of sides tried one after
// the other took 3.5 us of the host for 128 x 128 sides, twice per block call, where a launch takes 2.6.)
inline bool fewest_tiles(long long H, long long W, int pix, int rows, int &TH, int &TW)
{
    long long best = -1, down = 0, best_down = 1;
    int th = pix, counted = 0;
    for (int tw = 1; tw <= pix; ++tw) {
        while (th > 0 && ((long long)th * tw > pix || (long long)(th + 2) * (tw + 2) > rows)) --th;
        if (th == 0) break;
        if (th != counted) down = (H + th - 1) / th, counted = th;
        const long long tiles = down * ((W + tw - 1) / tw);
        if (best < 0 || tiles <= best) best = tiles, best_down = down, TW = tw;
    }
    if (best < 0) return false;
    TH = (int)((H + best_down - 1) / best_down);
    return true;
}

// floor(q / d) as (q * inv) >> 16 with inv = 65536 / d + 1 for every q < n: inv * d exceeds 65536 by 1 to d, and the quotient by that
// share of q / 65536, which must not reach the 1 / d between two of them.
inline bool inverse16_exact(unsigned d, unsigned inv, unsigned n)
{
    return n < 2 || (unsigned long long)(n - 1) * ((unsigned long long)inv * d - 65536u) < 65536u;
}

}  // namespace icnn
