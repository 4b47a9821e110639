"""The tile search of the block kernels against a search over every pair of sides, and its multiply-shift divisors against divisions (host code,
compiled here on its own)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2006_11735_amd", "csrc")

PROGRAM = r"""
#include "block_tile.h"
#include <cstdio>
#include <initializer_list>

static bool every_pair(int H, int W, int pix, int rows, int &TH, int &TW)
{
    long long best = -1;
    for (int th = 1; th <= pix; ++th)
        for (int tw = 1; tw <= pix; ++tw) {
            if (th * tw > pix || (th + 2) * (tw + 2) > rows) continue;
            const long long tiles = (long long)((H + th - 1) / th) * ((W + tw - 1) / tw);
            if (best < 0 || tiles < best || (tiles == best && tw > TW)) best = tiles, TH = th, TW = tw;
        }
    return best >= 0;
}

int main()
{
    const int limits[][2] = {{128, 192}, {64, 96}, {128, 256}, {16, 40}, {1, 9}, {4, 8}, {200, 30}};
    const int large[] = {97, 100, 113, 128, 224, 500, 1023, 4096, 65535, 65537, 1 << 20, 2147483000};
    auto side = [&](int i) { return i < 80 ? i + 1 : large[i - 80]; };
    long long checked = 0;
    for (const auto &l : limits)
        for (int i = 0; i < 92; ++i)
            for (int j = 0; j < 92; ++j) {
                int th = 0, tw = 0, th0 = 0, tw0 = 0;
                const bool ok = icnn::fewest_tiles(side(i), side(j), l[0], l[1], th, tw), ok0 = every_pair(side(i), side(j), l[0], l[1], th0, tw0);
                if (ok != ok0 || th != th0 || tw != tw0) {
                    printf("%d x %d, %d pixels, %d rows: %d x %d, not %d x %d\n", side(i), side(j), l[0], l[1], th, tw, th0, tw0);
                    return 1;
                }
                ++checked;
            }
    for (unsigned d = 1; d <= 400; ++d) {
        const unsigned inv = 65536u / d + 1;
        for (unsigned n : {1u, 2u, 64u, 96u, 128u, 192u, 256u, 5000u, 70000u}) {
            bool exact = true;
            for (unsigned q = 0; q < n; ++q) exact = exact && (unsigned)(((unsigned long long)q * inv) >> 16) == q / d;
            if (icnn::inverse16_exact(d, inv, n) && !exact) { printf("/ %u below %u\n", d, n); return 1; }
            if (!icnn::inverse16_exact(d, inv, n) && n <= 256 && d <= 255) { printf("/ %u below %u refused\n", d, n); return 1; }
        }
    }
    printf("%lld\n", checked);
    return 0;
}
"""


def test_against_every_pair_of_sides(tmp_path):
    source, program = tmp_path / "tile.cpp", tmp_path / "tile"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(program), str(source)], check=True)
    out = subprocess.run([str(program)], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) == 7 * 92 * 92
