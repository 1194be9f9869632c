"""Launch shape of the gain kernel over consecutive frames (fizi_shapes.h), over
every frame count and the ends of the accepted geometries and row strides:
its partial sums fit their array, and each sum the type it is held in."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <limits>
#include "fizi_shapes.h"
using namespace fizi;
int main()
{
    const int widths[] = {64, 128, 640, 1920, 4096, 4160, 8128, 8192};
    const int heights[] = {1, 7, 480, 1080, 4320, 8191, 8192};
    const int strides[] = {1, 2, 8, 64};
    long long checked = 0;
    for (int n = 1; n <= 256; ++n)
        for (int W : widths)
            for (int H : heights)
                for (int rs : strides)
                    for (int px : {16, 4}) {
                        const long long items = (long long)((H + rs - 1) / rs) * (W / px);
                        const GainShape g = gain_span_shape(items, n);
                        const unsigned long long most = 1020ull * px;      // R + 2 G + B of an item
                        const unsigned long long lane = most * g.rounds;
                        const bool ok =
                            g.parts >= 1 && (long long)g.parts * n <= kGainParts && g.threads >= 64 &&
                            g.threads <= 1024 && g.threads % 64 == 0 && g.rounds >= 1 &&
                            (long long)g.parts * g.threads * g.rounds >= items &&
                            most <= 0xFFFFull && lane * 64 <= 0xFFFFFFFFull &&
                            lane * g.threads <= (unsigned long long)std::numeric_limits<GainSum>::max();
                        if (!ok) {
                            std::printf("n %d %dx%d stride %d px %d: parts %d threads %d rounds %d\n", n, W, H, rs, px,
                                        g.parts, g.threads, g.rounds);
                            return 1;
                        }
                        ++checked;
                    }
    std::printf("%lld\n", checked);
    return 0;
}
"""


def test_sums_fit(tmp_path):
    src = tmp_path / "shape.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "shape"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_1907_04393_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) == 256 * 8 * 7 * 4 * 2
