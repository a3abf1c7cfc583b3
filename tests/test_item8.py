"""Offsets of the resident kernels' items of eight sites (csrc/item8.hpp),
compiled for the host: every LDS read of an item lies within its plane and the
eight bytes repeated behind it, and every neighbour byte of a site that is
stored is the right one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <stdio.h>
#include <vector>
#include "item8.hpp"
using u32 = uint32_t;
template <bool AL> int check(u32 W, u32 Ly) {
    const u32 plane = W * Ly, stride = (plane + 15u) & ~7u;
    for (u32 i = 0; i < (plane + 7u) / 8u; ++i) {
        spinmc::Item8<AL> t;
        t.init(i, W, 1.0f / (float)W, plane);
        const u32 near = AL ? plane : plane + 8u;
        const u32 wide = AL ? 8u : 12u, mask = AL ? ~0u : ~3u, one = AL ? 4u : 1u;
        bool ok = t.k == 8u * i && (t.uo & mask) + wide <= stride && (t.dof & mask) + wide <= stride &&
                  t.uo + 8u <= near && t.dof + 8u <= near && t.lo + one <= plane &&
                  t.hi + one <= plane && t.k + (AL ? 8u : 12u) <= stride;
        for (u32 n = 0; ok && n < 8u && t.k + n < plane; ++n) {
            const u32 at = t.k + n, y = at / W, j = at - y * W;
            ok = (t.uo + n) % plane == (y == 0 ? Ly - 1 : y - 1) * W + j &&
                 (t.dof + n) % plane == (y + 1 == Ly ? 0 : y + 1) * W + j;
            if (!AL) {
                const u32 sh = 8u * (n & 3u), w = n >> 2;
                const bool left = (t.left[w] >> sh) & 1u;  // in colour 0
                ok = ok && left == ((y & 1u) == 0u);
                if ((t.start[w] >> sh) & 1u) ok = ok && j == 0 && t.lo == y * W + W - 1;
                if ((t.end[w] >> sh) & 1u) ok = ok && j + 1 == W && t.hi == y * W;
                ok = ok && (j != 0 || ((t.start[w] >> sh) & 1u)) && (j + 1 != W || ((t.end[w] >> sh) & 1u));
            }
        }
        if (!ok) {
            printf("AL %d W %u Ly %u item %u: uo %u dof %u lo %u hi %u plane %u\n", (int)AL, W, Ly, i,
                   t.uo, t.dof, t.lo, t.hi, plane);
            return 1;
        }
    }
    return 0;
}
int main() {
    int bad = 0;
    for (u32 W = 8; W <= 200; ++W)
        for (u32 Ly = 2; Ly <= 40; Ly += 2) bad += W % 8 ? check<false>(W, Ly) : check<true>(W, Ly);
    for (u32 W : {255u, 361u, 1001u, 4094u, 16383u, 32767u})
        for (u32 Ly = 2; W * Ly <= 65536u; Ly += 2) bad += check<false>(W, Ly);
    return bad ? 1 : 0;
}
"""


def test_item_offsets_stay_within_the_planes(tmp_path):
    src, exe = tmp_path / "item8.cpp", tmp_path / "item8"
    src.write_text(SRC)
    inc = os.path.join(ROOT, "paper_2304_01772_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", inc, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[:2000]
