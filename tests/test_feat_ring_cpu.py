"""The feature step's reads of W, followed on the CPU: every launched variant's
ring of operand blocks holds the block that is used, and no load leaves W."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2106_07551_amd", "csrc")

# The loads in the kernel's order: the ring filled, then rounds of `depth` groups.
WALK = r"""
#include "feat_ring.hpp"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace malib;
int main(int, char** v)
{
    const int d = atoi(v[1]), waves = atoi(v[2]), depth = atoi(v[3]);
    const int kg = d / 16, ntw = kg / waves;
    int bad = kg % depth != 0 || ntw * waves != kg;
    for (int w = 0; w < waves && !bad; ++w)
        for (int i = 0; i < ntw; ++i) {
            const int tile = w * ntw + i;
            std::vector<int> ring(depth);
            auto load = [&](int g) {
                const int b = feat_block(tile, g, kg);
                bad |= b < 0 || b >= kg * kg;
                return b;
            };
            for (int s = 0; s < depth; ++s)
                ring[s] = load(s);
            for (int g0 = 0; g0 < kg; g0 += depth)
                for (int h = 0; h < depth; ++h) {
                    bad |= ring[h] != tile * kg + g0 + h;
                    if (feat_refills(g0, depth, kg))
                        ring[h] = load(g0 + h + depth);
                }
        }
    return bad;
}
"""


def test_w_blocks_stay_inside_w(tmp_path):
    src = open(os.path.join(CSRC, "k_env.hip")).read()
    variants = {tuple(map(int, m)) for m in
                re.findall(r"launch_feature<(\d+), (\d+), (\d+), (\d+)>\(f, s\)", src)}
    assert {v[0] for v in variants} == {64, 128, 256, 512}
    # the kernel's loads go through these two functions
    assert len(re.findall(r"load_w4\(W, feat_block\(", src)) == 2 == src.count("load_w4(W,")
    assert src.count("feat_refills(") == 1
    exe = tmp_path / "walk"
    (tmp_path / "walk.cpp").write_text(WALK)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "walk.cpp"),
                           "-o", str(exe)])
    for d, _, waves, depth in sorted(variants):
        assert subprocess.call([str(exe), str(d), str(waves), str(depth)]) == 0, (d, waves, depth)
