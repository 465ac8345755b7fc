"""Addresses of the general path's logits (plain_layout.h), walked on the CPU as fixed_score's waves ask for them."""
import os
import subprocess

import paper_2510_07651_amd
from paper_2510_07651_amd import build

CSRC = os.path.join(os.path.dirname(paper_2510_07651_amd.__file__), "csrc")

# Every wave of every workgroup of one KV head, the last of the piece's: row chunks of 128 rows (kRb = 8) or 64 (4), tiles of 32 or 64 tokens, one or
# more tiles per workgroup.  A wave asks for the first block of its part, then for the next while it works on one; all of it has to lie
# among the head's own logits, and a block is asked for before it is scored.
WALK = r"""
#include "plain_layout.h"
#include <algorithm>
#include <cstdio>
using namespace obc;
static int walk(int kRb, int kTok, int nr, int s0, int s1, int len, int n_tiles) {
    const int kPart = kTok / (8 / kRb), blocks = (nr + 15) / 16;
    const Piece w{0, 0, nr, s0, s1, (s1 - s0 + 63) / 64 * 64};
    const size_t head = z_block(w, 1, 0, s0);
    auto inside = [&](int block, int t) { return t >= s0 && t % 16 == s0 % 16 && t + 16 <= s0 + w.z_stride && z_block(w, 0, block, t) + 256 <= head; };
    for (int t_begin = s0; t_begin < s1; t_begin += n_tiles * kTok) {
        const int t_end = std::min(std::min(t_begin + n_tiles * kTok, s1), len);
        if (t_begin >= t_end) continue;
        for (int row0 = 0; row0 < nr; row0 += 16 * kRb)
            for (int wave = 0; wave < 8; ++wave) {
                const int part = wave / kRb, block = std::min(row0 / 16 + wave % kRb, blocks - 1);
                int ahead = t_begin + part * kPart;
                for (int t0 = t_begin; t0 < t_end; t0 += kTok)
                    for (int p0 = part * kPart; p0 < (part + 1) * kPart; p0 += 16) {
                        if (ahead != t0 + p0 || !inside(block, ahead)) return 1;
                        ahead = next_scored(t0, p0, part, kPart, kTok, t_end);
                        if (!inside(block, ahead)) return 2;
                    }
            }
    }
    return 0;
}
int main() {
    int n = 0;
    for (int kRb : {4, 8})
        for (int kTok : {32, 64})
            for (int nr : {1, 33, 64, 129, 200, 512})
                for (int s0 : {0, 128})
                    for (int tokens : {1, 31, 32, 33, 64, 100, 640, 1000})
                        for (int cut : {0, 1, 17, 50})
                            for (int n_tiles : {1, 2, 8}) {
                                const int len = std::max(s0 + tokens - cut, 1), bad = walk(kRb, kTok, nr, s0, s0 + tokens, len, n_tiles);
                                if (bad) return printf("%d: row blocks %d, tile %d, rows %d, tokens %d .. %d of %d, tiles %d\n", bad, kRb, kTok, nr, s0, s0 + tokens, len, n_tiles), 1;
                                ++n;
                            }
    printf("%d walks\n", n);
    return 0;
}
"""


def test_logits_asked_for_ahead_are_the_heads_own(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([build._hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
