"""Host-side check of the bytes the banded uint8 kernels load (no GPU).

band_cols.hpp says which four bytes a lane loads for a word of its window and
how a byte permute puts them in place.  The same header is compiled with g++
and checked for every width, border rule and tile: every load lies inside the
row, and every byte that a nonzero weight meets is the one the border rule
names (found here by a walk that bounces off the edges).
"""
import pathlib
import shutil
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2305_00515_amd" / "csrc"

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "band_cols.hpp"
using namespace s4x5;
static int bad = 0;
static void fail(const char *what, int W, int x, int bm) {
    if (bad++ < 10) std::printf("BAD %s W=%d x=%d rule=%d\n", what, W, x, bm);
}
// column that the rule reads for column c (-1: none)
static int want(int c, int n, int bm) {
    if (bm == kBandZero) return c < 0 || c >= n ? -1 : c;
    if (bm == kBandRep) return c < 0 ? 0 : c >= n ? n - 1 : c;
    while (c < 0 || c >= n) {
        if (n == 1) return 0;
        c = c < 0 ? -c : 2 * (n - 1) - c;
    }
    return c;
}
static void check_word(int W, int x, int bm, int lo, int hi) {   // columns [lo, hi) are needed
    const int at = window_load(x, W);
    if (at < 0 || (W >= 4 ? at + 4 > W : at != 0)) fail("load", W, x, bm);
    const unsigned sel = window_sel(x, W, bm);
    for (int t = 0; t < 4; ++t) {
        const int c = x + t, s = (sel >> (8 * t)) & 255;
        if (s != 0x0c && s > 3) fail("selector", W, x, bm);
        if (c < lo || c >= hi) continue;
        const int w = want(c, W, bm);
        // rows of fewer than 4 bytes are gathered as bytes 0, 1, 2 (clamped)
        const int got = s == 0x0c ? -1 : W >= 4 ? at + s : (s < W ? s : W - 1);
        if (got != w) fail("byte", W, c, bm);
    }
}
int main() {
    for (int W = 1; W <= 140; ++W)
        for (int bm = 0; bm < 3; ++bm)
            for (int off = 0; off <= 2; ++off) {            // 1, 2: the valid rule
                const int Wo = W - 2 * off, r = off == 1 ? 1 : 2;
                if (Wo < 1 || (off && bm)) continue;
                for (int nb : {1, 2, 4}) {
                    const int nc = 4 * nb, nt = (Wo + nc - 1) / nc;
                    for (int tx = 0; tx < nt; ++tx) {
                        int xo = nc * tx;
                        if (xo > Wo - nc) xo = Wo - nc > 0 ? Wo - nc : 0;
                        const int last = xo + nc < Wo ? xo + nc : Wo;
                        const int lo = xo + off - r, hi = last + off + r;
                        for (int b = 0; b < nb + 2; ++b) check_word(W, xo + off - 4 + 4 * b, bm, lo, hi);
                        // own words of a tile that fits are loaded as they are
                        if (Wo >= nc && (xo + off < 0 || xo + off + nc > W)) fail("own", W, xo, bm);
                    }
                }
            }
    for (int n = 1; n <= 40; ++n)
        for (int bm = 0; bm < 3; ++bm)
            for (int i = -40; i < n + 40; ++i) {
                const int got = band_index(i, n, bm);
                if (got < 0 || got >= n) fail("index range", n, i, bm);
                if (i >= -2 && i < n + 2 && want(i, n, bm) >= 0 && got != want(i, n, bm)) fail("index", n, i, bm);
            }
    std::printf(bad ? "FAIL %d\n" : "ok\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_window_bytes(tmp_path):
    src = tmp_path / "cols.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "cols"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", str(CSRC), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
