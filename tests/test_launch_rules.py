"""Host-side check of how launches are cut (launch_rules.hpp, no GPU): over
sizes up to the largest that the entry points take, every launch stays within
the 2^32 - 1 work-items that one may have."""
import pathlib
import shutil
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2305_00515_amd" / "csrc"

HEAD = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "launch_rules.hpp"
using namespace s4x5;
static int bad = 0;
#define CHECK(x, ...) do { if (!(x) && bad++ < 10) { std::printf("BAD %s: ", #x); std::printf(__VA_ARGS__); std::puts(""); } } while (0)
static const int64_t kItems = 0xffffffffll;
static std::vector<int64_t> sides() {
    std::vector<int64_t> v;
    for (int e = 0; e <= 30; ++e)
        for (int64_t d : {-1, 0, 1})
            if ((1ll << e) + d >= 1 && (1ll << e) + d <= 1 << 30) v.push_back((1ll << e) + d);
    return v;
}
"""

SINGLE = HEAD + r"""
int main() {
    for (int64_t H : sides())
        for (int64_t W : sides()) {
            // images that fit a GPU of 288 GiB beside their smallest outputs
            if ((double)H * W * 2 > 288.0 * (1ll << 30)) continue;
            for (int nb : {1, 2, 4}) {
                const bool planes = nb < 4;
                if (planes && (double)H * W * (nb == 1 ? 9 : 5) > 288.0 * (1ll << 30)) continue;
                const int64_t nt = (W + 4 * nb - 1) / (4 * nb), nq = (H + 3) / 4;
                const int bq = band_steps(nt, nq, 4096, planes);
                const int64_t tiles = nt * ((nq + bq - 1) / bq), groups = (tiles + 63) / 64;
                CHECK(bq >= 1 && tiles < 1ll << 31 && groups * 256 <= kItems, "H %lld W %lld nb %d bq %d", (long long)H, (long long)W, nb, bq);
                if (H * W <= 1ll << 28) CHECK(bq <= 8, "H %lld W %lld", (long long)H, (long long)W);
            }
            for (int64_t B : {1ll, 2ll, 32ll, 4096ll, 1ll << 20, 1ll << 24, 1ll << 26}) {
                if ((double)B * H * W * 8 > 288.0 * (1ll << 30)) continue;
                for (int own : {124, 116})
                    for (int64_t slots : {2048, 4096}) {
                        const int64_t strips = B * ((W + own - 1) / own);
                        if (strips > kLaunchWaves) continue;      // one wave a strip at the least
                        const int n = f32_ranges(slots, strips, (int)H, own == 124 ? 16 : 1 << 30);
                        CHECK(n >= 1 && n <= H && (strips * n + 3) / 4 * 256 <= kItems, "f32 B %lld H %lld W %lld: %d", (long long)B, (long long)H, (long long)W, n);
                    }
            }
        }
    // what the rules are for: short ranges in small batches, 16 rows in large ones
    CHECK(f32_ranges(4096, 3, 256, 16) == 64, "1 x 256^2");
    CHECK(f32_ranges(4096, 32 * 9, 1024, 16) == 64, "32 x 1024^2");
    CHECK(f32_ranges(4096, 1, 3, 16) == 1, "3 rows");
    CHECK(band_steps(512, 2048, 4096, false) == 8 && band_steps(512, 1024, 4096, true) == 1, "8192^2 and planes");
    if (!bad) std::puts("ok");
    return bad != 0;
}
"""

BATCH = HEAD + r"""
#include <random>
struct Job { uint32_t nt; int32_t Ho; };
static int doubled = 0;
static void noalloc(const std::vector<std::pair<int, int>> &sizes, int th) {      // (Wo, Ho) within the budget
    std::vector<Job> jobs;
    int64_t budget = 0, total = 0, again = 0;
    for (auto &s : sizes) {
        jobs.push_back({tile_columns(s.first, 16), s.second});
        budget += budget_tiles(s.first, s.second);
    }
    if (budget > kNoallocMaxTiles || jobs.size() > (size_t)kNoallocMaxImages) return;
    const int fit = batched_fit(jobs.data(), (int)jobs.size(), th, kNoallocTable, &total);
    for (auto &j : jobs) again += batched_count(j, fit ? fit : th);
    CHECK(fit >= th && total == again && total <= kNoallocTable, "%zu of %d x %d: th %d, %lld entries", jobs.size(),
          sizes[0].first, sizes[0].second, fit, (long long)total);
    doubled += fit > th;
    // no higher than needed
    if (fit > th) {
        int64_t less = 0;
        for (auto &j : jobs) less += batched_count(j, fit / 2);
        CHECK(less > kNoallocTable, "%zu of %d x %d: th %d", jobs.size(), sizes[0].first, sizes[0].second, fit);
    }
}
int main() {
    std::mt19937 rng(7);
    for (int th : {4, 16, 32}) {
        // as many as the budget takes of one size
        for (int64_t W : sides())
            for (int64_t H : sides()) {
                const int64_t one = budget_tiles((int)W, (int)H);
                if (one > kNoallocMaxTiles) continue;
                noalloc(std::vector<std::pair<int, int>>(std::min<int64_t>(kNoallocMaxImages, kNoallocMaxTiles / one), {(int)W, (int)H}), th);
            }
        // mixed sizes, filled up to the budget
        for (int rep = 0; rep < 300; ++rep) {
            std::vector<std::pair<int, int>> v;
            const double top = 6 + rng() % 10;
            int64_t budget = 0;
            while (v.size() < (size_t)kNoallocMaxImages) {
                auto side = [&] { return 1 + (int)(rng() % (uint64_t)(1 << (1 + rng() % (int)top))); };
                const int w = side(), h = side();
                if ((budget += budget_tiles(w, h)) > kNoallocMaxTiles) break;
                v.push_back({w, h});
            }
            if (!v.empty()) noalloc(v, th);
        }
    }
    CHECK(doubled > 100, "%d batches took higher bands", doubled);
    // plans: what a launch holds, and an image whose tiles need 32 bits
    int64_t total = 0;
    for (int ppl : {8, 16}) {
        std::vector<Job> tall(12, {tile_columns(1, ppl), 1 << 30});
        CHECK(batched_fit(tall.data(), 12, 4, kLaunchWaves, &total) > 4 && total <= kLaunchWaves && (total + 3) / 4 * 256 <= kItems, "tall");
    }
    Job wide{tile_columns(1 << 30, 8), 200};
    CHECK(batched_fit(&wide, 1, 4, INT32_MAX, &total) == 16 && batched_image_tiles(wide, 16) <= INT32_MAX, "wide");
    std::vector<Job> many(3000, {1u << 24, 8});
    CHECK(batched_fit(many.data(), 3000, 4, INT32_MAX, &total) == 0, "too large");
    if (!bad) std::puts("ok");
    return bad != 0;
}
"""


def run(tmp_path, program):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(program)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-I", str(CSRC), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-3000:]


def test_single_images_and_fp32_batches(tmp_path):
    run(tmp_path, SINGLE)


def test_bands_of_batches(tmp_path):
    run(tmp_path, BATCH)


@pytest.mark.gpu
def test_bands_that_the_table_makes_higher(sobel_lib, gpu, monkeypatch):
    """80 images of 2048 x 1024 in bands of 4 rows are more wave-tiles than the
    allocation-free call's table holds: it takes bands of 8, same bytes."""
    torch = pytest.importorskip("torch")
    from paper_2305_00515_amd import synth
    monkeypatch.setenv("SOBEL4X5_BATCH_TH", "4")
    srcs = [torch.from_numpy(synth.rect_image(2048, 1024, 7 + i)).to(gpu) for i in range(2)] * 40
    want = [sobel_lib.sobel4x5_u8(s)[0] for s in srcs[:2]]
    mags = sobel_lib.sobel4x5_batched_noalloc(srcs)
    torch.cuda.synchronize()
    assert all(torch.equal(m, want[i % 2]) for i, m in enumerate(mags))
