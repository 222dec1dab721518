"""The order of a launch's items (csrc/order.h), run on the host: every fragment of a frame is filtered once, with
and without merged pairs, for grids, fixations and ramps of all kinds."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "order.h"

using namespace fov;

static int fail(const FrameDesc& d, const char* what, int merge) {
    std::printf("%s (merge %d): h %d w %d block %d origin %d %d fix %g %g e0 %g slope %g cap %g map %d\n", what, merge, d.h, d.w,
                d.p.block, d.p.origin_x, d.p.origin_y, d.p.fix_x, d.p.fix_y, d.p.e0, d.p.slope, d.p.cap, d.p.sigma_map != nullptr);
    return 1;
}

int main() {
    std::mt19937_64 rng(7);
    const auto real = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
    const auto pick = [&](int n) { return (int)(rng() % n); };
    const float map_tag = 0.0f;
    for (int trial = 0; trial < 4000; ++trial) {
        const int nf = trial % 3 ? 1 : 1 + pick(4);
        const bool alike = pick(2);
        std::vector<FrameDesc> fr(nf);
        for (int f = 0; f < nf; ++f) {
            FrameDesc& d = fr[f];
            d = f && alike ? fr[0] : FrameDesc{};
            if (!f || !alike) {
                d.p.block = 1 + pick(64);
                d.h = 1 + pick(pick(3) ? 400 : 3 * d.p.block);
                d.w = 1 + pick(pick(3) ? 400 : 3 * d.p.block);
                d.p.origin_x = -pick(d.p.block);
                d.p.origin_y = -pick(d.p.block);
                d.p.nbx = grid_extent(d.w, d.p.origin_x, d.p.block);
                d.nby = grid_extent(d.h, d.p.origin_y, d.p.block);
            }
            const double far = pick(8) == 0 ? std::pow(10.0, real(0, 300)) : 400.0;
            d.p.fix_x = real(-0.3, 1.3) * (pick(4) ? d.w : far);
            d.p.fix_y = real(-0.3, 1.3) * (pick(4) ? d.h : far);
            d.p.e0 = pick(3) ? real(0, 60) : real(-80, 400);
            if (pick(40) == 0) d.p.e0 = (pick(2) ? 1 : -1) * std::pow(10.0, real(0, 308));
            d.p.slope = pick(20) ? std::pow(10.0, real(-3, 1)) : (pick(2) ? 0.0 : 1e-310);
            d.p.cap = pick(20) ? real(0, 20) : (pick(2) ? 0.0 : 1e-320);
            if (pick(5) == 0) {  // a cap that some fragment's sigma meets exactly, or misses by a rounding
                d.p.cap = 1e300;
                const double s = fragment_sigma_ramp(d.p, pick(d.p.nbx), pick(d.nby));
                if (s < 1e100) d.p.cap = std::nextafter(s, pick(2) ? 1e300 : 0.0);
                if (pick(2)) d.p.cap = s < 1e100 ? s : 1.0;
            }
            d.p.sigma_map = pick(10) ? nullptr : &map_tag;
            d.ahead_x = lines_ahead(d.p.fix_x, d.p.origin_x, d.p.block, d.p.nbx);
            d.ahead_y = lines_ahead(d.p.fix_y, d.p.origin_y, d.p.block, d.nby);
        }
        // sigmas: a map's are drawn, often the cap
        std::vector<std::vector<double>> sigma(nf);
        for (int f = 0; f < nf; ++f)
            for (int by = 0; by < fr[f].nby; ++by)
                for (int bx = 0; bx < fr[f].p.nbx; ++bx)
                    sigma[f].push_back(fr[f].p.sigma_map ? (pick(3) ? fr[f].p.cap : real(0, 1) * fr[f].p.cap)
                                                         : fragment_sigma_ramp(fr[f].p, bx, by));
        for (int merge = 0; merge < 2; ++merge) {
            std::vector<int32_t> prefix(nf + 1);
            const int64_t total = number_items(fr.data(), nf, merge, prefix.data());
            if (prefix[0] != 0 || prefix[nf] != total) return fail(fr[0], "prefix", merge);
            for (int f = 0; f < nf; ++f) {
                const FrameDesc& d = fr[f];
                if (alike && prefix[f + 1] - prefix[f] != prefix[1]) return fail(d, "frames of one grid differ", merge);
                std::vector<int> done((size_t)d.p.nbx * d.nby);
                int empty = 0;
                for (int k = 0; k < prefix[f + 1] - prefix[f]; ++k) {
                    const Place p = item_place(grid_of(d), k, merge);
                    if (p.bx < 0 || p.bx >= d.p.nbx || p.by < 0 || p.by >= d.nby) return fail(d, "out of the grid", merge);
                    const auto at = [&](int by) { return sigma[f][(size_t)by * d.p.nbx + p.bx]; };
                    int rows = 1, first = p.by;  // as decode() in forward.hip does
                    if (merge && at(p.by) == d.p.cap && radius_of(d.p.cap) > 0) {
                        const int by2 = p.by ^ 1;
                        if (by2 < d.nby && at(by2) == d.p.cap) {
                            rows = p.box && ((__builtin_popcount((p.by >> 1) ^ p.bx) ^ p.by) & 1) ? 0 : 2;
                            first = p.by & ~1;
                        }
                    }
                    empty += rows == 0;
                    for (int r = 0; r < rows; ++r) ++done[(size_t)(first + r) * d.p.nbx + p.bx];
                }
                for (int v : done)
                    if (v != 1) return fail(d, v ? "filtered twice" : "left out", merge);
                // a ramp's empty items lie in the corners of a rectangle around a disc
                if (nf == 1 && !d.p.sigma_map && d.p.slope > 1e-3 && std::fabs(d.p.e0) < 1e3 && d.p.cap > 0 && std::fabs(d.p.fix_x) + std::fabs(d.p.fix_y) < 1e4 &&
                    empty > 40 + (int)done.size() / 4)
                    return fail(d, "many empty items", merge);
            }
        }
    }
    std::puts("ok");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2012_08655_amd", "csrc"), "-o", str(d / "order"),
                    str(d / "order.cpp")], check=True)
    return d / "order"


def test_every_fragment_once(program):
    r = subprocess.run([str(program)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
