"""The host plan of the channel-parallel patch kernel (csrc/wide_plan.h), swept
on the CPU: the cut covers the image, a patch and its lists fit the kernel's
limits, the instantiation exists and holds every position that a patch's
depthwise reads (counted patch by patch here), the LDS fits, and the
multiplications that replace divisions are exact over their ranges."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <stdio.h>
#include <stdlib.h>
#include "wide_plan.h"
using namespace dynconv;
#define REQUIRE(x) do { if (!(x)) { printf("FAILED %s: n %d h %d w %d c %d elem %d e %d: R %d Wu %d\n", #x, s.n, \
    s.h, s.w, s.c, elem, e, g.R, g.Wu); exit(1); } } while (0)

static void check(dynconv_shape s, int elem) {
    const int e = 0;
    const WideGeom g = wide_geom(s, INT64_MAX);
    if (g.R == 0) {
        REQUIRE(elem == 2 && s.c > 128);  // nothing else runs the other widths
        return;
    }
    REQUIRE(g.R >= 1 && g.Wu >= 1 && g.Wu <= kWideMaxCols && g.R * g.Wu <= kWideOwn);
    REQUIRE(g.slots == (g.R + 2) * (g.Wu + 2) && g.slots <= kWideSlots);
    REQUIRE(g.nph * g.R >= s.h && (g.nph - 1) * g.R < s.h && g.npw * g.Wu >= s.w && (g.npw - 1) * g.Wu < s.w);
    // in-image rows and columns of a patch's region
    int need_h = 0, need_w = 0;
    for (int p = 0; p < g.nph; ++p)
        need_h = std::max(need_h, std::min(s.h, p * g.R + g.R + 1) - std::max(0, p * g.R - 1));
    for (int p = 0; p < g.npw; ++p)
        need_w = std::max(need_w, std::min(s.w, p * g.Wu + g.Wu + 1) - std::max(0, p * g.Wu - 1));
    const int pieces = s.c / 8;
    for (int e : {16, 64, 80, 128, 144, 1536}) {
        const WideForm f = wide_form(elem, s.c, e, g.tiles);
        bool built = false;
#define X(KS, EC, NT, ONE) built = built || (f.ks == KS && f.ec == EC && f.nt == NT && f.one == ONE);
        if (elem == 4) { DC_WIDE_FORMS_32(X) } else { DC_WIDE_FORMS_16(X) }
#undef X
        REQUIRE(built);
        REQUIRE(16 * f.nt >= need_h * need_w);
        REQUIRE(32 * f.ks >= s.c && 32 * (f.ks - 1) < s.c);
        REQUIRE(!f.one || e <= f.ec);
        REQUIRE(wide_lds_bytes(elem, f, s.c, g.slots) <= 160 * 1024);
    }
    // the kernel's divisions: i / d == (i * m) >> 20
    const int per = kWideThreads;
    auto exact = [&](int upto, int d, int m) {
        for (int i = 0; i <= upto; ++i)
            if ((unsigned)i * (unsigned)m >> 20 != (unsigned)(i / d)) return false;
        return true;
    };
    REQUIRE(exact(std::max(per, 2 * kWideSlots), g.Wu + 2, g.m_wp));
    REQUIRE(exact(2 * kWideOwn, g.Wu, g.m_wu));
    REQUIRE(exact(g.slots * pieces + 4 * per, pieces, div20_mul(pieces)));
}

static int64_t most(int c, int e, bool dense, int blocks = 1, int64_t fused_patches = 512) {
    WideWork w{};
    for (int b = 0; b < blocks; ++b) w.add(e);
    return wide_most_patches(c, w, dense, fused_patches);
}

// both sides of the measured lines against k_block_fused
static bool lines() {
    WideWork mixed{};
    mixed.add(384);
    mixed.add(160);  // 5 chunks, 544 of 640 channels
    return most(64, 64, true) == INT64_MAX && most(40, 128, false) == INT64_MAX && most(64, 384, true, 3) == 768 &&
           most(64, 384, false) == 768 && most(64, 256, true, 2) == 512 && most(64, 256, false) == 768 &&
           most(48, 288, true) == 512 && most(48, 192, false) == 512 && most(40, 160, false) == 256 &&
           most(32, 384, true) == 256 && wide_most_patches(64, mixed, true, 512) == 512 &&
           // a second round of k_block_fused
           most(64, 384, true, 2, 513) == 1024 && most(64, 256, true, 1, 560) == 1024 &&
           most(48, 288, false, 1, 560) == 1024 && most(40, 160, false, 1, 560) == 512 &&
           most(40, 128, false, 1, 560) == INT64_MAX && most(32, 384, true, 1, 560) == 256;
}

int main() {
    if (!lines()) {
        printf("FAILED lines\n");
        return 1;
    }
    static const int hs[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 14, 17, 20, 28, 31, 40, 48, 56, 64, 100, 109, 112, 128, 144, 224, 500};
    static const int ws[] = {1, 2, 3, 5, 7, 8, 9, 13, 14, 16, 20, 28, 33, 40, 41, 56, 64, 81, 109, 112, 128, 134, 153, 160, 224, 600,
                             1000, 4096};
    long n = 0;
    for (int batch : {1, 2, 8, 64, 1000})
        for (int h : hs)
            for (int w : ws)
                for (int c = 8; c <= 192; c += 8) {
                    if (c <= 64) check({batch, h, w, c}, 4), ++n;
                    if (c <= 128 || c % 32 == 0) check({batch, h, w, c}, 2), ++n;
                }
    printf("%ld plans\n", n);
    return 0;
}
"""


def test_every_plan_fits_its_kernel(tmp_path):
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(SRC)
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-comment", "-Werror=narrowing",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1912_03203_amd", "csrc"),
                        "-o", str(exe), str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "plans" in r.stdout
