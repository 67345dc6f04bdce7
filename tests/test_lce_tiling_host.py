"""The strips of the depth-wise convolution's passes are chosen on the host in every call: no more heights are looked at than there
are, and the choice is that of a search over every number of strips."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2303_08810_amd", "csrc")

DRIVER = r"""
#include "bra_lce_pairs.h"
#include <cstdio>
#include <cstdlib>
#include <set>
#include <chrono>
using namespace bra;
using namespace bra::lce;

// every number of strips in turn, which is what the shipped functions leave steps out of
static Tiling even_all(const Dims &D, int ldo, long want, long &tiles)
{
    for (int strips = (D.H + 19) / 20;; ++strips) {
        const int height = (D.H + strips - 1) / strips;
        const Tiling T = strips_of(D, height, tiles);
        if (height <= 5 || (tiles >= want && offsets_fit(D, T, ldo))) return T;
    }
}
static bool same(const Tiling &a, const Tiling &b)
{
    return a.pairs == b.pairs && a.xtiles == b.xtiles && a.height == b.height && a.subs == b.subs && a.ytiles == b.ytiles;
}
int main()
{
    Dims D = {};
    for (int H = 1; H < 700; H += 1 + H / 60) {
        for (int W : {1, 5, 28, 200}) for (int B : {1, 3, 40}) for (int C : {64, 768}) {
            D.B = B; D.H = H; D.W = W; D.C = C;
            for (long want : {1L, 30L, 500L, 100000L}) {
                long t0, t1;
                const Tiling a = even_all(D, C, want, t0), b = even_tiling(D, C, want, t1);
                if (!same(a, b) || t0 != t1) { printf("even %d %d %d %d %ld\n", H, W, B, C, want); return 1; }
            }
        }
        // the numbers of strips that forward_tiling() steps through have every height that there is, from the highest on, once
        std::set<int> all, seen;
        for (int strips = (H + 23) / 24, height = 99; height > 4; ++strips) all.insert(height = (H + strips - 1) / strips);
        D.H = H;
        int steps = 0;
        for (int strips = (H + 23) / 24, height;; strips = lower_strips(D, height)) {
            seen.insert(height = (H + strips - 1) / strips);
            ++steps;
            if (height <= 4) break;
        }
        if (all != seen || steps != (int)all.size()) { printf("heights of %d\n", H); return 1; }
    }
    auto ns = [&](int H) {
        D.B = 1; D.H = H; D.W = 64; D.C = 64;
        double best = 1e30;
        for (int r = 0; r < 50; ++r) {
            const auto a = std::chrono::steady_clock::now();
            long sum = 0, n;
            for (int i = 0; i < 20; ++i) { sum += forward_tiling(D, 64, 1, i, n).height + even_tiling(D, 64, 1L << 40, n).height; sum += n; }
            const double t = std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now() - a).count() / 20;
            if (sum == 42) abort();
            if (t < best) best = t;
        }
        return best;
    };
    const double low = ns(512), high = ns(1 << 20);
    printf("%.0f ns, %.0f ns\n", low, high);
    return high > 8 * low;      // 4000 times as many rows; with every number of strips it is more than a thousand times as long
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not found")
def test_strips_of_the_convolution(tmp_path):
    src, exe = tmp_path / "strips.hip", str(tmp_path / "strips")
    src.write_text(DRIVER)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--cuda-host-only", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
