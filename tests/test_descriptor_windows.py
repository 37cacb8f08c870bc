"""What the kernels' buffer descriptors cover, from csrc/windows.h compiled for the host:
every offset that a lane forms is a pixel of its row or frame (inside the descriptor and
inside the caller's buffer) or lies outside the descriptor, over sizes up to those where
32-bit byte counts of a whole slice or row would no longer hold."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MOTION = r"""
#include "windows.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
using namespace ulm;
// one slice size: every frame of every frame block, a few bands, every staged pixel
static void check(int K2, int F, int nz, int nu) {
    const size_t npix = (size_t)nz * nu, total = (size_t)K2 * F * npix;
    const int nrc = (nz + kMotRows - 1) / kMotRows, nfb = (F + kMotFrames - 1) / kMotFrames;
    for (int s : {0, K2 - 1})
        for (int f = 0; f < nfb * kMotFrames; ++f)
            for (int rc : {0, nrc / 2, nrc - 1}) {
                const int z0 = rc * kMotRows, rows = std::min(kMotRows, nz - z0), npx = rows * nu;
                const Window w = mot_window(s, F, f, nz, nu, z0, rows);
                bool ok = w.bytes >= 0 && w.at + (size_t)w.bytes / 8 <= total;
                if (f < F) ok = ok && w.at == ((size_t)s * F + f) * npix + (size_t)z0 * nu;
                // a lane's offset is 8 p for every p of the stages that cover the band
                const long long last = (long long)(npx + kMotStage - 1) / kMotStage * kMotStage;
                ok = ok && last * 8 < (1ll << 31);
                for (long long p = 0; p < last; ++p) {
                    const bool inside = (unsigned long long)(8 * p + 8) <= (unsigned)w.bytes;
                    ok = ok && inside == (f < F && p < npx);
                }
                if (!ok) { std::printf("slice %d frame %d band %d of %d x %d x %d\n", s, f, rc, F, nz, nu); std::exit(1); }
            }
}
int main() {
    const int sizes[][4] = {{2, 1, 1, 3}, {2, 31, 5, 7}, {4, 32, 16, 64}, {2, 33, 17, 45}, {18, 300, 250, 274},
                            {2, 64, 16400, 512}, {2, 33, 33001, 509}, {2, 1024, 262144, 553}};
    for (auto &x : sizes) check(x[0], x[1], x[2], x[3]);
    return 0;
}
"""

TRAINING = r"""
#include "windows.h"
#include <cstdio>
#include <cstdlib>
using namespace ulm;
// the first and last strips of a row of W pixels of 64 bytes (BF16) or 128 (FP32)
static void check(int W, int halo) {
    const int strips = (W + kStripCols - 1) / kStripCols;
    for (int s = 0; s < strips; ++s) {
        if (s == 3 && strips > 8) s = strips - 4;
        const int sx = s * kStripCols;
        const Columns c = strip_columns(W, sx, halo);
        bool ok = c.first >= 0 && c.n > 0 && c.first + c.n <= W;
        for (int px = sx - halo; px < sx + kStripCols + halo; ++px)
            for (int pb = 64; pb <= 128; pb *= 2) {
                if (px < 0) { ok = ok && c.n * pb < 0x7ffffff0; continue; }     // the kernels' kPastRow
                const long long off = (long long)(px - c.first) * pb;
                const bool inside = off >= 0 && off + pb <= (long long)c.n * pb;
                ok = ok && off >= 0 && off < (1ll << 31) && inside == (px < W);
            }
        if (!ok) { std::printf("strip %d of %d, halo %d\n", s, W, halo); std::exit(1); }
    }
}
int main() {
    const int widths[] = {1, 31, 32, 33, 64, 65, 274, (1 << 24) + 33, (1 << 25) - 1};
    for (int W : widths) {
        check(W, 0);
        check(W, 1);
    }
    return 0;
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(source)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2511_21647_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("source", [MOTION, TRAINING], ids=["motion", "training"])
def test_windows(tmp_path, source):
    _run(tmp_path, source)
