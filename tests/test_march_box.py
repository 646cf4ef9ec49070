"""The rule that chooses the boxes of the fused smoothing passes, over every grid
size that the library takes, one to three components, each pass, FP64 and FP32:
what the kernel, its launch and its scratch arrays rely on.  Compiled for the
host (the rule is plain C++)."""
import os
import subprocess

from tests.conftest import ROOT

PROGRAM = r'''
#include <cstdio>
#include <cstdint>
#include "march_box.h"
using namespace hipib;
struct Pass { int src, ns, res; bool fp32; };
int main() {
    // the passes that are compiled (mg.hip): FP32 has no norm
    const Pass passes[] = {{MARCH_ZERO, 3, MARCH_RESTRICT, true}, {MARCH_GUESS, 4, MARCH_RESTRICT, true},
                           {MARCH_CORRECT, 4, MARCH_DOTS, true},  {MARCH_CORRECT, 4, MARCH_X, true},
                           {MARCH_ZERO, 3, MARCH_X, true},        {MARCH_GUESS, 4, MARCH_X, true},
                           {MARCH_CORRECT, 4, MARCH_NORM, false}, {MARCH_GUESS, 4, MARCH_NORM, false}};
    int boxes = 0;
    for (int n : {24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024})
        for (int ncomp = 1; ncomp <= 3; ++ncomp)
            for (const Pass& p : passes)
                for (int esz : {8, 4}) {
                    if (esz == 4 && !p.fp32) continue;
                    const int halo = march_halo(p.ns, p.res), hx = march_halo_x(p.src, p.ns, p.res);
                    const int slots = march_slots(p.src, p.ns, p.res);
                    const MarchBox b = march_box(n, ncomp, halo, hx, march_lead(p.src, p.ns, p.res) - halo + march_extra(p.res), slots, esz);
                    const int H = n / 2;
                    const int64_t count = (int64_t)b.ntx * b.nty * b.ntz;
                    // partials (in doubles): the residual norm's workgroups of 64 x 4 columns of 4 cells
                    const int64_t np = (int64_t)((H + 63) / 64) * (n / 4) * 2 * (n / 4), cap = 6 * (np + 1024);
                    const int64_t used = p.res == MARCH_DOTS ? 2 * count : p.res == MARCH_NORM ? ncomp * count
                                         // ||r||^2 and sum x of conjugate gradients that leave steps open
                                         : p.src == MARCH_ZERO && p.res == MARCH_RESTRICT && ncomp == 1 && n <= 160 ? 5 * np + 2 * count : 0;
                    const bool ok = b.XO > 0 && b.threads % 64 == 0 && b.threads <= kMarchThreads &&
                                    b.threads >= b.W * (b.JO + 2 * halo) && b.lds == slots * b.threads * esz &&
                                    b.lds <= 160 * 1024 && b.lds >= 16 * 8 &&               // (16 doubles for its sums)
                                    b.W == b.XO + 2 * b.HX && (b.HX == hx || (b.HX == 0 && b.XO == H)) &&
                                    (int64_t)b.ntx * b.XO >= H && (b.ntx - 1) * b.XO < H && b.nty * b.JO >= n &&
                                    (b.nty - 1) * b.JO < n && b.ntz * b.ZO >= n && (b.ntz - 1) * b.ZO < n &&
                                    b.JO % 2 == 0 && b.ZO % 4 == 0 &&                       // even corners
                                    halo + 2 <= n && hx <= H &&                             // a halo wraps once
                                    (p.res != MARCH_DOTS || count <= 2 * np) && used <= cap &&
                                    count * ncomp + 7 < (int64_t)1 << 31;
                    if (!ok) {
                        std::printf("n %d comps %d src %d res %d esz %d: box %d x %d x %d, %d threads, %d B, %lld boxes\n", n, ncomp,
                                    p.src, p.res, esz, b.XO, b.JO, b.ZO, b.threads, b.lds, (long long)count);
                        return 1;
                    }
                    ++boxes;
                }
    std::printf("%d boxes\n", boxes);
}
'''


def test_every_pass_has_a_box(tmp_path):
    src, exe = tmp_path / "boxes.cpp", tmp_path / "boxes"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2503_22695_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout == f"{12 * 3 * (8 + 6)} boxes\n"
