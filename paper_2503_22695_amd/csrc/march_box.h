// Boxes of the fused smoothing passes (mg_march.h) and the rule that chooses them; plain
// C++, so that the rule can be checked without a GPU.
#pragma once

#include <algorithm>

namespace hipib {

// Box of a fused smoothing pass: a workgroup owns XO packed columns x JO rows x ZO
// planes; W = XO + 2 HX columns a row with the halo (HX = 0: the whole row)
struct MarchBox {
    int W, XO, HX, JO, ZO, ntx, nty, ntz, threads, lds;
};

enum MarchSource {
    MARCH_ZERO = 0,    // from a zero guess: the red half-sweep x = b / diag
    MARCH_GUESS = 1,   // from the black cells of x (over-relaxed: and the red ones)
    MARCH_CORRECT = 2  // from the red cells of x plus the prolongated coarse correction
};
enum MarchResult {
    MARCH_X = 0,         // both colours of the smoothed x
    MARCH_RESTRICT = 1,  // its red cells and the restricted residual
    MARCH_DOTS = 2,      // both colours, and the partial sums of r.z and z.q
    MARCH_NORM = 3       // both colours, and the partial sums of ||b - A x||^2
};

constexpr int kMarchThreads = 1024;   // threads of a workgroup at most: 128 registers each

// steps beyond the box and its halo: the restriction's two
constexpr int march_extra(int result) { return result == MARCH_RESTRICT ? 2 : 0; }
// halo of the source: one cell per half-sweep, one for a residual and one for its
// restriction
constexpr int march_halo(int ns, int result) {
    return result == MARCH_RESTRICT ? ns + 2 : result == MARCH_NORM ? ns + 1 : ns;
}
// planes before the box at which a pass starts: even where coarse planes go with it
constexpr int march_lead(int src, int ns, int result) {
    return src == MARCH_CORRECT ? (march_halo(ns, result) + 1) / 2 * 2 : march_halo(ns, result);
}
// the same in packed columns; a corrected cell also needs the next column's row value
constexpr int march_halo_x(int src, int ns, int result) {
    return (march_halo(ns, result) + 1) / 2 + (src == MARCH_CORRECT ? 1 : 0);
}
// LDS values per column: two planes of each stage that a later one reads
// in-plane (the last one too where a residual follows), two of the interpolated
// coarse rows, four of the restricted residuals and their x sums; odd, so that a wavefront's 8-byte accesses spread over all banks
constexpr int march_slots(int src, int ns, int result) {
    return 2 * (ns + (result == MARCH_RESTRICT ? 3 : result == MARCH_NORM ? 1 : 0) + (src == MARCH_CORRECT ? 1 : 0)) + 1;
}

// Box of a fused pass.  A step of one workgroup takes about 0.05 us and 0.62 us
// per 1024 resident threads (FP64, measured over boxes of 448 to 1024 threads on
// 64^3 and 128^3: LDS accesses bound it), whatever part of the threads is halo.  The
// box taken has the least rounds x steps x step time: large ones repeat less halo,
// small ones fill the 256 CUs (128^3, one component, down half: 32 x 16 x 8 19.7 us,
// 32 x 8 x 8 27.1, 32 x 16 x 16 24.5; the rule takes 16 x 16 x 16, 20.2, as for the
// down half that also takes the step of r).  FP32 is given half of the step time and
// 2048 threads a CU, the bound of its LDS accesses; the passes hold 46 to 98 registers
// (2048 to 1024 threads) and take 0.8 to 0.95 of the FP64 ones' time at 64^3 and
// 128^3.  With 1024 threads a CU a mixed 128^3 step takes as long (0.999x).
// 1 + 4 / XO stands for the cache lines of a row that are only partly used
// (192^3, three components, up half with the norm: 16 x 28 x 48 174 us,
// 24 x 20 x 48 157; 256^3, down half from an iterate: 32 x 14 x 64 332,
// 16 x 32 x 64 305).
inline MarchBox march_box(int n, int ncomp, int halo, int halo_x, int extra, int slots, int esz) {
    const int H = n / 2;
    MarchBox best{};
    double tbest = 0.0;
    const int resident = esz == 8 ? 1024 : 2048;   // threads per CU with the registers of a pass
    for (int XO : {H, 16, 24, 32, 48, 64}) {
        if (XO > H || XO > 64) continue;
        const int HX = XO == H ? 0 : halo_x, W = XO + 2 * HX;
        for (int JO = 4; JO <= 32 && JO <= n; JO += 2) {
            const int threads = (W * (JO + 2 * halo) + 63) / 64 * 64;
            const int lds = slots * threads * esz;
            if (threads > kMarchThreads || lds > 160 * 1024) break;
            for (int ZO : {4, 8, 12, 16, 24, 32, 48, 64}) {
                if (ZO > n) break;
                const int ntx = (H + XO - 1) / XO, nty = (n + JO - 1) / JO, ntz = (n + ZO - 1) / ZO;
                const int per_cu = (ntx * nty * ntz * ncomp + 255) / 256;
                const int fit = std::min(resident / threads, 160 * 1024 / lds), r = std::min(per_cu, fit);
                const int steps = (ZO + 2 * halo + extra + 3) / 4 * 4;
                const double t = (double)((per_cu + r - 1) / r) * steps * (0.05 + 0.62 * esz / 8 * threads * r / 1024.0) *
                                 (1.0 + 4.0 / XO);
                if (best.XO == 0 || t < tbest) {
                    tbest = t;
                    best = MarchBox{W, XO, HX, JO, ZO, ntx, nty, ntz, threads, lds};
                }
            }
        }
    }
    return best;
}

}  // namespace hipib
