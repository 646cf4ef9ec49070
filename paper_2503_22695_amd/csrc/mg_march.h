// Fused smoothing passes of a multigrid level: up to four half-sweeps, and
// what goes with them (the residual and its restriction, the coarse-grid
// correction, the conjugate-gradient dots), in one pass over the level.
//
// A workgroup owns a box of the level (XO packed columns x JO rows x ZO planes)
// and marches along z.  Each thread holds one column (packed ih, row j; both
// colours) of the box or of its halo.  Half-sweep s works on plane z - s at
// step z: the z-neighbours of its cells and one of their two x-neighbours are
// the thread's own values of half-sweep s - 1 (in registers), the other three
// lie in the same plane and were put in LDS by their threads one step earlier,
// so a step needs one barrier whatever the number of half-sweeps.  Every
// value of the halo is recomputed with the arithmetic of the separate
// half-sweeps in the same order; the halo of half-sweep s is DH - s cells wide.
// Rows and planes outside the halo that a half-sweep still needs are skipped.
//
// Why: separate half-sweeps move 12 B per cell (FP64) each and one level's
// V(2,2) half is four launches; fused, the down half reads b (and the guess's
// black cells) and writes the red cells and the coarse right-hand side
// (13 B, 17 with a guess), the up half reads the red cells, b and the coarse
// correction and writes x (21 B).  Small levels were bound by launches and by
// the latency of each pass, large ones by HBM; the fused pass is bound by LDS
// accesses (22 per column and step in the down half) and, from 192^3 with three
// components, by HBM.  Measured in FP64, separate kernels -> fused, us:
//   one component      64^3        128^3       192^3        256^3
//   down half          24 -> 10    35 -> 20    102 -> 35    238 -> 74
//   up half with dots  20 -> 13    35 -> 25    113 -> 57
//   three components, 192^3: down half from an iterate 385 -> 130, up half
//   330 -> 137; 128^3: two over-relaxed sweeps 64 -> 37.
#pragma once

#include "internal.h"

namespace hipib {
namespace {

template <typename T>
struct MarchArgs {
    const T* x;       // guess, or the pre-smoothed x (red cells read)
    const T* b;
    T* out;           // not x: neighbouring workgroups still read it
    const T* e;       // coarse correction (MARCH_CORRECT)
    T* bc;            // coarse right-hand side (MARCH_RESTRICT)
    int n;
    unsigned nboxes;  // boxes of all components
    MarchBox box;
    int64_t cs, ccs;  // component strides of the level and of the next one
    T c, inv_diag, sigma, omega;
    const MGState* st;
    // MARCH_DOTS: r (mixed mode: the FP64 residual; FP64: b itself) and q (also of CG); partial
    // sums of MARCH_DOTS and MARCH_NORM (pstride apart: r.z and z.q, or the components)
    const double* rd;
    const double* qd;
    double* part;
    int64_t pstride;
};

// (arguments of their own: 56 B more cost each launch of the other passes 0.5 us)
template <typename T>
struct MarchCgArgs : MarchArgs<T> {
    // CG: b is formed here as r = rold - alpha qd (mixed mode: r / ||b||, kept in b32),
    // alpha = *rz / (the sum of the npq partials pq), kept in the state; r of the box
    // goes to rnew and the partial sums of ||r||^2 to part
    const double* rold;
    double* rnew;
    float* b32;
    const double* pq;
    int npq;
    const double* rz;
    double* alpha;
};

constexpr int kMarchAhead = 4;        // planes read ahead

// s_barrier with the LDS writes before it visible to the workgroup; global
// memory is not waited for (no thread reads what another one of the launch
// writes there), so loads stay in flight across it
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// base + o + lane, in bytes: a uniform base + o in scalar registers (kept there:
// the compiler would otherwise hold base + lane, two registers per lane and
// array) and a 32-bit offset per lane.  The address space is spelled out because the
// asm hides where the pointer came from; a generic (flat) access would also be
// counted, and waited for, as an LDS access at every barrier.
template <typename T>
using global_t = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ T at_byte(const T* base, int64_t o, uint32_t lane) {
    auto g = (const global_t<char>*)base + o;
    asm("" : "+s"(g));
    return *(const global_t<T>*)(g + lane);
}
template <typename T>
__device__ __forceinline__ void put_byte(T* base, int64_t o, uint32_t lane, T v) {
    auto g = (global_t<char>*)base + o;
    asm("" : "+s"(g));
    *(global_t<T>*)(g + lane) = v;
}

// alpha = rz / (sum of the npq partials of p.q), for every thread of a workgroup of
// whole wavefronts; red: 8 doubles of LDS, free again on return.  The order of the
// sum is that of 512 threads whatever the workgroup, so that a step taken by
// k_cg_close and one taken by a down half are the same to the bit.
__device__ __forceinline__ double cg_alpha(const double* __restrict__ pq, int npq, double rz, double* red) {
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    for (int w = threadIdx.x >> 6; w < 8; w += nw) {
        double a = 0.0;
        for (int t = 64 * w + lane; t < npq; t += 512) a += pq[t];
        for (int o = 32; o > 0; o >>= 1) a += __shfl_down(a, o, 64);
        if (lane == 0) red[w] = a;
    }
    __syncthreads();
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) a += red[w];
    __syncthreads();
    return a != 0.0 ? rz / a : 0.0;
}

// a copy in registers of its own: without it a value read ahead stays where the
// load put it, the next load into its slot goes elsewhere, and the loop ends
// by moving loads in flight (and so by waiting for them)
__device__ __forceinline__ double own_copy(double v) {
    double r;
    asm("v_mov_b64 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ float own_copy(float v) {
    float r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

template <typename T, int SRC, int NS, bool SOR, int RES, bool CG = false>
__global__ void __launch_bounds__(kMarchThreads)
k_march(std::conditional_t<CG, MarchCgArgs<T>, MarchArgs<T>> A) {
    constexpr int PF = kMarchAhead;
    constexpr int DH = march_halo(NS, RES);
    constexpr int q0 = SRC == MARCH_GUESS ? 1 : 0;           // colour of the source
    constexpr int DZ = march_lead(SRC, NS, RES);
    constexpr bool RESID = RES == MARCH_RESTRICT || RES == MARCH_NORM;
    constexpr int NB = RESID ? NS + 1 : NS;                  // stages with a plane pair in LDS
    constexpr int qr = (q0 + NS - 1) & 1;                    // colour of the residual: not the last one's
    constexpr int SL = march_slots(SRC, NS, RES), EX = 2 * NB;   // (EX: row values or residuals)
    // age in planes at which b of a colour is first used
    constexpr int FR = SRC == MARCH_ZERO ? 0 : (q0 == 1 ? 1 : 2), FB = SRC == MARCH_GUESS ? 2 : 1;
    constexpr int NA = NS + 2;                               // ages 0 .. NS + 1
    static_assert(PF == 4, "the coarse rows are read ahead two coarse planes");
    extern __shared__ unsigned char march_lds[];
    T* const L = reinterpret_cast<T*>(march_lds);
    const int n = A.n, H = n >> 1, W = A.box.W, tid = threadIdx.x;
    // each XCD takes a contiguous eighth of the boxes (see xcd_block; the grid is the
    // boxes rounded up to a multiple of 8)
    const unsigned blk = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (blk >= A.nboxes) return;             // uniform
    const int tx = blk % A.box.ntx, ty = (blk / A.box.ntx) % A.box.nty, rest = blk / (A.box.ntx * A.box.nty);
    const int tz = rest % A.box.ntz, comp = rest / A.box.ntz;
    if (!A.st->active[comp]) return;  // uniform
    const int x0 = tx * A.box.XO, j0 = ty * A.box.JO, k0 = tz * A.box.ZO;
    const int xo = min(A.box.XO, H - x0), jo = min(A.box.JO, n - j0), zo = min(A.box.ZO, n - k0);
    const int R = jo + 2 * DH;
    const int64_t half3 = (int64_t)H * n * n;
    const int64_t pst = (int64_t)H * n;      // values per plane of one colour
    const T* const bR = A.b + comp * A.cs;
    const T* const bB = bR + half3;
    const T* const xr = A.x + comp * A.cs;   // red cells of x
    const T* const xs = xr + q0 * half3;     // the source's cells

    // the thread's column: row, LDS positions of its neighbours, global offset
    const int r_ = tid / W, lx = tid - r_ * W;
    const bool in = r_ < R;
    const int rr = in ? r_ : 0;
    const int pos = SL * tid;                // (a thread beyond the box has LDS of its own, too)
    const int sp = in && lx + 1 < W ? pos + SL : (in && A.box.HX == 0 ? pos + SL - SL * W : pos);
    const int sm = in && lx > 0 ? pos - SL : (in && A.box.HX == 0 ? pos - SL + SL * W : pos);
    // the x-neighbour that is not in the own column is at + when the cell's i is
    // odd: sE for an even plane + colour, sO for an odd one
    const bool jodd = ((j0 + rr - DH) & 1) != 0;
    const int sE = jodd ? sp : sm, sO = jodd ? sm : sp;
    const int up = r_ + 1 < R ? pos + SL * W : pos, dn = in && r_ > 0 ? pos - SL * W : pos;
    int ih = x0 + lx - A.box.HX;
    ih = ih < 0 ? ih + H : (ih >= H ? ih - H : ih);
    if (ih >= H) ih = 0;                     // (beyond a partial last tile's halo: not used)
    int j = j0 + rr - DH;
    j = j < 0 ? j + n : (j >= n ? j - n : j);
    const uint32_t goff = (uint32_t)sizeof(T) * (uint32_t)(ih + H * j);
    const bool own = in && r_ >= DH && r_ < DH + jo && lx >= A.box.HX && lx < A.box.HX + xo;

    // v = (b + c * neighbour sum) / diag, over-relaxed v = old + omega (v - old), as
    // wb (b + c * five neighbours) + wo old, then + wk * the neighbour at k + 1
    const T wb = SOR ? A.omega * A.inv_diag : A.inv_diag, wo = T(1) - A.omega, wk = wb * A.c;

    // values of each stage at its last two planes, newest first; b by colour and
    // age in planes; old red cells (over-relaxed guess); what is read ahead
    T hv[NS + 1][2], bh[2][NA], oh = T(0), pb[PF][2], px[PF], po[PF];
#pragma unroll
    for (int s = 0; s <= NS; ++s) hv[s][0] = hv[s][1] = T(0);
#pragma unroll
    for (int a = 0; a < NA; ++a) bh[0][a] = bh[1][a] = T(0);
    const int zs = k0 - DZ, zlast = k0 + zo - 1 + DH;       // planes of the source
    // the next planes to read: byte offsets of the source's plane and of the planes
    // of b that its step needs
    struct Plane {
        int z;
        int64_t o;
    };
    const int64_t pby = pst * (int64_t)sizeof(T);
    auto plane_at = [&](int z) {
        z = z < 0 ? z + n : z;
        return Plane{z, z * pby};
    };
    auto next_plane = [&](Plane& p) {
        p.z += 1;
        p.o += pby;
        if (p.z == n) p = Plane{0, 0};
    };
    Plane nS = plane_at(zs), nR = plane_at(zs - FR), nB = plane_at(zs - FB);
    int zread = zs;                                          // (past the last step: its planes again)
    double pr[PF][2], pq[PF][2], alpha = 0.0;                // CG: r and q in place of b
    constexpr int D8 = 8 / (int)sizeof(T);
    const double inv_bn = CG && sizeof(T) == 4 ? 1.0 / A.st->bn[0] : 1.0;
    auto read_plane = [&](int u) {
        if constexpr (CG) {
            pr[u][0] = at_byte(A.rold, D8 * nR.o, D8 * goff);
            pq[u][0] = at_byte(A.qd, D8 * nR.o, D8 * goff);
            pr[u][1] = at_byte(A.rold + half3, D8 * nB.o, D8 * goff);
            pq[u][1] = at_byte(A.qd + half3, D8 * nB.o, D8 * goff);
        } else {
            pb[u][0] = at_byte(bR, nR.o, goff);
            pb[u][1] = at_byte(bB, nB.o, goff);
        }
        if (SRC != MARCH_ZERO) px[u] = at_byte(xs, nS.o, goff);
        if (SRC == MARCH_GUESS && SOR) po[u] = at_byte(xr, nS.o, goff);
        if (zread < zlast) {
            ++zread;
            next_plane(nR);
            next_plane(nB);
            if (SRC != MARCH_ZERO) next_plane(nS);
        }
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) read_plane(u);
    if constexpr (CG) {
        alpha = cg_alpha(A.pq, A.npq, *A.rz, reinterpret_cast<double*>(march_lds));
        if (blk == 0 && tid == 0) *A.alpha = alpha;
    }

    // coarse correction: yI(K) = e interpolated along y at coarse plane K; the
    // row value of fine plane z is its interpolation along z
    const int nc = n >> 1, Hc = nc >> 1, I = ih, Jn = j >> 1;
    const int64_t halfc = (int64_t)Hc * nc * nc;
    T yA, yB, yC, er[2][2], rw;
    uint32_t eN, eF;
    bool eq;
    const T w0 = T(0.75), w1 = T(0.25);
    const T* const e0 = SRC == MARCH_CORRECT ? A.e + comp * A.ccs : nullptr;
    int Knext = 0;                           // the next coarse plane to read
    auto read_coarse = [&](T& vn, T& vf) {
        const int64_t o = (int64_t)Hc * nc * Knext * (int64_t)sizeof(T);
        const uint32_t hc = (uint32_t)(sizeof(T) * halfc);   // (under 4 GB: nc <= 512)
        const bool q = eq != ((Knext & 1) != 0);             // colour of the near cell; the far one has the other
        vn = at_byte(e0, o, eN + (q ? hc : 0u));
        vf = at_byte(e0, o, eF + (q ? 0u : hc));
        Knext = Knext + 1 == nc ? 0 : Knext + 1;
    };
    if constexpr (SRC == MARCH_CORRECT) {
        int Jf = (j & 1) ? Jn + 1 : Jn - 1;
        Jf = Jf < 0 ? Jf + nc : (Jf >= nc ? Jf - nc : Jf);
        eN = (uint32_t)sizeof(T) * (uint32_t)((I >> 1) + Hc * Jn);
        eF = (uint32_t)sizeof(T) * (uint32_t)((I >> 1) + Hc * Jf);
        eq = ((I + Jn) & 1) != 0;
        Knext = (zs >> 1) - 1;               // (zs is even)
        Knext = Knext < 0 ? Knext + nc : Knext;
        T vn[3], vf[3];
        read_coarse(vn[0], vf[0]);
        read_coarse(vn[1], vf[1]);
        read_coarse(vn[2], vf[2]);
        read_coarse(er[0][0], er[0][1]);
        read_coarse(er[1][0], er[1][1]);
        yA = w0 * vn[0] + w1 * vf[0];
        yB = w0 * vn[1] + w1 * vf[1];
        yC = w0 * vn[2] + w1 * vf[2];
        rw = w0 * yB + w1 * yA;
        L[pos + EX] = rw;
        lds_barrier();
    }
    // cells finished at step z: colour fin[0] (stage NS - 1) on plane z - NS + 1 and
    // (not before a restriction) fin[1] (stage NS) on plane z - NS; their bytes
    T* const outp[2] = {A.out + comp * A.cs + ((q0 + NS - 1) & 1) * half3, A.out + comp * A.cs + ((q0 + NS) & 1) * half3};
    // conjugate-gradient dots: r and q of the finished cells (outside the box those of
    // its nearest cell are read, and not used: no branch around the loads)
    double rq[PF][2][2], da = 0.0, dd = 0.0;
    const uint32_t doff = 8u * (uint32_t)((x0 + min(max(lx - A.box.HX, 0), xo - 1)) + H * (j0 + min(max(r_ - DH, 0), jo - 1)));
    const double zscale = (RES == MARCH_DOTS && sizeof(T) == 4) ? A.st->bn[0] : 1.0;
    auto read_dots = [&](int z, int u) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int P = min(max(z - NS + 1 - t, k0), k0 + zo - 1);
            const int64_t o = (P * pst + ((q0 + NS - 1 + t) & 1) * half3) * 8;
            rq[u][t][1] = at_byte(A.qd, o, doff);
            if (sizeof(T) == 4) rq[u][t][0] = at_byte(A.rd, o, doff);
        }
    };
    if constexpr (RES == MARCH_DOTS) {
#pragma unroll
        for (int u = 0; u < PF; ++u) read_dots(zs + u, u);
    }
    // Restriction of the red residuals: coarse cell (I, J) = (ih, j / 2) of an even
    // row sums rows j - 1 .. j + 2 and planes 2K - 1 .. 2K + 2 with weights 1, 3, 3, 1;
    // a row's two red cells in the window are at I and I + 1 (an odd j + k) or I - 1,
    // with weights 3 and 1.  The x sum of a row is formed one step after its
    // residuals, the sum over the rows one step later.
    T rown = T(0), town = T(0), accN = T(0), accO = T(0);   // own residual, x sum; sums of the planes
    const bool coarse = own && ((r_ - DH) & 1) == 0;
    auto restrict_rows = [&](int P, int ppar) {
        const T* const Lt = L + EX + 2 + ppar;
        const T pl = (Lt[dn] + Lt[pos + 2 * SL * W]) + T(3) * (town + Lt[up]);
        if (ppar) {                              // plane 2K - 1: first of K, third of K - 1
            accO += T(3) * pl;
            accN = pl;
        } else {                                 // plane 2K: second of K, last of K - 1
            const int K = (P >> 1) - 1;
            if (2 * K >= k0 && P <= k0 + zo)
                A.bc[comp * A.ccs + (((I + Jn + K) & 1) ? halfc : 0) + (I >> 1) +
                     (int64_t)Hc * (Jn + (int64_t)nc * K)] = (accO + pl) * T(1.0 / 512.0);
            accO = accN + T(3) * pl;
        }
    };

    // half-sweep s on plane z - s, all but the neighbour at k + 1: the in-plane sum
    // with the own values of half-sweep s - 1 at k and k - 1; old: of the cell itself
    T s4 = T(0);                             // (MARCH_NORM: its four neighbours in half-sweep 4)
    auto partial = [&](int s, int zpar, T own_k, T own_km, T old) {
        const int q = (q0 + s) & 1, ppar = (zpar + s) & 1, sl = 2 * (s - 1) + ppar;
        const T sn = (L[(((ppar + q) & 1) ? sO : sE) + sl] + own_k) + (L[up + sl] + L[dn + sl]) + own_km;
        if (RES == MARCH_NORM && s == 4) s4 = ((L[(((ppar + q) & 1) ? sO : sE) + sl] + own_k) + L[up + sl]) + L[dn + sl];
        T v = wb * (bh[q][s] + A.c * sn);
        if (SOR && (s >= 2 || SRC == MARCH_GUESS)) v += wo * old;
        return v;
    };
    // the rest of it; v: the value of half-sweep s - 1 at k + 1, then the new one
    auto finish = [&](int s, int z, int u, int zpar, T pre, T& v) {
        v = pre + wk * v;
        hv[s][1] = hv[s][0];
        hv[s][0] = v;
        if (s < NB) L[pos + 2 * s + ((zpar + s) & 1)] = v;
        const int P = z - s, t = s == NS ? 1 : 0;
        if (s >= NS - 1 && !(s == NS && RES == MARCH_RESTRICT) && P >= k0 && P < k0 + zo && own) {
            put_byte(outp[t], P * pby, goff, v);
            if constexpr (RES == MARCH_DOTS) {
                const double zv = zscale * (double)v;
                const double rv = sizeof(T) == 8 ? (double)bh[(q0 + s) & 1][s] : rq[u][t][0];
                da += rv * zv;
                dd += zv * rq[u][t][1];
            }
        }
    };

    // CG: ||r||^2 over the box by colour (k_cg_close sums in the same order)
    double rc[2] = {0.0, 0.0};
    // ||b - A x||^2 over the box, both colours (the last half-sweep's neighbours are
    // final, so its cells' residuals follow from what it read).  Where a tight
    // tolerance stops, the norm is the rounding of A x: half of it is in each colour,
    // and a sum of neighbours in the order in which the cell was relaxed would hide its
    // part.  So the terms are those of k_resid_norm.
    double rn = 0.0;
    auto residual = [&](T b, T x, T s4, T kp, T km) {
        return b - (A.sigma * x - A.c * (((s4 + kp) + km) - T(6) * x));
    };

    // A step runs the half-sweeps in three groups: the source and half-sweep 1, then
    // 2 and 3, then the rest.  Inside a group the code is straight-line: all in-plane
    // sums read what the steps before wrote, so the LDS reads are issued together,
    // and the chain from one half-sweep to the next is one operation long.  A group
    // is skipped by the wavefronts whose rows lie in the part of the halo that it
    // does not need, and in the steps before its first plane (LDS accesses bound
    // the pass); cells of a group that are not needed are computed from whatever
    // is there and used by no cell of the box, and the last steps, up to a
    // multiple of PF, finish none.
    const int r_lo = __builtin_amdgcn_readfirstlane(r_);
    const int r_hi = __builtin_amdgcn_readfirstlane((tid | 63) / W);
    const bool rows1 = r_hi >= 2 && r_lo < R - 2, rows2 = r_hi >= 4 && r_lo < R - 4;
    const int steps = zo + DZ + DH + march_extra(RES);
    for (int z0 = 0; z0 < steps; z0 += PF) {
        const bool group1 = rows1 && z0 >= 4, group2 = rows2 && z0 >= 8;
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int z = zs + z0 + u;
            constexpr int ZP = DZ & 1;       // parity of zs (k0 is even)
            const int zpar = (ZP + u) & 1;
#pragma unroll
            for (int a = NA - 1; a > 0; --a) {
                bh[0][a] = bh[0][a - 1];
                bh[1][a] = bh[1][a - 1];
            }
            if constexpr (CG) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const double r = pr[u][q] - alpha * pq[u][q];
                    bh[q][q ? FB : FR] = sizeof(T) == 4 ? (T)(r * inv_bn) : (T)r;
                    const int P = z - (q ? FB : FR);
                    if (P >= k0 && P < k0 + zo && own) {
                        rc[q] = fma(r, r, rc[q]);
                        put_byte(A.rnew + q * half3, D8 * (P * pby), D8 * goff, r);
                        if (sizeof(T) == 4) put_byte(A.b32 + q * half3, P * pby, goff, (float)(r * inv_bn));
                    }
                }
            } else {
                bh[0][FR] = own_copy(pb[u][0]);
                bh[1][FB] = own_copy(pb[u][1]);
            }
            const T pre1 = partial(1, zpar, hv[0][0], hv[0][1], oh);
            T v;
            if constexpr (SRC == MARCH_ZERO) {
                v = wb * bh[0][0];
            } else if constexpr (SRC == MARCH_GUESS) {
                v = own_copy(px[u]);
                if (SOR) oh = own_copy(po[u]);
            } else {
                // the correction at the red cell: I and I + 1 (odd i) or I - 1
                const T side = L[(zpar ? sO : sE) + EX + zpar];
                v = px[u] + (w0 * rw + w1 * side);
                // the row values of plane z + 1
                if (u & 1) {
                    yA = yB;
                    yB = yC;
                    yC = w0 * er[u >> 1][0] + w1 * er[u >> 1][1];
                    read_coarse(er[u >> 1][0], er[u >> 1][1]);
                    rw = w0 * yB + w1 * yA;
                } else {
                    rw = w0 * yB + w1 * yC;
                }
                L[pos + EX + 1 - zpar] = rw;
            }
            read_plane(u);
            const T m0 = hv[0][1], k1 = hv[1][0], m1 = hv[1][1];   // (own values the next group needs)
            hv[0][1] = hv[0][0];
            hv[0][0] = v;
            L[pos + zpar] = v;
            finish(1, z, u, zpar, pre1, v);
            if (group1) {
                const T pre2 = partial(2, zpar, k1, m1, m0), pre3 = partial(3, zpar, hv[2][0], hv[2][1], m1);
                const T m2 = hv[2][1], k3 = hv[3][0], m3 = hv[3][1];
                finish(2, z, u, zpar, pre2, v);
                finish(3, z, u, zpar, pre3, v);
                if (NB > 3 && group2) {
                    constexpr int S4 = NS >= 4 ? 4 : 3;
                    T pre4 = T(0), kr = k3, mr = m3, xv = m2;
                    if constexpr (NS >= 4) {
                        pre4 = partial(4, zpar, k3, m3, m2);
                        kr = hv[S4][0];
                        mr = hv[S4][1];
                        xv = m3;
                    }
                    T rpre = T(0), rside = T(0);
                    const int ppar = (zpar + NS + 1) & 1;         // parity of the residual's plane
                    if constexpr (RESID) {
                        const T* const Lp = L + 2 * NS + ppar;
                        const T side = Lp[((ppar + qr) & 1) ? sO : sE];
                        if constexpr (RES == MARCH_NORM) {
                            rpre = ((side + kr) + Lp[up]) + Lp[dn];
                        } else {
                            const T sn = (side + kr) + (Lp[up] + Lp[dn]) + mr;
                            rpre = bh[qr][NS + 1] - (A.sigma * xv - A.c * (sn - T(6) * xv));
                        }
                    }
                    if constexpr (RES == MARCH_RESTRICT) {
                        rside = L[EX + 1 - ppar + ((1 - ppar) ? sE : sO)];
                        if (coarse && z - NS - 3 >= k0 - 1) restrict_rows(z - NS - 3, ppar);
                    }
                    const T v3 = v;                               // of half-sweep 3 at k + 1
                    if constexpr (NS >= 4) finish(4, z, u, zpar, pre4, v);
                    if constexpr (RES == MARCH_RESTRICT) {
                        // x sum of the residuals of plane z - NS - 2, then the red residuals of
                        // plane z - NS - 1 (the last half-sweep was black)
                        town = T(3) * rown + rside;
                        L[pos + EX + 2 + 1 - ppar] = town;
                        rown = rpre + A.c * v;
                        L[pos + EX + ppar] = rown;
                    }
                    if constexpr (RES == MARCH_NORM) {
                        const int P = z - NS - 1;
                        const T res = residual(bh[qr][NS + 1], xv, rpre, v, mr), last = residual(bh[q0][4], v, s4, v3, m3);
                        if (own && P >= k0 && P < k0 + zo) rn += (double)res * (double)res;
                        if (own && P + 1 >= k0 && P + 1 < k0 + zo) rn += (double)last * (double)last;
                    }
                }
            }
            if constexpr (RES == MARCH_DOTS) read_dots(z + PF, u);
            lds_barrier();
        }
    }
    if constexpr (RES == MARCH_DOTS || RES == MARCH_NORM || CG) {
        double* const red = reinterpret_cast<double*>(march_lds);   // (the last barrier is behind every read)
        const double sa = block_sum(RES == MARCH_DOTS ? da : CG ? rc[0] + rc[1] : rn, red);
        const double sd = RES == MARCH_DOTS ? block_sum(dd, red) : 0.0;
        if (tid == 0) {
            if (RES == MARCH_DOTS) {
                A.part[blk] = sa;
                A.part[A.pstride + blk] = sd;
            } else {
                A.part[comp * A.pstride + blk % A.pstride] = sa;   // (pstride: boxes per component)
            }
        }
    }
}

}  // namespace
}  // namespace hipib
