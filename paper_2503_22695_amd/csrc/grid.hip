// Pointwise MAC-grid kernels of the Chorin step ("Spatial Discretization"):
// right-hand side with explicit flux-form convection, divergence of the
// intermediate velocity, and the velocity correction.  All three stream the
// grid once in 64x4 thread tiles, so each wavefront reads 64 consecutive
// x-cells (512 B) per array; one thread per cell, or per z column of cells for
// the right-hand side.
#include "internal.h"

#include <algorithm>

namespace hipib {
namespace {

constexpr int TX = 64, TY = 4;
constexpr int kColumn = 8, kColumnBlocks = 1024;   // k_rhs_build: cells of a column, workgroups it should leave

struct Grid3 {
    int n;
    int64_t n3;
    __device__ __forceinline__ int64_t at(int i, int j, int k) const {
        return (int64_t)i + (int64_t)n * ((int64_t)j + (int64_t)n * k);
    }
};

// the double at a byte offset from a base
__device__ __forceinline__ double at_byte(const double* base, uint32_t o) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + o);
}

// 0.5 (a + b) * 0.5 (v + w): the flux of one component through an edge
__device__ __forceinline__ double edge_flux(double a, double b, double v, double w) {
    return 0.5 * (a + b) * (0.5 * (v + w));
}
// (0.5 (c + p))^2 - (0.5 (m + c))^2: the difference of the normal flux over a face
__device__ __forceinline__ double normal_flux(double m, double c, double p) {
    const double ap = 0.5 * (c + p), am = 0.5 * (m + c);
    return ap * ap - am * am;
}

// As xcd_block with slabs of rows (y) in place of planes: workgroups in flight then
// cover a few planes of a slab, and three components with their neighbours fit
// the XCD's L2; a slab of planes holds whole planes in flight (256^3: 1.5 MB each,
// every one read 2.7 times).
__device__ __forceinline__ uint3 xcd_rows() {
    const unsigned gx = gridDim.x, gy = gridDim.y;
    if (gy & 7u) return xcd_block();
    const unsigned b = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), r = b >> 3, rows = gy >> 3;
    return make_uint3(r % gx, (b & 7u) * rows + (r / gx) % rows, r / (gx * rows));
}

// g = rho/dt u - rho C(u) + f with (upk) u packed as the Helmholtz guess.  C^d at
// face (i,j,k) of component d in conservative centred form:
//   normal flux at cell centres ((u^d[c] + u^d[c+e_d]) / 2)^2,
//   tangential flux at edges ((u^d[c-e_e] + u^d[c]) / 2)((u^e[c-e_d] + u^e[c]) / 2).
// HBM bound (48 B per cell, 24 more with f and 24 more with upk).
// A thread takes kz cells of a z column: the 27 values a cell needs are 17 reads,
// the others are those of the plane before; the rest is read through L1 and, with
// every XCD on its own slab of rows, its L2.  A cell's reads are issued before the
// stores of the one below: a wait for a read also waits for every store before it.
// One thread per cell, planes in launch order -> this: 58 -> 41 us at 128^3 (beside the
// element forces; 72 B), 265 -> 170 at 192^3, 634 -> 397 at 256^3 (96 B, 4.1 TB/s).
// kz: at most 8 (2, 4, 8, 16: 462, 407, 397, 393 us at 256^3; 44, 41, 41, 44 at 128^3) and
// such that four workgroups are left for each CU.
template <bool CONV>
__global__ void __launch_bounds__(TX * TY)
k_rhs_build(const double* __restrict__ u, const double* __restrict__ f, double* __restrict__ g,
            Grid3 G, double rho_dt, double rho, double inv_h, int kz, double* __restrict__ upk, int g_packed) {
    const uint3 bid = xcd_rows();
    const int n = G.n, i = bid.x * TX + threadIdx.x, j = bid.y * TY + threadIdx.y, k0 = bid.z * kz;
    if (i >= n || j >= n) return;
    const int64_t n2 = (int64_t)n * n, n3 = G.n3, half3 = n3 >> 1;
    const int k1 = k0 + kz < n ? k0 + kz : n;
    const double *X = u, *Y = u + n3, *Z = u + 2 * n3;
    const int ip = i + 1 < n ? i + 1 : 0, im = i > 0 ? i - 1 : n - 1;
    const int rj = n * j, rp = j + 1 < n ? rj + n : 0, rm = j > 0 ? rj - n : n * (n - 1);
    // (byte offsets in a plane: its base stays in scalar registers)
    const uint32_t c0 = 8 * (rj + i), cxp = 8 * (rj + ip), cxm = 8 * (rj + im), cyp = 8 * (rp + i), cym = 8 * (rm + i);
    const uint32_t cd = 8 * (rm + ip), ce = 8 * (rp + im);
    // the column's cell on planes k-1 and k; Z's -x and -y neighbours on k, X's +x
    // and Y's +y ones on k-1
    double xm = 0.0, ym = 0.0, zm = 0.0, zxm = 0.0, zym = 0.0, xxl = 0.0, yyl = 0.0;
    const int64_t P0 = n2 * k0;
    if (CONV) {
        const int64_t M = n2 * (k0 > 0 ? k0 - 1 : n - 1);
        xm = at_byte(X + M, c0);
        ym = at_byte(Y + M, c0);
        zm = at_byte(Z + M, c0);
        xxl = at_byte(X + M, cxp);
        yyl = at_byte(Y + M, cyp);
        zxm = at_byte(Z + P0, cxm);
        zym = at_byte(Z + P0, cym);
    }
    double x0 = at_byte(X + P0, c0), y0 = at_byte(Y + P0, c0), z0 = at_byte(Z + P0, c0);
    // what cell k reads of its own: the in-plane neighbours and those on k+1
    struct Reads {
        double xp, yp, zp, xxp, xxm, xyp, xym, xd, yxp, yxm, yyp, yym, yd, zxp, zyp, zxn, zyn, fx, fy, fz;
    };
    const auto read = [&](Reads& r, int k) {
        const int64_t P = n2 * k, N = k + 1 < n ? P + n2 : 0;
        if (CONV || k + 1 < k1) {
            r.xp = at_byte(X + N, c0);
            r.yp = at_byte(Y + N, c0);
            r.zp = at_byte(Z + N, c0);
        }
        if (CONV) {
            r.xxp = at_byte(X + P, cxp), r.xxm = at_byte(X + P, cxm), r.xyp = at_byte(X + P, cyp), r.xym = at_byte(X + P, cym), r.xd = at_byte(X + P, cd);
            r.yxp = at_byte(Y + P, cxp), r.yxm = at_byte(Y + P, cxm), r.yyp = at_byte(Y + P, cyp), r.yym = at_byte(Y + P, cym), r.yd = at_byte(Y + P, ce);
            r.zxp = at_byte(Z + P, cxp), r.zyp = at_byte(Z + P, cyp), r.zxn = at_byte(Z + N, cxm), r.zyn = at_byte(Z + N, cym);
        }
        if (f) {
            r.fx = at_byte(f + P, c0);
            r.fy = at_byte(f + n3 + P, c0);
            r.fz = at_byte(f + 2 * n3 + P, c0);
        }
    };
    const int64_t po = (i >> 1) + (n >> 1) * j;
    const auto write = [&](const Reads& r, int k) {
        double cx = 0.0, cy = 0.0, cz = 0.0;
        if (CONV) {
            cx = normal_flux(r.xxm, x0, r.xxp) * inv_h;
            cx += (edge_flux(x0, r.xyp, r.yd, r.yyp) - edge_flux(r.xym, x0, r.yxm, y0)) * inv_h;
            cx += (edge_flux(x0, r.xp, r.zxn, r.zp) - edge_flux(xm, x0, zxm, z0)) * inv_h;
            cy = normal_flux(r.yym, y0, r.yyp) * inv_h;
            cy += (edge_flux(y0, r.yxp, r.xd, r.xxp) - edge_flux(r.yxm, y0, r.xym, x0)) * inv_h;
            cy += (edge_flux(y0, r.yp, r.zyn, r.zp) - edge_flux(ym, y0, zym, z0)) * inv_h;
            cz = normal_flux(zm, z0, r.zp) * inv_h;
            cz += (edge_flux(z0, r.zxp, xxl, r.xxp) - edge_flux(zxm, z0, xm, x0)) * inv_h;
            cz += (edge_flux(z0, r.zyp, yyl, r.yyp) - edge_flux(zym, z0, ym, y0)) * inv_h;
            zxm = r.zxn;
            zym = r.zyn;
            xxl = r.xxp;
            yyl = r.yyp;
        }
        double gx = rho_dt * x0 - rho * cx, gy = rho_dt * y0 - rho * cy, gz = rho_dt * z0 - rho * cz;
        if (f) {
            gx += r.fx;
            gy += r.fy;
            gz += r.fz;
        }
        const int64_t P = n2 * k, Q = P >> 1;
        const int64_t o = Q + po + ((i + j + k) & 1 ? half3 : 0), og = g_packed ? o : P + rj + i;
        g[og] = gx;
        g[n3 + og] = gy;
        g[2 * n3 + og] = gz;
        if (upk) {
            upk[o] = x0;
            upk[n3 + o] = y0;
            upk[2 * n3 + o] = z0;
        }
        xm = x0;
        ym = y0;
        zm = z0;
        x0 = r.xp;
        y0 = r.yp;
        z0 = r.zp;
    };
    Reads ra, rb;
    int k = k0;
    read(ra, k);
    for (; k + 2 < k1; k += 2) {
        read(rb, k + 1);
        write(ra, k);
        read(ra, k + 2);
        write(rb, k + 1);
    }
    if (k + 1 < k1) {
        read(rb, k + 1);
        write(ra, k);
        write(rb, k + 1);
    } else {
        write(ra, k);
    }
}

// b = -(rho/dt) D u, D u = sum_d (u^d[c+e_d] - u^d[c]) / h
__global__ void __launch_bounds__(TX * TY)
k_divergence_rhs(const double* __restrict__ u, double* __restrict__ b, Grid3 G, double rho_dt,
                 double inv_h) {
    const int i = blockIdx.x * TX + threadIdx.x, j = blockIdx.y * TY + threadIdx.y, k = blockIdx.z;
    if (i >= G.n || j >= G.n) return;
    const int n = G.n;
    const int64_t c = G.at(i, j, k);
    double s = (u[G.at(wrap_idx(i + 1, n), j, k)] - u[c]) * inv_h;
    s += (u[G.n3 + G.at(i, wrap_idx(j + 1, n), k)] - u[G.n3 + c]) * inv_h;
    s += (u[2 * G.n3 + G.at(i, j, wrap_idx(k + 1, n))] - u[2 * G.n3 + c]) * inv_h;
    b[c] = -rho_dt * s;
}

// u^d -= (dt/rho) (p[c] - p[c - e_d]) / h
__global__ void __launch_bounds__(TX * TY)
k_project(double* __restrict__ u, const double* __restrict__ p, Grid3 G, double dt_rho,
          double inv_h) {
    const int i = blockIdx.x * TX + threadIdx.x, j = blockIdx.y * TY + threadIdx.y, k = blockIdx.z;
    if (i >= G.n || j >= G.n) return;
    const int n = G.n;
    const int64_t c = G.at(i, j, k);
    const double pc = p[c];
    const double gx = (pc - p[G.at(wrap_idx(i - 1, n), j, k)]) * inv_h;
    const double gy = (pc - p[G.at(i, wrap_idx(j - 1, n), k)]) * inv_h;
    const double gz = (pc - p[G.at(i, j, wrap_idx(k - 1, n))]) * inv_h;
    u[c] = u[c] - dt_rho * gx;
    u[G.n3 + c] = u[G.n3 + c] - dt_rho * gy;
    u[2 * G.n3 + c] = u[2 * G.n3 + c] - dt_rho * gz;
}

__global__ void k_zero(double* __restrict__ p, int64_t count) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count;
         t += (int64_t)gridDim.x * blockDim.x)
        p[t] = 0.0;
}

dim3 plane_grid(int n) { return dim3((n + TX - 1) / TX, (n + TY - 1) / TY, n); }

}  // namespace

hipib_status launch_rhs_build_coef(hipib_ctx* ctx, const double* u, const double* f, double* g,
                                   double rho_dt, double rho_conv, double* upk, bool g_packed) {
    Grid3 G{ctx->n, ctx->n3};
    const double bytes = (f ? 72.0 : 48.0) + (upk ? 24.0 : 0.0);
    const int n = ctx->n, tiles = ((n + TX - 1) / TX) * ((n + TY - 1) / TY);
    const int kz = std::max(1, std::min(kColumn, tiles * n / kColumnBlocks));
    return launch_k(ctx, HIPIB_TIMER_RHS, bytes * (double)ctx->n3,
                    ctx->cfg.convection ? k_rhs_build<true> : k_rhs_build<false>,
                    dim3((n + TX - 1) / TX, (n + TY - 1) / TY, (n + kz - 1) / kz), dim3(TX, TY), 0, u, f, g, G, rho_dt,
                    rho_conv, 1.0 / ctx->h, kz, upk, g_packed ? 1 : 0);
}

hipib_status launch_rhs_build(hipib_ctx* ctx, const double* u, const double* f, double* g, double* upk,
                              bool g_packed) {
    return launch_rhs_build_coef(ctx, u, f, g, ctx->cfg.rho / ctx->cfg.dt, ctx->cfg.rho, upk, g_packed);
}

hipib_status launch_divergence_rhs_coef(hipib_ctx* ctx, const double* u, double* b, double coef) {
    Grid3 G{ctx->n, ctx->n3};
    return launch_k(ctx, HIPIB_TIMER_DIVERGENCE, 32.0 * (double)ctx->n3, k_divergence_rhs, plane_grid(ctx->n),
                    dim3(TX, TY), 0, u, b, G, coef, 1.0 / ctx->h);
}

hipib_status launch_divergence_rhs(hipib_ctx* ctx, const double* u, double* b) {
    return launch_divergence_rhs_coef(ctx, u, b, ctx->cfg.rho / ctx->cfg.dt);
}

hipib_status launch_project_coef(hipib_ctx* ctx, double* u, const double* p, double coef) {
    Grid3 G{ctx->n, ctx->n3};
    return launch_k(ctx, HIPIB_TIMER_PROJECT, 56.0 * (double)ctx->n3, k_project, plane_grid(ctx->n), dim3(TX, TY), 0,
                    u, p, G, coef, 1.0 / ctx->h);
}

hipib_status launch_project(hipib_ctx* ctx, double* u, const double* p) {
    return launch_project_coef(ctx, u, p, ctx->cfg.dt / ctx->cfg.rho);
}

hipib_status launch_zero(hipib_ctx* ctx, double* p, int64_t count) {
    if (count <= 0) return HIPIB_OK;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    k_zero<<<(unsigned)blocks, 256, 0, ctx->stream>>>(p, count);
    HIPIB_HIP(hipGetLastError());
    return HIPIB_OK;
}

}  // namespace hipib
