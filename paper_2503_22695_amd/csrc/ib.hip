// Eulerian-Lagrangian coupling ("Eulerian-Lagrangian coupling operators"):
//   spreading      f^d[idx] += sum_q F^d_q delta_h(x^d_idx - X_q)
//   interpolation  U^d_q = sum_idx u^d[idx] delta_h(x^d_idx - X_q) h^3
// with Peskin's four-point kernel delta_h(x) = prod_e phi(x_e / h) / h^3.
// For a lattice coordinate r = X_e / h - offset (offset 0 along the face
// direction d, 1/2 along the others), the support is b-1 .. b+2 with
// b = floor(r), f = r - b, s = sqrt(1 + 4 f (1 - f)) and weights
//   ((3 - 2f - s), (3 - 2f + s), (1 + 2f + s), (1 + 2f - s)) / 8,
// which is phi evaluated at f+1, f, 1-f, 2-f.
//
// Spreading is binned: nodes are counting-sorted by the Eulerian tile (T^3
// cells) holding floor(X/h); every stencil point of a node in tile t lies in
// the (T+4)^3 box starting two cells below the tile, on all three lattices.
// One workgroup per work item (at most kSpreadChunk nodes of one tile) and
// lattice accumulates its box in LDS with FP64 LDS atomics, then adds the box
// to the grid with one coalesced pass of global atomics (boxes of
// neighbouring tiles overlap by four cells).  Interpolation
// walks the nodes in the same tile order so a wavefront gathers from a small
// neighbourhood.  Summation order is not fixed, so results agree with a serial
// sum to rounding.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "delta.h"

namespace hipib {
namespace {

// Work items share at most so many workgroups (a grid stride): the list's length is
// not known to the host, and a grid of its capacity is mostly workgroups without an
// item.  An empirical cap that matters little: with 8192, 2048 and 768, spreading
// takes 33.9, 34.5 and 36.5 us at 128^3 and 89.7, 90.0 and 90.9 at 192^3,
// interpolation 25.6 and 40.1 to 40.8 in all three.
constexpr int64_t kTileBlocks = 2048;

// ---------------------------------------------------------------------------
// Workspace of hipib_spread_noalloc: the node bins live in one static device
// array instead of memory the library allocates.  Limits: grids of at most
// kNaMaxN cells per side (8^3-cell tiles: at most (kNaMaxN/8)^3 tiles; the
// one smaller valid size that is not a multiple of 8, n = 12, has 27 tiles of
// 4^3) and at most kNaMaxNodes nodes.  Layout in int32 words: tile counts
// [ntiles], offsets [ntiles + 1], work list [2 * cap], list length [1], node
// tiles [nn], node ranks [nn], node order [nn].
// ---------------------------------------------------------------------------
constexpr int kNaMaxN = 256;
constexpr int kNaMaxNodes = 1 << 20;
constexpr int64_t kNaMaxTiles = (int64_t)(kNaMaxN / 8) * (kNaMaxN / 8) * (kNaMaxN / 8);
constexpr int64_t kNaMaxList = kNaMaxTiles + (kNaMaxNodes + kSpreadChunk - 1) / kSpreadChunk + 1;
constexpr int64_t kNaWords = kNaMaxTiles + (kNaMaxTiles + 1) + 2 * kNaMaxList + 1 + 3 * (int64_t)kNaMaxNodes;

static __device__ __align__(256) int32_t scratch[kNaWords];

__global__ void __launch_bounds__(256) k_zero_i32(int32_t* __restrict__ p, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}


// tile of each node and its rank inside the tile.  Consecutive nodes of a
// mesh mostly share a tile, so the lanes of a wavefront with equal tiles are
// grouped and one lane adds the group's size to the count (one atomic per
// distinct tile per wavefront instead of one per node, all of them at once: 7.8 us
// for 126000 nodes; waiting for each before the next group, 9.2).
__global__ void k_clear_flag(int32_t* flag) {
    if (threadIdx.x == 0) *flag = 0;
}

// A non-finite position, or one 1e9 cells or more from the origin, sets
// `bad` (when given) and is binned (and later spread and interpolated) at the
// origin, so every index stays in range; the entry points then fail with
// HIPIB_E_NUMERIC.
__global__ void __launch_bounds__(256)
k_bin_count(const double* __restrict__ X, int nn, int n, int T, int ta, double inv_h,
            int32_t* __restrict__ node_tile, int32_t* __restrict__ node_rank,
            int32_t* __restrict__ count, int32_t* __restrict__ bad) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = q < nn;
    int tile = -1;
    if (valid) {
        int t[3];
        for (int e = 0; e < 3; ++e) {
            const double r = X[3 * q + e] * inv_h;
            if (bad && !(fabs(r) < 1.0e9)) *bad = 1;
            const int c = (int)floor(safe_coord(r));
            t[e] = wrap_mod(c, n) / T;
        }
        tile = t[0] + ta * (t[1] + ta * t[2]);
        node_tile[q] = tile;
    }
    const int lane = (int)__lane_id();
    unsigned long long pending = __ballot(valid);
    int first = lane, rank = 0, size = 0;
    while (pending) {  // uniform over the wavefront
        const int leader = __ffsll((long long)pending) - 1;
        const bool mine = valid && tile == __shfl(tile, leader, 64);
        const unsigned long long m = __ballot(mine);
        if (mine) {
            first = leader;
            rank = __popcll(m & ((1ull << lane) - 1ull));
            size = __popcll(m);
        }
        pending &= ~m;
    }
    int base = 0;
    if (valid && lane == first) base = atomicAdd(count + tile, size);
    rank += __shfl(base, first, 64);
    if (valid) node_rank[q] = rank;
}

// Exclusive scan of the tile counts and the list of work items: each
// occupied tile is cut into chunks of at most kSpreadChunk nodes, listed as
// (tile, first rank) pairs, so a tile crowded with nodes is spread by several
// workgroups.  Counts are reset to 0 for the next binning.  When given,
// lfirst[t] receives the list index of tile t's first work item.
// One workgroup in rounds of 4096 tiles, four to a thread, the next round's counts
// read ahead.  (Each thread a contiguous share of all tiles, one count at a time:
// a chain of reads, 8.2 us for 16^3 tiles and 57 for 24^3 in place of 5.8 and 31.)
__global__ void __launch_bounds__(1024)
k_bin_scan(int32_t* __restrict__ count, int64_t ntiles, int32_t* __restrict__ off,
           int32_t* __restrict__ list, int32_t* __restrict__ nlist, int32_t* __restrict__ lfirst) {
    __shared__ int32_t wsum[2][2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto read = [&](int64_t i, int32_t* c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = i + r < ntiles ? count[i + r] : 0;
    };
    int32_t c[4], run0 = 0, list0 = 0;   // (totals of the rounds before)
    read(4 * tid, c);
    for (int64_t base = 0, round = 0; base < ntiles; base += 4096, ++round) {
        const int64_t i0 = base + 4 * tid;
        int32_t next[4] = {0, 0, 0, 0}, chunks[4];
        if (base + 4096 < ntiles) read(i0 + 4096, next);
#pragma unroll
        for (int r = 0; r < 4; ++r) chunks[r] = (c[r] + kSpreadChunk - 1) / kSpreadChunk;
        const int32_t sum = c[0] + c[1] + c[2] + c[3], nz = chunks[0] + chunks[1] + chunks[2] + chunks[3];
        int32_t a = sum, b = nz;         // inclusive over the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t pa = __shfl_up(a, o, 64), pb = __shfl_up(b, o, 64);
            if (lane >= o) {
                a += pa;
                b += pb;
            }
        }
        int32_t (*const ws)[16] = wsum[round & 1];
        if (lane == 63) {
            ws[0][wave] = a;
            ws[1][wave] = b;
        }
        __syncthreads();
        int32_t run = run0 + a - sum, lrun = list0 + b - nz;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int32_t ta = ws[0][w], tb = ws[1][w];
            if (w < wave) {
                run += ta;
                lrun += tb;
            }
            run0 += ta;
            list0 += tb;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = i0 + r;
            if (i < ntiles) {
                off[i] = run;
                if (lfirst) lfirst[i] = lrun;
                count[i] = 0;
                for (int32_t q = 0; q < c[r]; q += kSpreadChunk) {
                    list[2 * lrun] = (int32_t)i;
                    list[2 * lrun + 1] = q;
                    ++lrun;
                }
                run += c[r];
            }
            c[r] = next[r];
        }
    }
    if (tid == 0) {
        off[ntiles] = run0;
        *nlist = list0;
    }
}

__global__ void __launch_bounds__(256)
k_bin_scatter(const int32_t* __restrict__ node_tile, const int32_t* __restrict__ node_rank,
              const int32_t* __restrict__ off, int32_t* __restrict__ perm, int nn) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nn) return;
    perm[off[node_tile[q]] + node_rank[q]] = q;
}

// one workgroup per (work item, lattice d = blockIdx.y) (grid-stride over the
// list): up to kSpreadChunk nodes of one tile, one node per thread; LDS box of
// E^3 cells of lattice d, E = T + 4, starting at T * tile - 2 (a workgroup per
// lattice: a third of the LDS atomics per thread and three times the
// workgroups of a single box of all three lattices).  Ranks inside the chunk
// are dealt to threads with an odd stride, so the lanes of a wavefront take
// nodes that are far apart in mesh order, which keeps apart the LDS addresses
// they add to in the same instruction.  (Four threads to a node, a plane each: more
// of an instruction's additions collide, 35 -> 48 us at 128^3.)  TW: type of the
// weights and their products (the lattice coordinate, its floor and the
// fractional offset are always FP64); the LDS box and the grid accumulate in
// FP64, since neighbouring nodes' forces partly cancel there.
template <int T, typename TW>
__global__ void __launch_bounds__(kSpreadChunk)
k_spread_tiles(const double* __restrict__ X, const double* __restrict__ F, double* __restrict__ f,
               const int32_t* __restrict__ perm, const int32_t* __restrict__ off,
               const int32_t* __restrict__ list, const int32_t* __restrict__ nlist, int n, int ta,
               int64_t n3, double inv_h, double ih3, int f_packed) {
    constexpr int E = T + 4, E3 = E * E * E;
    __shared__ double box[E3];
    const int d = blockIdx.y;
    const int ntl = *nlist;
    for (int li = blockIdx.x; li < ntl; li += gridDim.x) {
        const int tile = list[2 * li];
        const int tb[3] = {T * (tile % ta), T * ((tile / ta) % ta), T * (tile / (ta * ta))};
        for (int e = threadIdx.x; e < E3; e += blockDim.x) box[e] = 0.0;
        __syncthreads();
        const int idx = off[tile] + list[2 * li + 1] + ((threadIdx.x * 109) & (kSpreadChunk - 1));
        if (idx < off[tile + 1]) {
            const int q = perm[idx];
            double xs[3];
            int cw[3];
            for (int e = 0; e < 3; ++e) {
                xs[e] = safe_coord(X[3 * q + e] * inv_h);
                cw[e] = wrap_mod((int)floor(xs[e]), n);
            }
            {
                const TW val = (TW)(F[3 * q + d] * ih3);
                int ls[3];
                TW w[3][4];
                for (int e = 0; e < 3; ++e) {
                    const double r = xs[e] - (e == d ? 0.0 : 0.5);
                    const double bf = floor(r);
                    const TW fr = (TW)(r - bf);
                    const TW sq = sqrt(TW(1) + TW(4) * fr * (TW(1) - fr));
                    w[e][0] = (TW(3) - TW(2) * fr - sq) * TW(0.125);
                    w[e][1] = (TW(3) - TW(2) * fr + sq) * TW(0.125);
                    w[e][2] = (TW(1) + TW(2) * fr + sq) * TW(0.125);
                    w[e][3] = (TW(1) + TW(2) * fr - sq) * TW(0.125);
                    // stencil start relative to the node's cell is -1 or -2
                    const int ds = (int)bf - 1 - (int)floor(xs[e]);
                    ls[e] = cw[e] - tb[e] + 2 + ds;
                }
                double* bd = box;
                for (int c = 0; c < 4; ++c)
                    for (int b = 0; b < 4; ++b) {
                        const TW wyz = w[1][b] * w[2][c];
                        const int row = (ls[0]) + E * ((ls[1] + b) + E * (ls[2] + c));
                        for (int a = 0; a < 4; ++a) atomicAdd(bd + row + a, (double)(val * (w[0][a] * wyz)));
                    }
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < E3; e += blockDim.x) {
            const double v = box[e];
            if (v != 0.0) {
                const int r = e;
                const int lx = r % E, ly = (r / E) % E, lz = r / (E * E);
                const int gx = wrap_idx(tb[0] - 2 + lx, n), gy = wrap_idx(tb[1] - 2 + ly, n),
                          gz = wrap_idx(tb[2] - 2 + lz, n);   // (within two cells of the grid)
                const int64_t g = f_packed ? pk(gx, gy, gz, n) : gx + (int64_t)n * (gy + (int64_t)n * gz);
                atomicAdd(f + d * n3 + g, v);
            }
        }
        __syncthreads();
    }
}

// Interpolation U = J(X) u, optionally X += dt U (in place, FP64), by the
// binning's work items: one workgroup per item (grid-stride over the list),
// up to kSpreadChunk nodes of one tile, one node per thread.  The E^3 box of
// each velocity component around the tile (E = T + 4, from T * tile - 2, the
// reach of every node's 4x4x4 stencils on all three staggered lattices) is
// staged in LDS with coalesced row loads, so the stencil values a tile's nodes
// share are fetched from L2 once, all of a thread's reads in flight (three components
// of a cell to a thread); each node's 3 x 64-term sums then read LDS.  At most 64
// nodes: four threads to a node, one plane of its stencils each, so that the sums of
// a sparse item are a quarter as long (216 elements at 32^3: 14.6 -> 6.7 us, 126000
// nodes at 128^3 30.6 -> 26.0, 281000 at 192^3 53.6 -> 40.7; four threads for every item
// 31.4 at 128^3).  In FP64 a node's sum has one order wherever it lands: each plane
// in the order of a direct gather, then (0 + 1) + (2 + 3), by one thread or by four.
// Which nodes share an item depends on the order of the binning's atomics.  In FP32
// one thread sums in the order of a direct gather, which FP32 results depend on.
// TW: type of the box, the weights and the accumulation.
template <int T, typename TW>
__global__ void __launch_bounds__(kSpreadChunk)
k_interp_tiles(const double* X, const double* __restrict__ u, double* __restrict__ U, double* Xupd, double dt,
               const int32_t* __restrict__ perm, const int32_t* __restrict__ off,
               const int32_t* __restrict__ list, const int32_t* __restrict__ nlist, int n, int ta,
               int64_t n3, double inv_h) {
    constexpr int E = T + 4, E3 = E * E * E;
    __shared__ TW box[3 * E3];
    const int ntl = *nlist;
    for (int li = blockIdx.x; li < ntl; li += gridDim.x) {
        const int tile = list[2 * li];
        const int tb[3] = {T * (tile % ta), T * ((tile / ta) % ta), T * (tile / (ta * ta))};
        const int first = off[tile] + list[2 * li + 1], cnt = min(off[tile + 1] - first, kSpreadChunk);
        // the box's cells, the three components of a cell by the same thread
        constexpr int R = (E3 + kSpreadChunk - 1) / kSpreadChunk;
        TW v[R][3];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = min((int)threadIdx.x + r * kSpreadChunk, E3 - 1);
            const int lx = e % E, ly = (e / E) % E, lz = e / (E * E);
            const int gx = wrap_idx(tb[0] - 2 + lx, n), gy = wrap_idx(tb[1] - 2 + ly, n),
                      gz = wrap_idx(tb[2] - 2 + lz, n);   // (within two cells of the grid)
            const int64_t g = gx + (int64_t)n * (gy + (int64_t)n * gz);
#pragma unroll
            for (int d = 0; d < 3; ++d) v[r][d] = (TW)u[d * n3 + g];
        }
        __syncthreads();   // the previous item's reads of the box are done
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = threadIdx.x + r * kSpreadChunk;
            if (e < E3)
#pragma unroll
                for (int d = 0; d < 3; ++d) box[d * E3 + e] = v[r][d];
        }
        __syncthreads();
        constexpr bool planes = sizeof(TW) == 8;
        const auto nodes = [&](auto lanes) {
            constexpr int L = decltype(lanes)::value;
            for (int i = threadIdx.x / L; i < cnt; i += kSpreadChunk / L) {
                const int q = perm[first + i], c0 = threadIdx.x % L;
                const double X0 = X[3 * q], X1 = X[3 * q + 1], X2 = X[3 * q + 2];
                const double xs[3] = {safe_coord(X0 * inv_h), safe_coord(X1 * inv_h), safe_coord(X2 * inv_h)};
                int cw[3];
                for (int e = 0; e < 3; ++e) cw[e] = wrap_mod((int)floor(xs[e]), n);
                TW Uq[3];
                for (int d = 0; d < 3; ++d) {
                    int ls[3];
                    TW w[3][4];
                    for (int e = 0; e < 3; ++e) {
                        const double r = xs[e] - (e == d ? 0.0 : 0.5);
                        const double bf = floor(r);
                        const TW fr = (TW)(r - bf);
                        const TW sq = sqrt(TW(1) + TW(4) * fr * (TW(1) - fr));
                        w[e][0] = (TW(3) - TW(2) * fr - sq) * TW(0.125);
                        w[e][1] = (TW(3) - TW(2) * fr + sq) * TW(0.125);
                        w[e][2] = (TW(1) + TW(2) * fr + sq) * TW(0.125);
                        w[e][3] = (TW(1) + TW(2) * fr - sq) * TW(0.125);
                        // stencil start relative to the node's cell is -1 or -2
                        const int ds = (int)bf - 1 - (int)floor(xs[e]);
                        ls[e] = cw[e] - tb[e] + 2 + ds;
                    }
                    const TW* bd = box + d * E3;
                    TW acc = TW(0), plane[4 / L];
    #pragma unroll
                    for (int t = 0; t < 4 / L; ++t) {
                        if (planes) acc = TW(0);
                        const int c = L == 1 ? t : c0;
                        const TW wz = L == 1 ? w[2][t] : c == 0 ? w[2][0] : c == 1 ? w[2][1] : c == 2 ? w[2][2] : w[2][3];
                        for (int b = 0; b < 4; ++b) {
                            const TW wyz = w[1][b] * wz;
                            const int row = ls[0] + E * ((ls[1] + b) + E * (ls[2] + c));
                            for (int a = 0; a < 4; ++a) acc += bd[row + a] * (w[0][a] * wyz);
                        }
                        plane[t] = acc;
                    }
                    if constexpr (L == 1 && planes) acc = (plane[0] + plane[1]) + (plane[2] + plane[3]);
                    for (int o = 1; o < L; o <<= 1) acc += __shfl_xor(acc, o, 64);   // (a node's lanes stay together)
                    Uq[d] = acc;
                }
                if (c0 != 0) continue;
                if (U) {
                    U[3 * q] = (double)Uq[0];
                    U[3 * q + 1] = (double)Uq[1];
                    U[3 * q + 2] = (double)Uq[2];
                }
                if (Xupd) {
                    Xupd[3 * q] = X0 + dt * (double)Uq[0];
                    Xupd[3 * q + 1] = X1 + dt * (double)Uq[1];
                    Xupd[3 * q + 2] = X2 + dt * (double)Uq[2];
                }
            }
        };
        bool four = false;
        if constexpr (planes) {
            four = cnt <= kSpreadChunk / 4;
            if (four) nodes(std::integral_constant<int, 4>{});
        }
        if (!four) nodes(std::integral_constant<int, 1>{});
    }
}

}  // namespace

hipib_status launch_bin(hipib_ctx* ctx, const double* X) {
    if (ctx->nn == 0) return HIPIB_OK;
    const int nb = (ctx->nn + 255) / 256;
    k_clear_flag<<<1, 64, 0, ctx->stream>>>(&ctx->st->bad_position);
    k_bin_count<<<nb, 256, 0, ctx->stream>>>(X, ctx->nn, ctx->n, ctx->tile, ctx->tiles_axis,
                                             1.0 / ctx->h, ctx->node_tile, ctx->node_rank,
                                             ctx->bin_count, &ctx->st->bad_position);
    k_bin_scan<<<1, 1024, 0, ctx->stream>>>(ctx->bin_count, ctx->ntiles, ctx->bin_off,
                                            ctx->tile_list, ctx->n_list, ctx->det_lfirst);
    k_bin_scatter<<<nb, 256, 0, ctx->stream>>>(ctx->node_tile, ctx->node_rank, ctx->bin_off,
                                               ctx->perm, ctx->nn);
    HIPIB_HIP(hipGetLastError());
    return HIPIB_OK;
}

// expects launch_bin(ctx, X) to have been enqueued for the same X
hipib_status launch_spread(hipib_ctx* ctx, const double* X, const double* F, double* f, bool f_packed) {
    if (ctx->nn == 0) return HIPIB_OK;
    if (ctx->cfg.deterministic) return det_spread(ctx, X, F, f, f_packed);
    const double h = ctx->h;
    const int64_t cap = spread_list_cap(ctx->ntiles, ctx->nn);
    const int blocks = (int)std::min(cap, kTileBlocks);
    const bool mixed = ctx->cfg.precision == HIPIB_MIXED;
#define HIPIB_SPREAD(TT, TW)                                                                       \
    HIPIB_TRY(launch_k(ctx, HIPIB_TIMER_SPREAD, 0.0, k_spread_tiles<TT, TW>, dim3(blocks, 3), dim3(kSpreadChunk), 0,  \
                       X, F, f, ctx->perm, ctx->bin_off, ctx->tile_list, ctx->n_list, ctx->n,                 \
                       ctx->tiles_axis, ctx->n3, 1.0 / h, 1.0 / (h * h * h), f_packed ? 1 : 0))
    if (ctx->tile == 8) {
        if (mixed) HIPIB_SPREAD(8, float); else HIPIB_SPREAD(8, double);
    } else {
        if (mixed) HIPIB_SPREAD(4, float); else HIPIB_SPREAD(4, double);
    }
#undef HIPIB_SPREAD
    HIPIB_HIP(hipGetLastError());
    return HIPIB_OK;
}

// expects launch_bin(ctx, X) to have been enqueued for the same X
hipib_status launch_interpolate(hipib_ctx* ctx, const double* X, const double* u, double* U,
                                double* Xupd, double dt) {
    if (ctx->nn == 0) return HIPIB_OK;
    const int64_t cap = spread_list_cap(ctx->ntiles, ctx->nn);
    const int blocks = (int)std::min(cap, kTileBlocks);
    const bool mixed = ctx->cfg.precision == HIPIB_MIXED;
#define HIPIB_INTERP(TT, TW)                                                                               \
    return launch_k(ctx, HIPIB_TIMER_INTERP, 0.0, k_interp_tiles<TT, TW>, dim3(blocks), dim3(kSpreadChunk), 0, X, \
                    u, U, Xupd, dt, ctx->perm, ctx->bin_off, ctx->tile_list, ctx->n_list, ctx->n,               \
                    ctx->tiles_axis, ctx->n3, 1.0 / ctx->h)
    if (ctx->tile == 8) {
        if (mixed) HIPIB_INTERP(8, float);
        HIPIB_INTERP(8, double);
    }
    if (mixed) HIPIB_INTERP(4, float);
    HIPIB_INTERP(4, double);
#undef HIPIB_INTERP
}

}  // namespace hipib

// ---------------------------------------------------------------------------
// hipib_spread_noalloc
// ---------------------------------------------------------------------------

namespace hipib {
namespace {

constexpr int kNaMaxDevices = 64;
std::mutex g_na_mutex;
int32_t* g_na_ptr[kNaMaxDevices] = {};   // device address of `scratch`, per device

// Device address of this device's copy of `scratch`, looked up on the first
// call on each device (with that device current).  Host code never passes the
// array's own name to a kernel: on the host it is only a stand-in.
hipib_status noalloc_scratch(int32_t** out) {
    hipib_ctx* ctx = nullptr;   // (no context to mark broken)
    int dev = 0;
    HIPIB_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNaMaxDevices) return fail(HIPIB_E_INVAL, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_na_mutex);
    if (!g_na_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return fail(HIPIB_E_HIP, "hipGetSymbolAddress(scratch) failed on device %d: HIP error %d",
                        dev, (int)e);
        }
        g_na_ptr[dev] = static_cast<int32_t*>(p);
    }
    *out = g_na_ptr[dev];
    return HIPIB_OK;
}

}  // namespace

}  // namespace hipib

using namespace hipib;

hipib_status hipib_spread_noalloc(int32_t n, int32_t n_nodes, const double* X, const double* F,
                                  double* f, void* stream) {
    hipib_ctx* ctx = nullptr;   // (no context to mark broken)
    if (n < 8 || n > kNaMaxN)
        return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: n = %d outside [8, %d]", n, kNaMaxN);
    {
        int m = n;
        while (m >= 8) {
            if (m % 2) return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: n = %d is not 4*2^k or 6*2^k", n);
            m /= 2;
        }
        if (m != 4 && m != 6)
            return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: n = %d is not 4*2^k or 6*2^k", n);
    }
    if (n_nodes < 0 || n_nodes > kNaMaxNodes)
        return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: n_nodes = %d outside [0, %d]", n_nodes,
                    kNaMaxNodes);
    if (f == nullptr || (reinterpret_cast<uintptr_t>(f) & 7u) ||
        (n_nodes > 0 && (X == nullptr || F == nullptr || (reinterpret_cast<uintptr_t>(X) & 7u) ||
                         (reinterpret_cast<uintptr_t>(F) & 7u))))
        return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: bad pointer");
    if (n_nodes == 0) return HIPIB_OK;
    int32_t* base = nullptr;
    HIPIB_TRY(noalloc_scratch(&base));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int T = (n % 8 == 0) ? 8 : 4;
    const int ta = n / T;
    const int64_t ntiles = (int64_t)ta * ta * ta;
    const int64_t cap = spread_list_cap(ntiles, n_nodes);
    int32_t* count = base;
    int32_t* off = count + ntiles;
    int32_t* list = off + ntiles + 1;
    int32_t* nlist = list + 2 * cap;
    int32_t* node_tile = nlist + 1;
    int32_t* node_rank = node_tile + n_nodes;
    int32_t* perm = node_rank + n_nodes;
    if (perm + n_nodes > base + kNaWords)
        return fail(HIPIB_E_INVAL, "hipib_spread_noalloc: workspace exceeds its %lld words",
                    (long long)kNaWords);
    const double h = 1.0 / n;
    const int nb = (n_nodes + 255) / 256;
    // the tile counts start at zero (a fill kernel, so the call can be captured in a graph)
    k_zero_i32<<<(unsigned)((ntiles + 255) / 256), 256, 0, st>>>(count, ntiles);
    k_bin_count<<<nb, 256, 0, st>>>(X, n_nodes, n, T, ta, 1.0 / h, node_tile, node_rank, count, nullptr);
    k_bin_scan<<<1, 1024, 0, st>>>(count, ntiles, off, list, nlist, nullptr);
    k_bin_scatter<<<nb, 256, 0, st>>>(node_tile, node_rank, off, perm, n_nodes);
    const int blocks = (int)std::min(cap, kTileBlocks);
    const int64_t n3 = (int64_t)n * n * n;
    if (T == 8)
        k_spread_tiles<8, double><<<dim3(blocks, 3), kSpreadChunk, 0, st>>>(X, F, f, perm, off, list, nlist, n, ta,
                                                                   n3, 1.0 / h, 1.0 / (h * h * h), 0);
    else
        k_spread_tiles<4, double><<<dim3(blocks, 3), kSpreadChunk, 0, st>>>(X, F, f, perm, off, list, nlist, n, ta,
                                                                   n3, 1.0 / h, 1.0 / (h * h * h), 0);
    HIPIB_HIP(hipGetLastError());
    return HIPIB_OK;
}
