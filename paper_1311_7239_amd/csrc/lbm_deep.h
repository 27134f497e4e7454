// The deep pass: many collide-and-stream cycles per launch for domains that
// leave most of the chip idle, where a pass costs its launch and its memory
// latency (about 4.5 us on 512 nodes and on 65,536) and not its arithmetic.
//
// A workgroup owns a tile of the domain, loads it with a ring of C nodes around
// it into LDS and runs C cycles there, each on a ring one node thinner than the
// one before; the last one stores the tile. No workgroup waits for another; the
// price is the ring's redundant collisions, which are cheap where the SIMDs
// would idle. An axis that one tile covers has no ring at
// all (walls close it, a periodic one wraps inside LDS), so a domain that fits
// one workgroup runs any number of cycles in one launch.
//
// Which thread computes which node is fixed for the whole pass: the nodes are
// numbered from the tile outwards, ring by ring, so the nodes of cycle c are a
// prefix of the numbering and whole wavefronts drop out as the ring shrinks. A
// node's eight LDS sources (with walls, wrap and on-node walls resolved), its
// drag coefficients and its offset are computed once, so a cycle is the eight
// LDS reads, the 99 vector instructions of the update and the eight writes. Two
// LDS buffers alternate (one barrier per cycle); their distance is a compile-time
// constant, which the LDS instructions take as their immediate offset.
//
// What bounds it: on one CU (40^2 cavity, 25 wavefronts of nodes) a cycle takes
// 1.15 to 1.3 us, vector issue alone 1.12; on 512 nodes 0.52 us, the latency of
// one update; tiled, about 4 us per launch for the launch, the load and the
// store, and 0.4 us or the issue time for each cycle, whichever is longer.
#pragma once

#include <algorithm>
#include <cmath>

#include "lbm_launch.h"

namespace mrt {

// One axis of a tile: its nodes [a, b), and how far the ring around it reaches
// (not past a wall, and nowhere on an axis that one tile covers).
struct DeepAxis {
    int a, b, lo, hi;
    __device__ DeepAxis(int k, int tiles, int n, bool periodic) {
        // tiles of nearly equal size: tile k of T spans [k n / T, (k + 1) n / T)
        // (products below 2^31: the host admits domains of that size only)
        a = k * n / tiles;
        b = (k + 1) * n / tiles;
        lo = tiles == 1 || !periodic ? 0 : -(1 << 30);
        hi = tiles == 1 || !periodic ? n : 1 << 30;
    }
    // the nodes within g of the tile
    __device__ int first(int g) const { return a - g < lo ? lo : a - g; }
    __device__ int last(int g) const { return b + g > hi ? hi : b + g; }
};

// s / w for s below 2^20 (inv = 1 / w)
__device__ __forceinline__ int small_div(int s, float inv) { return (int)(((float)s + 0.5f) * inv); }

// Node number s of a tile and its ring (0: the tile itself): the tile row by
// row, then ring after ring: the row above, the row below, the left and right
// columns; a side at a wall has none. Only the first `rings` rings are numbered.
__device__ __forceinline__ int deep_node(const DeepAxis &X, const DeepAxis &Y, int rings, int s, int &x, int &y) {
    int g = 0;
    for (int j = 0; j < rings; ++j) g += s >= (X.last(j) - X.first(j)) * (Y.last(j) - Y.first(j)) ? 1 : 0;
    const int gi = g > 0 ? g - 1 : 0;
    const int ix0 = X.first(gi), ix1 = X.last(gi), iy0 = Y.first(gi), iy1 = Y.last(gi);
    if (g == 0) {
        const int w = ix1 - ix0, r = small_div(s, 1.0f / (float)w);
        x = ix0 + s - r * w;
        y = iy0 + r;
        return 0;
    }
    const int ox0 = X.first(g), oy0 = Y.first(g), w = X.last(g) - ox0, h = iy1 - iy0;
    int q = s - (ix1 - ix0) * h;
    const bool above = oy0 < iy0, left = ox0 < ix0;
    const int rows = w * ((above ? 1 : 0) + (Y.last(g) > iy1 ? 1 : 0));
    if (q < rows) {
        x = ox0 + (q >= w ? q - w : q);
        y = above && q < w ? oy0 : iy1;
    } else {
        q -= rows;
        x = left && q < h ? ox0 : ix1;
        y = iy0 + (q >= h ? q - h : q);
    }
    return g;
}

// A workgroup's tile with its ring as it lies in LDS: the nodes that cycle 0
// reads, row by row.
struct DeepFrame {
    DeepAxis X, Y;
    int x0, y0, w, n, s;   // s: row stride in LDS
    bool per_x, per_y, wrap_x, wrap_y;   // wrap: a periodic axis that one tile covers
    int nx, ny;
    __device__ DeepFrame(const Dom &d, const DeepPlan &p, int C)
        : X((int)blockIdx.x % p.tiles_x, p.tiles_x, d.nx, d.bc_x == BC_PERIODIC),
          Y((int)blockIdx.x / p.tiles_x, p.tiles_y, d.ny, d.bc_y == BC_PERIODIC) {
        x0 = X.first(C);
        y0 = Y.first(C);
        w = X.last(C) - x0;
        n = w * (Y.last(C) - y0);
        s = p.stride;
        per_x = d.bc_x == BC_PERIODIC;
        per_y = d.bc_y == BC_PERIODIC;
        wrap_x = p.tiles_x == 1 && per_x;
        wrap_y = p.tiles_y == 1 && per_y;
        nx = d.nx;
        ny = d.ny;
    }
    __device__ static int wrapped(int v, int m) { return v < 0 ? v + m : (v >= m ? v - m : v); }
    // node offset in a plane, and LDS position, of the frame's k-th node
    __device__ uint32_t offset(int k, float inv, int pitch, int &at) const {
        const int row = small_div(k, inv), col = k - row * w;
        at = row * s + col;
        return (uint32_t)(wrapped(y0 + row, ny) * pitch + wrapped(x0 + col, nx));
    }
};

// LDS columns and row offsets of a node (bx, by), at column cx and row cy of the
// frame, and of the nodes beside it, and the walls next to it.
struct DeepLinks {
    int cx, colm, colp, row0, rowm, rowp;
    bool outl, outr, outb, outt;
    __device__ DeepLinks(const DeepFrame &F, int bx, int by, int cx_, int cy) {
        const bool xl = bx == 0, xr = bx == F.nx - 1, yl = by == 0, yr = by == F.ny - 1;
        cx = cx_;
        colm = xl && F.wrap_x ? F.nx - 1 : cx - 1;
        colp = xr && F.wrap_x ? 0 : cx + 1;
        row0 = cy * F.s;
        rowm = (yl && F.wrap_y ? F.ny - 1 : cy - 1) * F.s;
        rowp = (yr && F.wrap_y ? 0 : cy + 1) * F.s;
        outl = xl && !F.per_x;
        outr = xr && !F.per_x;
        outb = yl && !F.per_y;
        outt = yr && !F.per_y;
    }
    // position (planes of `cap` floats) of what comes along (ex, ey): plane `plane`
    // of the node at -(ex, ey), or across a wall the own plane `oplane`
    __device__ int source(int ex, int ey, int plane, int oplane, int cap) const {
        const bool out = (ex > 0 && outl) || (ex < 0 && outr) || (ey > 0 && outb) || (ey < 0 && outt);
        const int at = (ey > 0 ? rowm : (ey < 0 ? rowp : row0)) + (ex > 0 ? colm : (ex < 0 ? colp : cx));
        return out ? oplane * cap + row0 + cx : plane * cap + at;
    }
};

// REC: every cycle also records its velocity for the adjoint (and the stress
// moments and the temperature), cycle k five planes after cycle k - 1.
template <typename S, int MK, bool THERMAL, bool NEE, bool REC, int CAP, int NT>
__global__ __launch_bounds__(NT) void k_step_deep(Dom d, DeepPlan p, int C, int direct) {
    constexpr int R = (CAP + NT - 1) / NT;
    constexpr int ES = (int)sizeof(S);
    __shared__ float lds[2 * 8 * CAP];
    __shared__ float ldsg[THERMAL ? 2 * 5 * CAP : 1];
    const DeepFrame F(d, p, C);
    const uint32_t fbytes = (uint32_t)(8 * d.plane * ES);
    const BufRes rin = buf_res(d.fin, fbytes), rout = buf_res(d.fout, fbytes);
    const uint32_t gbytes = THERMAL ? (uint32_t)(5 * d.plane * 4) : 0u;
    const BufRes rgin = buf_res(THERMAL ? d.gin : nullptr, gbytes), rgout = buf_res(THERMAL ? d.gout : nullptr, gbytes);
    const MediumSrc<MK> med(d);

    // the frame's populations into the first LDS buffer, row by row
    float *ldsB = lds + 8 * CAP, *ldsgB = ldsg + (THERMAL ? 5 * CAP : 0);
    {
        const float inv = 1.0f / (float)F.w;
        float f[R][8], g[R][THERMAL ? 5 : 1];
        int at[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int s = (int)threadIdx.x + r * NT;
            if (s >= F.n) continue;
            const uint32_t v = F.offset(s, inv, d.pitch, at[r]);
#pragma unroll
            for (int i = 0; i < 8; ++i) f[r][i] = BufIO<S>::ld(rin, v * ES, (uint32_t)(i * d.plane * ES));
            if (THERMAL) {
#pragma unroll
                for (int j = 0; j < 5; ++j) g[r][THERMAL ? j : 0] = BufIO<float>::ld(rgin, v * 4, (uint32_t)(j * d.plane * 4));
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int s = (int)threadIdx.x + r * NT;
            if (s >= F.n) continue;
#pragma unroll
            for (int i = 0; i < 8; ++i) lds[i * CAP + at[r]] = f[r][i];
            if (THERMAL) {
#pragma unroll
                for (int j = 0; j < 5; ++j) ldsg[j * CAP + at[r]] = g[r][THERMAL ? j : 0];
            }
        }
    }

    int ring[R];                         // the node's ring: it takes part while so many cycles follow
    int src[R][8], gsrc[R][5], own[R];   // LDS positions of the links' sources and of the node
    uint32_t kind[R];                    // two bits per D2Q5 link: 0 as it is, 2 hot, 3 cold anti-bounce-back
    uint32_t o[R];                       // node offset in a plane
    bool top[R], wall[R];                // next to the moving lid; on an on-node wall
    Cell c[R], cB[NEE ? R : 1];          // the node's cell, and its inner neighbour's
    int wx[NEE ? R : 1], wy[NEE ? R : 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int x, y;
        ring[r] = deep_node(F.X, F.Y, C, (int)threadIdx.x + r * NT, x, y);
        if (ring[r] >= C || x >= F.X.last(C) || y >= F.Y.last(C)) {
            ring[r] = C;   // no node left for this thread
            continue;
        }
        const int gx = F.wrapped(x, d.nx), gy = F.wrapped(y, d.ny);
        o[r] = (uint32_t)(gy * d.pitch + gx);
        own[r] = (y - F.y0) * F.s + (x - F.x0);
        c[r] = med.cell(d, med.load(o[r] * 4));
        // the node that the links are gathered for: on an on-node wall its inner neighbour
        int bx = gx, by = gy;
        wall[r] = false;
        if (NEE) {
            wall[r] = nee_wall(d, gx, gy, bx, by);
            cB[r] = med.cell(d, med.load((uint32_t)(by * d.pitch + bx) * 4));
            wx[r] = gx;
            wy[r] = gy;
        }
        const DeepLinks at(F, bx, by, x + (bx - gx) - F.x0, y + (by - gy) - F.y0);
        top[r] = at.outt;
#pragma unroll
        for (int i = 0; i < 8; ++i) src[r][i] = at.source(EX[i], EY[i], i, OPP[i], CAP);
        if (THERMAL) {
#pragma unroll
            for (int j = 0; j < 5; ++j) gsrc[r][j] = at.source(TXv[j], TYv[j], j, TOPP[j], CAP);
            kind[r] = (at.outl ? 2u << 2 : 0u) | (at.outr ? 3u << 6 : 0u);   // links 1 and 3
        }
    }

    // cycle k from one LDS buffer into the other, or, the last one, to HBM
    auto cycle = [&](int k, const float *from, const float *fromg, float *to, float *tog) {
        lds_barrier();
        const bool as_is = k == 0 && direct;   // the state is f(0): nothing to stream
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (ring[r] > C - 1 - k) continue;
            float f[8], g[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            if (as_is) {
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = from[i * CAP + own[r]];
                if (THERMAL) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) g[j] = fromg[j * CAP + own[r]];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = from[src[r][i]];
                if (top[r]) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (EY[i] < 0) f[i] = f[i] + (float)EX[i] * d.lid6;
                }
                if (THERMAL) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) {
                        const float v = fromg[gsrc[r][j]];
                        const uint32_t q = (kind[r] >> (2 * j)) & 3u;
                        g[j] = q == 0u ? v : ((q == 2u) ? d.abbh - v : d.abbc - v);
                    }
                }
                if (NEE && wall[r])
                    nee_rebuild<THERMAL>(d, wx[NEE ? r : 0], wy[NEE ? r : 0], cB[NEE ? r : 0], c[r], f, g);
            }
            float ux, uy, n7, n8, dT;
            node_update<THERMAL>(d, c[r], f, g, ux, uy, n7, n8, dT);
            if (REC && ring[r] == 0) {
                const uint32_t pb4 = (uint32_t)(d.plane * 4);
                const BufRes rec = buf_res(d.urec + (int64_t)k * 5 * d.plane, 5 * pb4);
                BufIO<float>::st(rec, o[r] * 4, 0u, ux);
                BufIO<float>::st(rec, o[r] * 4, pb4, uy);
                if (d.rec_stress) {
                    BufIO<float>::st(rec, o[r] * 4, 2 * pb4, n7);
                    BufIO<float>::st(rec, o[r] * 4, 3 * pb4, n8);
                }
                if (THERMAL) BufIO<float>::st(rec, o[r] * 4, 4 * pb4, dT);
            }
            if (k < C - 1) {
#pragma unroll
                for (int i = 0; i < 8; ++i) to[i * CAP + own[r]] = (float)(S)f[i];
                if (THERMAL) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) tog[j * CAP + own[r]] = g[j];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) BufIO<S>::st(rout, o[r] * ES, (uint32_t)(i * d.plane * ES), f[i]);
                if (THERMAL) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) BufIO<float>::st(rgout, o[r] * 4, (uint32_t)(j * d.plane * 4), g[j]);
                }
                if (d.uprev) store_uprev(d, o[r] * 4, ux, uy);
            }
        }
    };
    for (int k = 0; k < C; k += 2) {
        cycle(k, lds, ldsg, ldsB, ldsgB);
        if (k + 1 < C) cycle(k + 1, ldsB, ldsgB, lds, ldsg);
    }
}

// Compiled frames: nodes a workgroup can hold (LDS: two buffers of 8 or 13 FP32
// planes, at most 160 KB) and its threads, one or two nodes each.
constexpr int DEEP_CAP = 2040, DEEP_CAP_HEAT = 1536;

// The widest frame of n nodes cut into `tiles`, with a ring of C nodes.
static int deep_width(int n, int tiles, bool periodic, int C) {
    if (tiles == 1) return n;
    const int w = (n + tiles - 1) / tiles + 2 * C;
    return !periodic && w > n ? n : w;
}

// Row stride of the frames in LDS: their width, except that a ring's columns would
// meet in one or two LDS banks at a stride of 32 or 33 (256^2 cavity, eight cycles:
// 1.80 us per step with rows of 32, 1.50 with 34; 200^2, ten: 1.88 with 33, 1.35).
static int deep_stride(const Dom &d, const DeepPlan &p, int C) {
    const int w = deep_width(d.nx, p.tiles_x, d.bc_x == BC_PERIODIC, C);
    return p.tiles_x > 1 && w % 32 < 2 ? w - w % 32 + 2 : w;
}

// LDS nodes of a frame (0 for one beyond every compiled size)
static int deep_frame(const Dom &d, const DeepPlan &p, int C) {
    const int64_t n = (int64_t)deep_stride(d, p, C) * deep_width(d.ny, p.tiles_y, d.bc_y == BC_PERIODIC, C);
    return n <= (d.thermal ? DEEP_CAP_HEAT : DEEP_CAP) ? (int)n : 0;
}

// (the kernel wraps a ring around a periodic axis once)
static bool deep_fits(const Dom &d, const DeepPlan &p, int C) {
    if ((p.tiles_x > 1 && d.bc_x == BC_PERIODIC && C > d.nx) || (p.tiles_y > 1 && d.bc_y == BC_PERIODIC && C > d.ny))
        return false;
    return C >= 1 && p.tiles_x >= 1 && p.tiles_y >= 1 && p.tiles_x <= d.nx && p.tiles_y <= d.ny;
}

// Where the deep pass is taken, and its tiles (us per step, other pass against
// deep pass, one box, 240-step calls):
//   * One workgroup for the whole domain up to 800 nodes (8 x 64: 2.7 against 0.59,
//     24 x 32: 2.6 against 0.76; one-CU arithmetic overtakes the launches there:
//     32 x 32 0.89 alone against 0.84 on 256 tiles), 640 with the D2Q5 field
//     (8 x 64: 3.8 against 1.05) and 512 with on-node walls, whose rebuilt nodes
//     double a wavefront's arithmetic (7.6 against 1.10; 24 x 32 alone 1.67, tiled
//     1.12). 1024 cycles at most, so that no launch holds the chip for long.
//   * Else one tile per CU, as square as they come, and the most cycles up to 10
//     that its frame holds (128^2 lid cavity: 2.5 against 0.98, 256^2 2.6 against
//     1.42, 512^2 3.1 against 2.5, 600 x 500 3.8 against 3.1; convection 200^2 3.2
//     against 1.9, 450^2 4.2 against 3.6). More cycles lose to the ring (128^2: 8
//     cycles 1.03, 12 1.22, 16 1.20). With fewer than five, or in two rounds of
//     tiles, the other passes are as fast or faster (600^2 3.8 against 3.8; 850^2
//     5.7 against 6.7; convection 512^2 4.3 against 5.0).
//   * With on-node walls, whose other pass takes one cycle, up to five rounds
//     (convection 200^2 9.5 against 2.3, 1000^2 22.7 against 17.4; cavity 512^2 7.1
//     against 3.2, 1000^2 14.1 against 11.3).
//   * Where a frame of one node per thread holds seven cycles, no more of them in a
//     larger frame (200^2 cavity: nine 1.22, ten 1.35; 240^2: eight 1.42, ten 1.53;
//     256^2: seven 1.42, nine 1.47; 300^2: six 1.83, ten 1.68).
constexpr int DEEP_MOST_CYCLES = 10, DEEP_LEAST_CYCLES = 5;
constexpr int DEEP_ONE_NODE = 1024, DEEP_ONE_NODE_CYCLES = 7;

bool deep_plan(const Dom &d, int64_t most_tiles, DeepPlan *plan, int *cycles) {
    constexpr int CUS = 256;
    if (most_tiles < 1) return false;
    const bool nee = d.bc_x == BC_NEE || d.bc_y == BC_NEE;
    if ((int64_t)d.nx * d.ny <= (nee ? 512 : (d.thermal ? 640 : 800))) {
        *plan = DeepPlan{1, 1, 0};
        *cycles = 1024;
        return true;
    }
    for (int rounds = 1; rounds <= (nee ? 5 : 1); ++rounds) {
        const int wgs = (int)std::min<int64_t>(CUS * rounds, most_tiles);
        int tx = (int)(std::sqrt((double)wgs * d.nx / d.ny) + 0.5);
        tx = std::min(std::max(tx, 1), std::min(d.nx, wgs));
        const int ty = std::min(wgs / tx, d.ny);
        const DeepPlan p{tx, ty, 0};
        int best = 0;
        for (int C = DEEP_LEAST_CYCLES; C <= DEEP_MOST_CYCLES; ++C) {
            if (!deep_fits(d, p, C) || !deep_frame(d, p, C)) continue;
            if (best >= DEEP_ONE_NODE_CYCLES && deep_frame(d, p, best) <= DEEP_ONE_NODE && deep_frame(d, p, C) > DEEP_ONE_NODE) break;
            best = C;
        }
        if (best > 0) {
            *plan = p;
            *cycles = best;
            return true;
        }
    }
    return false;
}

template <typename S, int MK, bool THERMAL, bool NEE, bool REC>
static hipError_t launch_deep_t(const Dom &d, const DeepPlan &p, int C, int direct, hipStream_t st) {
    const int n = deep_frame(d, p, C);
    if (n == 0) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(p.tiles_x * p.tiles_y));
    const DeepPlan q{p.tiles_x, p.tiles_y, deep_stride(d, p, C)};
#define MRT_DEEP(CAP, NT) \
    if (n <= CAP) { \
        hipLaunchKernelGGL((k_step_deep<S, MK, THERMAL, NEE, REC, CAP, NT>), grid, dim3(NT), 0, st, d, q, C, direct); \
        return hipGetLastError(); \
    }
    MRT_DEEP(512, 512)
    MRT_DEEP(1024, 1024)
    if constexpr (THERMAL) { MRT_DEEP(DEEP_CAP_HEAT, 768) }
    else { MRT_DEEP(DEEP_CAP, 1024) }
#undef MRT_DEEP
    return hipErrorInvalidValue;
}

template <typename S, int MK>
static hipError_t launch_deep_mk(const Dom &d, const DeepPlan &p, int C, int direct, hipStream_t st) {
    const bool nee = d.bc_x == BC_NEE || d.bc_y == BC_NEE;
    if (d.thermal)
        return nee ? launch_deep_t<S, MK, true, true, false>(d, p, C, direct, st)
                   : launch_deep_t<S, MK, true, false, false>(d, p, C, direct, st);
    return nee ? launch_deep_t<S, MK, false, true, false>(d, p, C, direct, st)
               : launch_deep_t<S, MK, false, false, false>(d, p, C, direct, st);
}

hipError_t launch_step_deep(const Dom &d, int storage, const DeepPlan &p, int C, bool direct, hipStream_t st) {
    if (!deep_fits(d, p, C)) return hipErrorInvalidValue;
    const bool uniform = medium_kind(d) == MK_UNIFORM;
    const int dir = direct ? 1 : 0;
    if (storage == ST_F32)
        return uniform ? launch_deep_mk<float, MK_UNIFORM>(d, p, C, dir, st) : launch_deep_mk<float, MK_ANY>(d, p, C, dir, st);
    return uniform ? launch_deep_mk<_Float16, MK_UNIFORM>(d, p, C, dir, st) : launch_deep_mk<_Float16, MK_ANY>(d, p, C, dir, st);
}

// FP32, no on-node walls: what the adjoint takes.
hipError_t launch_step_deep_rec(const Dom &d, const DeepPlan &p, int C, bool direct, hipStream_t st) {
    if (!deep_fits(d, p, C) || d.bc_x == BC_NEE || d.bc_y == BC_NEE) return hipErrorInvalidValue;
    const int dir = direct ? 1 : 0;
    return d.thermal ? launch_deep_t<float, MK_ANY, true, false, true>(d, p, C, dir, st)
                     : launch_deep_t<float, MK_ANY, false, false, true>(d, p, C, dir, st);
}

}  // namespace mrt
