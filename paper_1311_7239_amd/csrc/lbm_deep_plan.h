// The deep pass's tiles: which domains it serves and on what plan, and how a
// workgroup's tile and the ring around it lie in LDS. Host and device code, without
// kernels, so that a host program can follow every LDS position of a plan.
#pragma once

#include <algorithm>
#include <cmath>

#include "lbm_launch.h"

namespace mrt {

#define MRT_HD __host__ __device__

// One axis of a tile: its nodes [a, b), and how far the ring around it reaches
// (not past a wall, and nowhere on an axis that one tile covers).
struct DeepAxis {
    int a, b, lo, hi;
    MRT_HD DeepAxis(int k, int tiles, int n, bool periodic) {
        // tiles of nearly equal size: tile k of T spans [k n / T, (k + 1) n / T)
        // (products below 2^31: deep_fits refuses others)
        a = k * n / tiles;
        b = (k + 1) * n / tiles;
        lo = tiles == 1 || !periodic ? 0 : -(1 << 30);
        hi = tiles == 1 || !periodic ? n : 1 << 30;
    }
    // the nodes within g of the tile
    MRT_HD int first(int g) const { return a - g < lo ? lo : a - g; }
    MRT_HD int last(int g) const { return b + g > hi ? hi : b + g; }
};

// s / w for s below 2^20 (inv = 1 / w)
MRT_HD __forceinline__ int small_div(int s, float inv) { return (int)(((float)s + 0.5f) * inv); }

// Node number s of a tile and its ring (0: the tile itself): the tile row by
// row, then ring after ring: the row above, the row below, the left and right
// columns; a side at a wall has none. Only the first `rings` rings are numbered.
MRT_HD __forceinline__ int deep_node(const DeepAxis &X, const DeepAxis &Y, int rings, int s, int &x, int &y) {
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
    MRT_HD DeepFrame(const Dom &d, const DeepPlan &p, int C, int block)
        : X(block % p.tiles_x, p.tiles_x, d.nx, d.bc_x == BC_PERIODIC),
          Y(block / p.tiles_x, p.tiles_y, d.ny, d.bc_y == BC_PERIODIC) {
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
    MRT_HD static int wrapped(int v, int m) { return v < 0 ? v + m : (v >= m ? v - m : v); }
    // node offset in a plane, and LDS position, of the frame's k-th node
    MRT_HD uint32_t offset(int k, float inv, int pitch, int &at) const {
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
    MRT_HD DeepLinks(const DeepFrame &F, int bx, int by, int cx_, int cy) {
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
    MRT_HD int source(int ex, int ey, int plane, int oplane, int cap) const {
        const bool out = (ex > 0 && outl) || (ex < 0 && outr) || (ey > 0 && outb) || (ey < 0 && outt);
        const int at = (ey > 0 ? rowm : (ey < 0 ? rowp : row0)) + (ex > 0 ? colm : (ex < 0 ? colp : cx));
        return out ? oplane * cap + row0 + cx : plane * cap + at;
    }
};

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

// The most tiles an axis of n nodes is cut into. A node on an on-node wall is rebuilt from
// the gather of its inner neighbour and so needs nodes two away from the wall, one ring
// more than other nodes do unless the second of the two lies in the tile as well: tiles
// of two nodes at least there.
static int deep_most_tiles(int n, int bc) { return bc == BC_NEE ? std::max(n / 2, 1) : n; }

// (the kernel wraps a ring around a periodic axis once)
static bool deep_fits(const Dom &d, const DeepPlan &p, int C) {
    if ((p.tiles_x > 1 && d.bc_x == BC_PERIODIC && C > d.nx) || (p.tiles_y > 1 && d.bc_y == BC_PERIODIC && C > d.ny))
        return false;
    if ((int64_t)p.tiles_x * d.nx > INT32_MAX || (int64_t)p.tiles_y * d.ny > INT32_MAX) return false;   // DeepAxis
    return C >= 1 && p.tiles_x >= 1 && p.tiles_y >= 1 && p.tiles_x <= deep_most_tiles(d.nx, d.bc_x) &&
           p.tiles_y <= deep_most_tiles(d.ny, d.bc_y);
}

// Where the deep pass is taken, and its tiles (us per step, other pass against
// deep pass, one box, 240-step calls):
//   * One workgroup for the whole domain up to 800 nodes (8 x 64: 2.7 against 0.59,
//     24 x 32: 2.6 against 0.76; one-CU arithmetic overtakes the launches there:
//     32 x 32 0.89 alone against 0.84 on 256 tiles), 640 with the D2Q5 field
//     (8 x 64: 3.8 against 1.05) and 512 with on-node walls, whose rebuilt nodes
//     double a wavefront's arithmetic (7.6 against 1.10; 24 x 32 alone 1.67, tiled
//     1.01). 1024 cycles at most, so that no launch holds the chip for long.
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
        tx = std::min(std::max(tx, 1), std::min(deep_most_tiles(d.nx, d.bc_x), wgs));
        const int ty = std::min(wgs / tx, deep_most_tiles(d.ny, d.bc_y));
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

}  // namespace mrt
