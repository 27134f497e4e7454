// Follows the LDS positions of deep-pass plans on the host (test code only): the
// index arithmetic is the kernels' own (lbm_deep_plan.h), and every read is compared
// with what the cycle before wrote.
//
// Input lines: nx ny bc_x bc_y thermal most_tiles tiles_x tiles_y (tiles_x = 0: the plan
// that the library takes). Output per line:
//   tiles_x tiles_y cycles fits bad
// cycles 0: no plan. fits: the launch accepts it. bad: reads that are not the node and
// cycle that the collision needs, positions outside the frame, nodes not computed exactly
// once and tiles that do not cover an axis, over launches of 1, 2, 3 and `cycles` cycles,
// in the first, second, middle and last tiles of each axis.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "lbm_deep_plan.h"

using namespace mrt;

static long bad_axis(int tiles, int n, bool periodic) {
    long bad = 0;
    for (int k = 0; k < tiles; ++k) {
        const DeepAxis A(k, tiles, n, periodic);
        const int64_t a = (int64_t)k * n / tiles, b = (int64_t)(k + 1) * n / tiles;
        if (A.a != a || A.b != b || a >= b) ++bad;
    }
    return bad;
}

struct Cell_ {
    int cycle = -1;   // the cycle that reads it next, -1: nothing written
    int gx = -1, gy = -1;
};

// One workgroup; reverse: the adjoint's direction of the links.
static long bad_reads(const Dom &d, const DeepPlan &q, int C, int block, bool reverse) {
    long bad = 0;
    const int cap = deep_frame(d, q, C);
    const DeepFrame F(d, q, C, block);
    if (F.n > cap || F.w > F.s || F.n < 1) return 1;
    std::vector<Cell_> lds[2];
    lds[0].resize(cap);
    lds[1].resize(cap);
    const float inv = 1.0f / (float)F.w;
    for (int k = 0; k < F.n; ++k) {
        int at;
        const uint32_t o = F.offset(k, inv, d.pitch, at);
        if (at < 0 || at >= cap || (int)(o % d.pitch) >= d.nx || (int)(o / d.pitch) >= d.ny) {
            ++bad;
            continue;
        }
        lds[0][at] = Cell_{0, (int)(o % d.pitch), (int)(o / d.pitch)};
    }
    struct Node {
        int ring, own, gx, gy, bx, by;
        bool out[8];
        int src[8];
    };
    std::vector<Node> nodes;
    std::set<int> owns;
    long tile = 0;
    for (int s = 0; s < 2048; ++s) {
        int x, y;
        const int ring = deep_node(F.X, F.Y, C, s, x, y);
        if (ring >= C || x >= F.X.last(C) || y >= F.Y.last(C)) continue;
        Node n;
        n.ring = ring;
        n.gx = F.wrapped(x, d.nx);
        n.gy = F.wrapped(y, d.ny);
        n.own = (y - F.y0) * F.s + (x - F.x0);
        n.bx = n.gx;
        n.by = n.gy;
        (void)nee_wall(d, n.gx, n.gy, n.bx, n.by);
        const DeepLinks at(F, n.bx, n.by, x + (n.bx - n.gx) - F.x0, y + (n.by - n.gy) - F.y0);
        for (int i = 0; i < 8; ++i) {
            const int ex = reverse ? -EX[i] : EX[i], ey = reverse ? -EY[i] : EY[i];
            const int p = at.source(ex, ey, i, OPP[i], 1 << 20);
            n.out[i] = (d.bc_x != BC_PERIODIC && (n.bx - ex < 0 || n.bx - ex >= d.nx)) ||
                       (d.bc_y != BC_PERIODIC && (n.by - ey < 0 || n.by - ey >= d.ny));
            const int plane = n.out[i] ? OPP[i] : i;
            n.src[i] = p - (plane << 20);
        }
        if (!owns.insert(n.own).second || n.own < 0 || n.own >= cap) ++bad;
        if (ring == 0) ++tile;
        nodes.push_back(n);
    }
    if (tile != (long)(F.X.b - F.X.a) * (F.Y.b - F.Y.a)) ++bad;
    for (int k = 0; k < C; ++k) {
        const std::vector<Cell_> &from = lds[k & 1];
        std::vector<Cell_> &to = lds[(k + 1) & 1];
        for (const Node &n : nodes) {
            if (n.ring > C - 1 - k) continue;
            for (int i = 0; i < 8; ++i) {
                const int ex = reverse ? -EX[i] : EX[i], ey = reverse ? -EY[i] : EY[i];
                const int wx = n.out[i] ? n.bx : (n.bx - ex + d.nx) % d.nx, wy = n.out[i] ? n.by : (n.by - ey + d.ny) % d.ny;
                const int p = n.src[i];
                if (p < 0 || p >= cap || from[p].cycle != k || from[p].gx != wx || from[p].gy != wy) ++bad;
            }
        }
        for (const Node &n : nodes)
            if (n.ring <= C - 1 - k) to[n.own] = Cell_{k + 1, n.gx, n.gy};
    }
    return bad;
}

int main() {
    int nx, ny, bx, by, thermal, most, tx, ty;
    while (std::scanf("%d %d %d %d %d %d %d %d", &nx, &ny, &bx, &by, &thermal, &most, &tx, &ty) == 8) {
        Dom d;
        std::memset((void *)&d, 0, sizeof(d));
        d.nx = nx;
        d.ny = ny;
        d.pitch = (nx + 63) / 64 * 64;
        d.bc_x = bx;
        d.bc_y = by;
        d.thermal = thermal;
        DeepPlan p{tx, ty, 0};
        int cycles = 5;
        if (tx == 0 && !deep_plan(d, most, &p, &cycles)) {
            std::printf("0 0 0 0 0\n");
            continue;
        }
        const bool fits = deep_fits(d, p, cycles);
        long bad = bad_axis(p.tiles_x, nx, bx == BC_PERIODIC) + bad_axis(p.tiles_y, ny, by == BC_PERIODIC);
        const int lengths[4] = {1, 2, 3, cycles > 16 ? 16 : cycles};
        for (int q = 0; q < 4 && bad == 0; ++q) {
            const int C = lengths[q];
            const DeepPlan pl{p.tiles_x, p.tiles_y, deep_stride(d, p, C)};
            if (C > cycles || deep_frame(d, p, C) == 0) continue;
            std::set<int> xs{0, std::min(1, p.tiles_x - 1), p.tiles_x / 2, p.tiles_x - 1};
            std::set<int> ys{0, std::min(1, p.tiles_y - 1), p.tiles_y / 2, p.tiles_y - 1};
            for (int x : xs)
                for (int y : ys)
                    for (int reverse = 0; reverse < (bx == BC_NEE || by == BC_NEE ? 1 : 2); ++reverse)
                        bad += bad_reads(d, pl, C, y * p.tiles_x + x, reverse != 0);
        }
        std::printf("%d %d %d %d %ld\n", p.tiles_x, p.tiles_y, cycles, fits ? 1 : 0, bad);
    }
    return 0;
}
