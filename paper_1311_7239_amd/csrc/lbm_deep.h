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

#include "lbm_deep_plan.h"
#include "lbm_launch.h"

namespace mrt {

// REC: every cycle also records its velocity for the adjoint (and the stress
// moments and the temperature), cycle k five planes after cycle k - 1.
template <typename S, int MK, bool THERMAL, bool NEE, bool REC, int CAP, int NT>
__global__ __launch_bounds__(NT) void k_step_deep(Dom d, DeepPlan p, int C, int direct) {
    constexpr int R = (CAP + NT - 1) / NT;
    constexpr int ES = (int)sizeof(S);
    __shared__ float lds[2 * 8 * CAP];
    __shared__ float ldsg[THERMAL ? 2 * 5 * CAP : 1];
    const DeepFrame F(d, p, C, (int)blockIdx.x);
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
