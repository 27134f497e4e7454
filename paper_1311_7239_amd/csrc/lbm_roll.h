// The rolling pass: C cycles per launch for mid-size domains.
//
// A workgroup owns a strip of 64 columns and a run of its rows, and rolls over
// them eight rows at a time, one row per wavefront: cycle 0 on the next eight rows
// from HBM, then cycle 1 on the eight rows one behind, cycle 2 two behind, ... What
// cycle k - 1 made of the last ten rows lies in LDS, a ring of rows per cycle, so no
// row is collided twice but the few at the ends of a run. The links that a node
// pulls from the row above are the wavefront's own from the cycle before and stay
// in registers (the diagonal ones move a lane by DPP); the other five go through
// LDS, at one address per row and without a branch: what comes back from a wall is
// written by the node next to it where the pull across the wall reads. The next
// eight rows' loads are in flight during all the cycles of these.
//
// Against the tiles of the other passes (load a tile, collide it, exchange it,
// collide it, store it, with every workgroup of the chip in the same phase): 96
// vector instructions per update, no re-collided ring above and below, six cycles a
// launch (four with the D2Q5 field) instead of two or three, and memory busy
// throughout. What bounds it: at 1024^2 vector issue, of which 60% is reached: the
// first and last turns of a run, when not every wavefront has a row (39 rows take
// seven turns, a fifth of them idle), a launch and its first load (5 of 37 us).
// us per step, tiles -> rolling: 1024^2 cavity 7.0 -> 6.1, log-normal channel 7.7 ->
// 6.7, with a J plane 7.9 -> 6.9, convection 10.4 -> 8.3; 1700^2 convection 37 -> 21;
// 2048^2 channel 22.6 -> 19.7. Two workgroups of eight wavefronts per CU are the best
// shape: four cycles (LDS for four workgroups) 6.1 with two, 6.6 with four, 6.2 with
// one of sixteen wavefronts.
//
// A batch runs the strips of all its domains from one table (k_step3_roll_batch), and
// the adjoint's recomputation records in these passes too (REC).
#pragma once

#include <algorithm>
#include <type_traits>
#include <vector>

#include "lbm_launch.h"
#include "lbm_strip.h"

namespace mrt {

constexpr int ROLL_COLS = 64;    // columns a workgroup holds, its ring of C - 1 on each side included
constexpr int ROLL_ROWS = 8;     // rows (wavefronts)

// The columns [c0, c1) that strip k writes and the first one it holds. At a wall
// a strip has no ring on that side.
__host__ __device__ inline int roll_strips(int nx, bool periodic, int C) {
    const int w = ROLL_COLS - 2 * (C - 1), e = ROLL_COLS - (C - 1);
    if (periodic) return (nx + w - 1) / w;
    if (nx <= ROLL_COLS) return 1;
    if (nx <= 2 * e) return 2;
    return 2 + (nx - 2 * e + w - 1) / w;
}
__host__ __device__ inline int roll_begin(int k, int nx, bool periodic, int C) {
    // strips of nearly equal width, where the first and the last are wider by a ring at a wall
    const int n = roll_strips(nx, periodic, C), g = periodic ? 0 : C - 1;
    if (k <= 0) return 0;
    if (k >= n) return nx;
    return g + (int)((int64_t)k * (nx - 2 * g) / n);
}

// Strip sk of p.strips and run rk of p.runs of a domain. REC: every cycle also records
// its velocity for the adjoint (and the stress moments and the temperature), cycle k
// five planes after cycle k - 1.
template <typename S, int C, int MK, bool THERMAL, bool REC>
__device__ __forceinline__ void roll_run(const Dom &d, const RollPlan &p, int sk, int rk) {
    static_assert(C >= 3, "a barrier between a cycle's reads and the next rows' writes");
    constexpr int H = ROLL_ROWS, RING = H + 2, G = C - 1, ES = (int)sizeof(S);
    constexpr bool CELLS = MK != MK_UNIFORM, SNU = MK == MK_ANY;
    // Planes of the links that the next cycle pulls from the same row or the one below
    // (those from the row above, its wavefront has just made itself). A row is a column
    // longer than the strip: what a link along +x pulls across the wall x = 0 lies
    // before the row, along -x after it, and no plane has both; so the planes with a
    // column before come first, and a float follows the last one.
    constexpr int NF = 5, NG = 4, ROW = ROLL_COLS + 1, PL = RING * ROW, LF = NF * PL + 1, LG = NG * PL + 1;
    constexpr int AT[8] = {0, 2, 3, -1, 1, 4, -1, -1}, ATG[5] = {1, 0, 2, 3, -1};
    __shared__ float lds[(C - 1) * LF];
    __shared__ float ldsg[THERMAL ? (C - 1) * LG : 1];
    constexpr int CR = H + C - 1;
    __shared__ float4 cells[CELLS ? CR * 64 : 1];
    __shared__ float snus[SNU ? CR * 64 : 1];
    const int lane = (int)threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool per_x = d.bc_x == BC_PERIODIC, per_y = d.bc_y == BC_PERIODIC;
    const int c0 = roll_begin(sk, d.nx, per_x, C), c1 = roll_begin(sk + 1, d.nx, per_x, C);
    const int y0 = (int)((int64_t)rk * d.ny / p.runs), y1 = (int)((int64_t)(rk + 1) * d.ny / p.runs);
    const int xa = (per_x ? c0 - G : std::max(c0 - G, 0)) + lane;
    // the lane's column and those beside it; a lane beyond a wall holds whatever column 0 holds
    int col = xa;
    if (per_x) col = xa < 0 ? xa + d.nx : (xa >= d.nx ? xa - d.nx : xa);
    else if (xa >= d.nx) col = 0;
    const int colm = col == 0 ? d.nx - 1 : col - 1, colp = col == d.nx - 1 ? 0 : col + 1;
    const bool in = xa >= c0 && xa < c1, inside = per_x || xa < d.nx;
    const bool xw = !per_x && (sk == 0 || sk == p.strips - 1);
    const bool la = xw && xa == 0, ra = xw && xa == d.nx - 1;   // next to an x wall

    const uint32_t pl = (uint32_t)(d.plane * ES), rowb = (uint32_t)(d.pitch * ES);
    const uint32_t plg = (uint32_t)(d.plane * 4), rowg = (uint32_t)(d.pitch * 4);
    const BufRes rin = buf_res(d.fin, 8 * pl), rout = buf_res(d.fout, 8 * pl);
    const BufRes rgin = buf_res(THERMAL ? d.gin : nullptr, THERMAL ? 5 * plg : 0u);
    const BufRes rgout = buf_res(THERMAL ? d.gout : nullptr, THERMAL ? 5 * plg : 0u);
    const MediumSrc<MK> med(d);
    constexpr uint32_t NOWHERE = 0xfffffff0u;   // beyond the buffers: a store there is dropped
    const uint32_t vst = in ? (uint32_t)(col * ES) : NOWHERE, vs4 = in ? (uint32_t)(col * 4) : NOWHERE;

    const int lo = per_y ? y0 - G : std::max(y0 - G, 0), hi = per_y ? y1 + G : std::min(y1 + G, d.ny);
    auto wrap_row = [&](int y) -> int {
        if (!per_y) return y;
        y = y < 0 ? y + d.ny : y;
        return y >= d.ny ? y - d.ny : y;
    };

    // row y as cycle 0 pulls it; across a wall the node's own opposite link
    struct Raw {
        float f[8], g[5];
        CellRaw c;
    };
    auto fetch = [&](auto plain, auto edge, int y, Raw &w) {
        constexpr bool PLAIN = decltype(plain)::value, EDGE = decltype(edge)::value;
        const int yc = wrap_row(y), ym = wrap_row(y - 1), yp = wrap_row(y + 1);
        const bool bot = !PLAIN && !per_y && y == 0, top = !PLAIN && !per_y && y == d.ny - 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool out = (EY[i] > 0 && bot) || (EY[i] < 0 && top);
            const uint32_t so = (uint32_t)i * pl + (uint32_t)(EY[i] > 0 ? ym : (EY[i] < 0 ? yp : yc)) * rowb;
            const uint32_t oo = (uint32_t)OPP[i] * pl + (uint32_t)yc * rowb;
            const uint32_t v = (uint32_t)((EX[i] > 0 ? colm : (EX[i] < 0 ? colp : col)) * ES), vo = (uint32_t)(col * ES);
            if (EDGE && EX[i] != 0) {
                const bool own = out || (EX[i] > 0 ? la : ra);
                w.f[i] = BufIO<S>::ld(rin, own ? vo + oo : v + (out ? oo : so), 0u);
            } else {
                w.f[i] = BufIO<S>::ld(rin, out ? vo : v, out ? oo : so);
            }
        }
        if (THERMAL) {
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                const bool out = (TYv[j] > 0 && bot) || (TYv[j] < 0 && top);
                const uint32_t so = (uint32_t)j * plg + (uint32_t)(TYv[j] > 0 ? ym : (TYv[j] < 0 ? yp : yc)) * rowg;
                const uint32_t oo = (uint32_t)TOPP[j] * plg + (uint32_t)yc * rowg;
                const uint32_t v = (uint32_t)((TXv[j] > 0 ? colm : (TXv[j] < 0 ? colp : col)) * 4), vo = (uint32_t)(col * 4);
                if (EDGE && TXv[j] != 0) w.g[j] = BufIO<float>::ld(rgin, (TXv[j] > 0 ? la : ra) ? vo + oo : v + so, 0u);
                else w.g[j] = BufIO<float>::ld(rgin, v, out ? oo : so);
            }
        }
        w.c = med.load((uint32_t)yc * rowg + (uint32_t)(col * 4));
    };

    Raw w;
    int slot = wv;   // of the wavefront's row of cycle 0 in the rings of H + 2 rows
    int cslot = wv;  // and in that of the cells
    auto back = [](int s, int n, int ring) -> int { return s >= n ? s - n : s + ring - n; };

    // H rows through every cycle, the first of cycle 0 at row r. FULL: every wavefront
    // has a row in each cycle, none of them (nor the next ones) next to a y wall.
    auto advance = [&](auto full, auto edge, int r) {
        constexpr bool FULL = decltype(full)::value, EDGE = decltype(edge)::value;
        Cell kept[C - 1];
        float f[8], g[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const int y = r + wv - k;
            const bool act = FULL || (y >= std::max(lo, y0 - (G - k)) && y < std::min(hi, y1 + (G - k)));
            const bool bot = !FULL && !per_y && y == 0, top = !FULL && !per_y && y == d.ny - 1;
            // LDS positions of the lane's node in rows y and y - 1
            const int a0 = back(slot, k, RING) * ROW + 1 + lane, am = back(slot, k + 1, RING) * ROW + 1 + lane;
            Cell c;
            if (k == 0) {
                const CellRaw raw = w.c;
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = w.f[i];
                if (THERMAL) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) g[j] = w.g[j];
                    if (EDGE) {
                        g[1] = la ? d.abbh - g[1] : g[1];
                        g[3] = ra ? d.abbc - g[3] : g[3];
                    }
                }
                fetch(full, edge, std::min(y + H, hi - 1), w);
                c = med.cell(d, raw);
                if (CELLS && act) cells[cslot * 64 + lane] = make_float4(c.phi, c.inv_phi, c.cdh, c.cfh);
                if (SNU && act) snus[cslot * 64 + lane] = c.s_nu;
            } else if (act) {
                // f holds row y + 1 of the cycle before
                const float *B = lds + (k - 1) * LF, *Bg = ldsg + (THERMAL ? (k - 1) * LG : 0);
                f[6] = from_right(f[6]);
                f[7] = from_left(f[7]);
                if (top) {
                    f[3] = B[AT[1] * PL + a0];
                    f[6] = B[AT[4] * PL + a0];
                    f[7] = B[AT[5] * PL + a0];
                } else if (EDGE) {
                    const float own4 = B[AT[4] * PL + a0], own5 = B[AT[5] * PL + a0];
                    f[6] = ra ? own4 : f[6];
                    f[7] = la ? own5 : f[7];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (EY[i] >= 0) f[i] = B[AT[i] * PL + (EY[i] > 0 ? am : a0) - EX[i]];
                if (THERMAL) {
                    if (top) g[4] = Bg[ATG[2] * PL + a0];
#pragma unroll
                    for (int j = 0; j < 4; ++j) g[j] = Bg[ATG[j] * PL + (TYv[j] > 0 ? am : a0) - TXv[j]];
                }
                c = kept[k - 1];
            }
            if (act) {
                if (top) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (EY[i] < 0) f[i] = f[i] + (float)EX[i] * d.lid6;
                }
                float ux, uy, n7, n8, dT;
                node_update<THERMAL>(d, c, f, g, ux, uy, n7, n8, dT);
                if (REC && y >= y0 && y < y1) {
                    const BufRes rec = buf_res(d.urec + (int64_t)k * 5 * d.plane, 5 * plg);
                    const uint32_t so = (uint32_t)y * rowg;
                    BufIO<float>::st_nt(rec, vs4, so, ux);
                    BufIO<float>::st_nt(rec, vs4, so + plg, uy);
                    if (d.rec_stress) {
                        BufIO<float>::st_nt(rec, vs4, so + 2 * plg, n7);
                        BufIO<float>::st_nt(rec, vs4, so + 3 * plg, n8);
                    }
                    if (THERMAL) BufIO<float>::st_nt(rec, vs4, so + 4 * plg, dT);
                }
                if (k < C - 1) {
                    float *B = lds + k * LF, *Bg = ldsg + (THERMAL ? k * LG : 0);
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] = (float)(S)f[i];
                    if (!EDGE || inside) {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (AT[i] >= 0) B[AT[i] * PL + a0] = f[i];
                        if (THERMAL) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) Bg[ATG[j] * PL + a0] = g[j];
                        }
                        // what comes back from a wall, where the pull across it reads
                        if (EDGE && la) {
                            B[AT[0] * PL + a0 - 1] = f[2];
                            B[AT[4] * PL + am - 1] = f[6];
                            if (THERMAL) Bg[ATG[1] * PL + a0 - 1] = d.abbh - g[3];
                        }
                        if (EDGE && ra) {
                            B[AT[2] * PL + a0 + 1] = f[0];
                            B[AT[5] * PL + am + 1] = f[7];
                            if (THERMAL) Bg[ATG[3] * PL + a0 + 1] = d.abbc - g[1];
                        }
                        if (bot) {
                            B[AT[1] * PL + am] = f[3];
                            B[AT[4] * PL + am - 1] = f[6];
                            B[AT[5] * PL + am + 1] = f[7];
                            if (THERMAL) Bg[ATG[2] * PL + am] = g[4];
                        }
                    }
                } else {
                    const uint32_t so = (uint32_t)y * rowb, sg = (uint32_t)y * rowg;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (d.nt_store) BufIO<S>::st_nt(rout, vst, so + (uint32_t)i * pl, f[i]);
                        else BufIO<S>::st(rout, vst, so + (uint32_t)i * pl, f[i]);
                    }
                    if (THERMAL) {
#pragma unroll
                        for (int j = 0; j < 5; ++j) {
                            if (d.nt_store) BufIO<float>::st_nt(rgout, vs4, sg + (uint32_t)j * plg, g[j]);
                            else BufIO<float>::st(rgout, vs4, sg + (uint32_t)j * plg, g[j]);
                        }
                    }
                    if (d.uprev && in) store_uprev(d, sg + (uint32_t)(col * 4), ux, uy);
                }
            }
            if (k < C - 1) lds_barrier();
            if (k == 0) {
                // the cells of the later cycles' rows, before another wavefront overwrites them
#pragma unroll
                for (int m = 1; m < C; ++m) {
                    if (!CELLS) {
                        kept[m - 1] = med.cell(d, CellRaw{0.0f, 0.0f, 0.0f});
                        continue;
                    }
                    const int cs = back(cslot, m, CR) * 64 + lane;
                    const float4 u = cells[cs];
                    Cell &q = kept[m - 1];
                    q.phi = u.x;
                    q.inv_phi = u.y;
                    q.cdh = u.z;
                    q.cfh = u.w;
                    q.s_nu = d.s_nu;
                    q.h_nu2 = d.h_nu2;
                    q.h_nu4 = d.h_nu4;
                    if (SNU) {
                        // with a s_nu plane its entry, without one d.s_nu, whose multiples are these too
                        q.s_nu = snus[cs];
                        if (d.snu) {
                            q.h_nu2 = 2.0f - q.s_nu;
                            q.h_nu4 = fmaf(-2.0f, q.s_nu, 4.0f);
                        }
                    }
                }
            }
        }
        slot = slot + H >= RING ? slot + H - RING : slot + H;
        cslot = cslot + H >= CR ? cslot + H - CR : cslot + H;
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    const int end = y1 + G;   // cycle C - 1 has made row y1 - 1 when cycle 0 stands here
    int full0 = y0 + G, full1 = hi;   // FULL: r >= full0 and r + H <= full1
    if (!per_y) {
        full0 = std::max(full0, C);
        full1 = std::min(full1, d.ny - 1 - H);
    }
    int r = lo;
    if (xw) {
        fetch(no, yes, std::min(lo + wv, hi - 1), w);
        for (; r < full0 && r < end; r += H) advance(no, yes, r);
        for (; r + H <= full1; r += H) advance(yes, yes, r);
        for (; r < end; r += H) advance(no, yes, r);
    } else {
        fetch(no, no, std::min(lo + wv, hi - 1), w);
        for (; r < full0 && r < end; r += H) advance(no, no, r);
        for (; r + H <= full1; r += H) advance(yes, no, r);
        for (; r < end; r += H) advance(no, no, r);
    }
}

template <typename S, int C, int MK, bool THERMAL, bool REC>
__global__ __launch_bounds__(64 * ROLL_ROWS) __attribute__((amdgpu_waves_per_eu(4))) void k_step3_roll(
    Dom d, RollPlan p) {
    const int item = xcd_swizzle((int)blockIdx.x, (int)gridDim.x);
    roll_run<S, C, MK, THERMAL, REC>(d, p, item % p.strips, item / p.strips);
}

// The same over a table of runs (domain, strip, run, runs of the domain; domain -1: none),
// for the domains of a batch: every run of all of them in one launch, against tiles of
// four cycles (two with the D2Q5 field) whose rings cost a small domain the most. 60
// cavities of 64 to 768 nodes a side 70 -> 62 us per step, the 27 heated cavities of
// Table 1 16.0 -> 9.4, 60 heated ones of 64 to 400 51 -> 27.
template <typename S, int C, int MK, bool THERMAL>
__global__ __launch_bounds__(64 * ROLL_ROWS) __attribute__((amdgpu_waves_per_eu(4))) void k_step3_roll_batch(
    const Dom *__restrict__ doms, const int4 *__restrict__ items, int parity, int nt_store) {
    const int4 it = items[blockIdx.x];
    if (it.x < 0) return;
    Dom d = doms[2 * it.x + parity];
    d.nt_store = nt_store;
    roll_run<S, C, MK, THERMAL, false>(d, RollPlan{roll_strips(d.nx, d.bc_x == BC_PERIODIC, C), it.w}, it.y, it.z);
}

// Two workgroups per CU (LDS: at most 80 KB each) in one round.
static RollPlan roll_plan(const Dom &d, int C) {
    RollPlan p{roll_strips(d.nx, d.bc_x == BC_PERIODIC, C), 0};
    p.runs = std::min(std::max(512 / p.strips, 1), d.ny);
    return p;
}

// The kernel of a pass (NULL: none compiled), the most cycles that two workgroups'
// LDS holds being six, with the D2Q5 field four, and three beside the cells of
// MK_ANY.
template <typename S, bool THERMAL, bool REC, int MK>
static const void *roll_fn_t(int cycles) {
    if (cycles == 3) return (const void *)&k_step3_roll<S, 3, MK, THERMAL, REC>;
    if constexpr (!THERMAL || MK != MK_ANY)
        if (cycles == 4) return (const void *)&k_step3_roll<S, 4, MK, THERMAL, REC>;
    if constexpr (!THERMAL)
        if (cycles == 6) return (const void *)&k_step3_roll<S, 6, MK, THERMAL, REC>;
    return nullptr;
}

template <typename S, bool THERMAL>
static const void *roll_fn_mk(const Dom &d, int cycles) {
    switch (medium_kind(d)) {
    case MK_ERGUN: return roll_fn_t<S, THERMAL, false, MK_ERGUN>(cycles);
    case MK_UNIFORM: return roll_fn_t<S, THERMAL, false, MK_UNIFORM>(cycles);
    default: return roll_fn_t<S, THERMAL, false, MK_ANY>(cycles);
    }
}

// Cycles of the next rolling pass with n left (0: another pass): six, or with the
// D2Q5 field four (three in a medium of any kind), and fours and threes where they
// come out even.
int roll_cycles(bool thermal, bool any_medium, int64_t n) {
    if (n < 3) return 0;
    if (!thermal) return strip_cycles(n);
    if (any_medium) return 3;
    return n == 3 || n == 6 || n == 9 ? 3 : (n == 5 ? 3 : 4);
}

// Where the rolling pass is taken (us per step in 96-step calls, the other pass
// against it, one box), beyond the domains that step in deep passes:
//   * bounce-back walls, strips that fill half their lanes and runs of some rows;
//   * upwards until the populations leave the Infinity Cache, from where on a
//     strip's rows, 216 to 240 bytes off their alignment, cost more than the wider
//     strips' and tiles' (cavity 2240^2 26.6 against 19.9, 2900^2 32.7 against 36.2;
//     channel 2240^2 25.7 against 23.6, 2900^2 36.1 against 38.2; convection 2048^2 42
//     against 35, 3400 x 1500 41 against 49); with a 1/K or a viscosity plane, which
//     the strip pass does not take, 2900^2 43.2 against 41.7, and heated, in three
//     cycles, to 2^22 nodes (2100^2, three cycles: 141 against 151);
//   * binary16 storage, whose loads convert, from 400,000 nodes (channel 600^2 3.9
//     against 4.2, 700^2 4.8 against 4.4; 2048^2 20.7 against 19.6) and in uniform media
//     to 3 x 2^20 (cavity 1700^2 13.5 against 13.3, 4099 x 1001 16.9 against 18.2).
bool roll_domain(const Dom &d, int storage) {
    const int64_t nodes = (int64_t)d.nx * d.ny, M = (int64_t)1 << 20;
    const int mk = medium_kind(d);
    if (d.bc_x == BC_NEE || d.bc_y == BC_NEE || d.nx < 2 * ROLL_COLS || d.ny < ROLL_COLS) return false;
    if (storage == ST_F16 && !d.thermal)
        return mk == MK_UNIFORM ? nodes <= 3 * M : (nodes >= 400000 && nodes <= 4 * M);
    if (d.thermal) return mk == MK_ANY ? nodes < 4 * M : nodes <= 9 * M / 2;
    return nodes <= (mk == MK_ANY ? 8 * M : 5 * M);
}

hipError_t launch_step_roll(const Dom &d, int storage, int cycles, hipStream_t st) {
    const void *fn = storage == ST_F32 ? (d.thermal ? roll_fn_mk<float, true>(d, cycles) : roll_fn_mk<float, false>(d, cycles))
                                       : (d.thermal ? roll_fn_mk<_Float16, true>(d, cycles) : roll_fn_mk<_Float16, false>(d, cycles));
    if (!fn || !roll_domain(d, storage)) return hipErrorInvalidValue;
    Dom dd = d;
    RollPlan p = roll_plan(d, cycles);
    void *args[2] = {&dd, &p};
    return hipLaunchKernel(fn, dim3((unsigned)(p.strips * p.runs)), dim3(64 * ROLL_ROWS), args, 0, st);
}

// FP32; a uniform medium takes the kernel of any.
hipError_t launch_step_roll_rec(const Dom &d, int cycles, hipStream_t st) {
    const bool ergun = medium_kind(d) == MK_ERGUN;
    const void *fn = nullptr;
    if (d.thermal) fn = ergun ? roll_fn_t<float, true, true, MK_ERGUN>(cycles) : roll_fn_t<float, true, true, MK_ANY>(cycles);
    else fn = ergun ? roll_fn_t<float, false, true, MK_ERGUN>(cycles) : roll_fn_t<float, false, true, MK_ANY>(cycles);
    if (!fn || !roll_domain(d, ST_F32)) return hipErrorInvalidValue;
    Dom dd = d;
    RollPlan p = roll_plan(d, cycles);
    void *args[2] = {&dd, &p};
    return hipLaunchKernel(fn, dim3((unsigned)(p.strips * p.runs)), dim3(64 * ROLL_ROWS), args, 0, st);
}

// ---- batches

template <typename S, bool THERMAL, int MK>
static const void *roll_batch_fn_t(int cycles) {
    if (cycles == 3) return (const void *)&k_step3_roll_batch<S, 3, MK, THERMAL>;
    if constexpr (!THERMAL || MK != MK_ANY)
        if (cycles == 4) return (const void *)&k_step3_roll_batch<S, 4, MK, THERMAL>;
    if constexpr (!THERMAL)
        if (cycles == 6) return (const void *)&k_step3_roll_batch<S, 6, MK, THERMAL>;
    return nullptr;
}

template <typename S>
static const void *roll_batch_fn(int cycles, bool thermal, bool uniform) {
    if (thermal)
        return uniform ? roll_batch_fn_t<S, true, MK_UNIFORM>(cycles) : roll_batch_fn_t<S, true, MK_ANY>(cycles);
    return uniform ? roll_batch_fn_t<S, false, MK_UNIFORM>(cycles) : roll_batch_fn_t<S, false, MK_ANY>(cycles);
}

// Turns of eight rows that a run of `rows` rows takes, and one for its first load.
static int64_t roll_turns(int rows, int C) { return (rows + 2 * (C - 1) + ROLL_ROWS - 1) / ROLL_ROWS + 1; }

// The runs of a batch in the order of their launch. At most R rows each, for the R
// that ends first: no sooner than the longest run, nor (in more than one round of
// workgroups, two per CU) than the turns of all together and a tenth of the longest.
// The longest run goes first, and eight strips side by side go to one XCD (which
// workgroup b % 8 tells), so that every XCD has its share of long ones (12 cavities of
// 160 to 760 nodes 17.9 us per step in the order of the domains, 16.6 so; the 27 heated
// cavities of Table 1 10.0, 9.4).
std::vector<int4> roll_batch_items(const std::vector<RollShape> &doms, int first, int C) {
    constexpr int64_t SLOTS = 512;
    int tallest = 1;
    for (const RollShape &s : doms) tallest = std::max(tallest, s.ny);
    auto count = [&](int R) -> int64_t {
        int64_t n = 0;
        for (const RollShape &s : doms) n += (int64_t)roll_strips(s.nx, s.per_x, C) * ((s.ny + R - 1) / R);
        return n;
    };
    int best_rows = tallest;
    double best = 1e300;
    for (int rounds = 1; rounds <= 8; ++rounds) {
        int lo = 1, hi = tallest;   // the fewest rows that need no more rounds
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (count(mid) <= SLOTS * rounds) hi = mid;
            else lo = mid + 1;
        }
        int64_t all = 0, longest = 0;
        for (const RollShape &s : doms) {
            const int runs = (s.ny + lo - 1) / lo;
            const int64_t t = roll_turns((s.ny + runs - 1) / runs, C);
            all += t * runs * roll_strips(s.nx, s.per_x, C);
            longest = std::max(longest, t);
        }
        const double one = (double)longest, many = (double)all / SLOTS + 0.1 * (double)longest;
        const double cost = count(lo) <= SLOTS ? one : std::max(one, many);
        if (cost < best) {
            best = cost;
            best_rows = lo;
        }
    }
    struct Run {
        int domain, run, runs, rows;
    };
    std::vector<Run> order;
    for (size_t k = 0; k < doms.size(); ++k) {
        const int64_t runs = (doms[k].ny + best_rows - 1) / best_rows;
        for (int64_t r = 0; r < runs; ++r)
            order.push_back(Run{(int)k, (int)r, (int)runs, (int)((r + 1) * doms[k].ny / runs - r * doms[k].ny / runs)});
    }
    std::stable_sort(order.begin(), order.end(), [](const Run &a, const Run &b) { return a.rows > b.rows; });
    std::vector<int4> list;
    for (const Run &q : order)
        for (int s = 0; s < roll_strips(doms[(size_t)q.domain].nx, doms[(size_t)q.domain].per_x, C); ++s)
            list.push_back(make_int4(first + q.domain, s, q.run, q.runs));
    constexpr size_t XCDS = 8, SIDE = 8;
    std::vector<int4> items((list.size() + XCDS * SIDE - 1) / (XCDS * SIDE) * (XCDS * SIDE), make_int4(-1, 0, 0, 0));
    for (size_t j = 0; j < list.size(); ++j) {
        const size_t chunk = j / SIDE;
        items[((chunk / XCDS) * SIDE + j % SIDE) * XCDS + chunk % XCDS] = list[j];
    }
    return items;
}

// What the rolling pass can run in a batch (bounce-back walls): the ring wraps around a
// periodic axis once.
bool roll_batch_domain(const RollShape &s, bool per_y) {
    return s.nx >= (s.per_x ? ROLL_COLS : 16) && s.ny >= (per_y ? ROLL_COLS : 16);
}

hipError_t launch_step_roll_batch(const Dom *doms, const int4 *items, int nitems, int cycles, int parity, int nt_store,
                                  int storage, bool thermal, bool uniform, hipStream_t st) {
    const void *fn = storage == ST_F32 ? roll_batch_fn<float>(cycles, thermal, uniform)
                                       : roll_batch_fn<_Float16>(cycles, thermal, uniform);
    if (!fn || nitems < 1) return hipErrorInvalidValue;
    void *args[4] = {&doms, &items, &parity, &nt_store};
    return hipLaunchKernel(fn, dim3((unsigned)nitems), dim3(64 * ROLL_ROWS), args, 0, st);
}

}  // namespace mrt
