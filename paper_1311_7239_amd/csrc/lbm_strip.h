// The strip pass: C cycles per launch for large domains, in registers.
//
// A wavefront owns a strip of 128 columns (two per lane) and walks it row by
// row. At each row it gathers one row of f from HBM and runs cycle 0 on it,
// then cycle 1 on the row behind, cycle 2 on the row behind that, ...: cycle k
// takes row r - k from what cycle k - 1 left of rows r - k - 1, r - k and
// r - k + 1. The links along x come from the neighbouring lane (a DPP move, one
// per two nodes), those along y from registers that wait one or two rows. So
// nothing goes through LDS but the cells of the last C rows (each lane its
// own), and no wavefront waits for another.
//
// Against the tiles of the other passes (64 x 26 for four cycles) there is no
// ring above and below but at the ends of a strip's rows, so six cycles fit in a
// launch and fewer collisions are redundant: a strip's outer C columns on each
// side (128 / 116 for C = 6), and on average C - 1 rows at its ends.
//
// What bounds it: vector issue. At 8192^2 (FP32, Ergun medium, six cycles) a launch
// issues 7.5e8 vector instructions, 119 per node update with the redundant ones against
// 143 in the four-cycle tiles: 1.22 ms at 2.4 GHz, of the 1.30 that it takes, and a
// cycle moves 14 bytes per node instead of 20. 224 us per step against 294 (217 on
// another box). Two columns per lane and six cycles are what 168 registers hold
// (three wavefronts per SIMD); four cycles move a half more bytes and took 295 us, eight
// need two wavefronts per SIMD and a wider ring (272 us).
#pragma once

#include <type_traits>

#include "lbm_launch.h"

namespace mrt {

// Lane i's value in lane i + 1, and in lane i - 1 (0 comes in at the ends).
__device__ __forceinline__ float from_left(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x138, 0xf, 0xf, true));   // wave_shr:1
}
__device__ __forceinline__ float from_right(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x130, 0xf, 0xf, true));   // wave_shl:1
}

// A lane's two columns of one quantity.
struct Two {
    float a, b;
};

// The value that a pull along +x / -x brings: the left / right neighbour's.
__device__ __forceinline__ Two pull_right(const Two &v) { return Two{from_left(v.b), v.a}; }
__device__ __forceinline__ Two pull_left(const Two &v) { return Two{v.b, from_right(v.a)}; }

// A lane's two adjacent columns in memory, as loaded and as stored.
typedef unsigned int Uint2 __attribute__((ext_vector_type(2)));
typedef _Float16 Half2 __attribute__((ext_vector_type(2)));

// ODD: pairs may start on an odd element (an odd periodic width wraps to one),
// which only binary16 cares about: two words are loaded and shifted into place.
template <typename S, bool ODD> struct PairIO;
template <bool ODD> struct PairIO<float, ODD> {
    typedef Uint2 Raw;
    __device__ __forceinline__ static Raw ld(BufRes r, uint32_t col, uint32_t so) {
        return __builtin_amdgcn_raw_buffer_load_b64(r, (int)(col * 4), (int)so, 0);
    }
    __device__ __forceinline__ static Two get(Raw v, uint32_t) { return Two{__uint_as_float(v.x), __uint_as_float(v.y)}; }
    __device__ __forceinline__ static Raw put(const Two &v) {
        Raw u;
        u.x = __float_as_uint(v.a);
        u.y = __float_as_uint(v.b);
        return u;
    }
    template <int CPOL>
    __device__ __forceinline__ static void st(BufRes r, uint32_t vo, uint32_t so, const Two &v) {
        __builtin_amdgcn_raw_buffer_store_b64(put(v), r, (int)vo, (int)so, CPOL);
    }
};
template <bool ODD> struct PairIO<_Float16, ODD> {
    typedef std::conditional_t<ODD, Uint2, unsigned int> Raw;
    __device__ __forceinline__ static Raw ld(BufRes r, uint32_t col, uint32_t so) {
        if constexpr (ODD) return __builtin_amdgcn_raw_buffer_load_b64(r, (int)((col & ~1u) * 2), (int)so, 0);
        else return __builtin_amdgcn_raw_buffer_load_b32(r, (int)(col * 2), (int)so, 0);
    }
    __device__ __forceinline__ static Two get(Raw v, uint32_t col) {
        unsigned int u;
        if constexpr (ODD) u = __builtin_amdgcn_alignbit(v.y, v.x, (col & 1u) << 4);
        else u = v;
        Half2 h;
        __builtin_memcpy(&h, &u, 4);
        return Two{(float)h.x, (float)h.y};
    }
    template <int CPOL>
    __device__ __forceinline__ static void st(BufRes r, uint32_t vo, uint32_t so, const Two &v) {
        Half2 h;
        h.x = (_Float16)v.a;
        h.y = (_Float16)v.b;
        unsigned int u;
        __builtin_memcpy(&u, &h, 4);
        __builtin_amdgcn_raw_buffer_store_b32(u, r, (int)vo, (int)so, CPOL);
    }
};

constexpr int STRIP_COLS = 128;   // columns a wavefront holds
constexpr int STRIP_WAVES = 4;    // wavefronts (strips) per workgroup

// The columns [c0, c1) that strip k writes and the first one it holds. At a wall
// a strip has no ring on that side; across a periodic seam the ring wraps.
__host__ __device__ inline int strip_count(int nx, bool periodic, int C) {
    const int w = STRIP_COLS - 2 * C, e = STRIP_COLS - C;
    if (periodic) return (nx + w - 1) / w;
    if (nx <= STRIP_COLS) return 1;
    if (nx <= 2 * e) return 2;
    return 2 + (nx - 2 * e + w - 1) / w;
}
__host__ __device__ inline int strip_begin(int k, int nx, bool periodic, int C) {
    const int n = strip_count(nx, periodic, C);
    if (k <= 0) return 0;
    if (k >= n) return nx;
    int c = periodic ? k * (STRIP_COLS - 2 * C) : (STRIP_COLS - C) + (k - 1) * (STRIP_COLS - 2 * C);
    // the last strip is at least a ring wide, so that only its own ring crosses a seam
    if (k == n - 1) {
        const int m = (nx - C) & ~1;
        if (c > m) c = m;
    }
    return c;
}
__host__ __device__ inline int strip_first(int k, int nx, bool periodic, int C) {
    const int c = strip_begin(k, nx, periodic, C);
    if (!periodic) return k == 0 ? 0 : c - C;
    // a lane's two columns must not lie on two sides of the seam
    return c - C - ((k == strip_count(nx, periodic, C) - 1 && ((nx - c) & 1)) ? 1 : 0);
}

// What a cycle keeps of the rows of the cycle before it: links 0, 2, 1, 4, 5 of
// its next row as gathered, and links 1, 4, 5 of the newest row, which the row
// after that will pull.
struct StripHold {
    Two g0, g2, g1, g4, g5, r1, r4, r5;
};

template <typename S, int C, int MK, bool ODD, bool NT, bool LAST>
__global__ __launch_bounds__(64 * STRIP_WAVES) __attribute__((amdgpu_waves_per_eu(3))) void k_step4_strip(
    Dom d, StripPlan p) {
    constexpr int ES = (int)sizeof(S);
    // the cells of the last C rows: phi, 1/phi, cd/2, cf/2 of the lane's two columns
    constexpr bool CELLS = MK != MK_UNIFORM;
    __shared__ float4 cells[CELLS ? STRIP_WAVES * C * 2 * 64 : 1];
    const int lane = (int)threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int item = xcd_swizzle((int)blockIdx.x, (int)gridDim.x) * STRIP_WAVES + wv;
    if (item >= p.strips * p.chunks) return;
    const bool per_x = d.bc_x == BC_PERIODIC, per_y = d.bc_y == BC_PERIODIC;
    const int sk = item % p.strips, ck = item / p.strips;
    const int c0 = strip_begin(sk, d.nx, per_x, C), c1 = strip_begin(sk + 1, d.nx, per_x, C);
    const int xf = strip_first(sk, d.nx, per_x, C);
    const int y0 = (int)((int64_t)ck * d.ny / p.chunks), y1 = (int)((int64_t)(ck + 1) * d.ny / p.chunks);
    // the lane's columns; those beyond a wall hold whatever column 0 holds
    const int xa = xf + 2 * lane;
    int col = xa;
    if (per_x) col = xa < 0 ? xa + d.nx : (xa >= d.nx ? xa - d.nx : xa);
    else if (xa >= d.nx) col = 0;
    const bool ina = xa >= c0 && xa < c1, inb = xa + 1 >= c0 && xa + 1 < c1;
    // a strip whose columns pair up off their alignment, or that ends in half a pair
    const bool ragged = (xf & 1) != 0 || (c1 & 1) != 0;
    // next to an x wall
    const bool xw = !per_x && (sk == 0 || sk == p.strips - 1);
    const bool la = xw && xa == 0, ra = xw && xa == d.nx - 1, rb = xw && xa + 1 == d.nx - 1;

    const uint32_t fbytes = (uint32_t)(8 * d.plane * ES);
    const BufRes rin = buf_res(d.fin, fbytes), rout = buf_res(d.fout, fbytes);
    const MediumSrc<MK> med(d);
    const uint32_t pl = (uint32_t)(d.plane * ES), rowb = (uint32_t)(d.pitch * ES);
    // at x = 0 links 4 and 7 come from the own 6 and 5, at x = nx - 1 links 5 and 6 from 7 and 4
    const uint32_t vw1 = (uint32_t)(col * ES) + (la ? 6u : 7u) * pl + (rb ? (uint32_t)ES : 0u);
    const uint32_t vw2 = (uint32_t)(col * ES) + (la ? 5u : 4u) * pl + (rb ? (uint32_t)ES : 0u);

    typedef PairIO<S, ODD> IO;
    // one plane's row of the lane's columns
    auto row_two = [&](int plane, int y) -> typename IO::Raw {
        return IO::ld(rin, (uint32_t)col, (uint32_t)plane * pl + (uint32_t)y * rowb);
    };
    const int whi = per_y ? d.ny : 1 << 30;   // rows from here on wrap (selects, no branch)
    auto wrap_row = [&](int y) -> int {
        y = y < 0 && per_y ? y + d.ny : y;
        return y >= whi ? y - d.ny : y;
    };

    // f of row y as cycle 0 pulls it, not yet shifted along x, and the cells' inputs;
    // no branch between the loads and their use a row later, so they stay in flight
    struct Raw {
        typename IO::Raw f[8];
        float s1, s2;   // at an x wall: the own opposite of the links across it
        CellRaw ca, cb;
    };
    auto fetch = [&](auto plain, auto edge, int y, Raw &w) {
        const int yy = wrap_row(y), ym = wrap_row(y - 1), yp = wrap_row(y + 1);
        const bool bot = !plain.value && !per_y && y == 0, top = !plain.value && !per_y && y == d.ny - 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // across a y wall the node's own opposite link, which is not shifted
            const bool out = (EY[i] > 0 && bot) || (EY[i] < 0 && top);
            w.f[i] = row_two(out ? OPP[i] : i, out ? yy : (EY[i] > 0 ? ym : (EY[i] < 0 ? yp : yy)));
        }
        if (edge.value) {
            const uint32_t so = (uint32_t)yy * rowb;
            w.s1 = BufIO<S>::ld(rin, vw1, so);
            w.s2 = BufIO<S>::ld(rin, vw2, so);
        }
        const uint32_t so = (uint32_t)(yy * d.pitch * 4);
        if constexpr (MK == MK_ERGUN) {
            const Two p = PairIO<float, false>::get(PairIO<float, false>::ld(med.phi, (uint32_t)col, so), 0u);
            w.ca = CellRaw{p.a, 0.0f, 0.0f};
            w.cb = CellRaw{p.b, 0.0f, 0.0f};
        } else {
            w.ca = med.load(so + (uint32_t)col * 4);
            w.cb = med.load(so + (uint32_t)col * 4 + 4);
        }
    };

    // Stores: a lane whose two columns are another strip's aims beyond the buffer,
    // where a store is dropped. An edge strip (at an x wall, or whose columns end in
    // half a pair) stores column by column.
    constexpr uint32_t NOWHERE = 0xfffffff0u;
    const BufRes rup = buf_res(d.uprev, LAST ? (uint32_t)(2 * d.plane * 4) : 0u);
    const uint32_t va = ina ? (uint32_t)(col * ES) : NOWHERE, vb = inb ? (uint32_t)(col * ES + ES) : NOWHERE;
    const uint32_t ua = ina ? (uint32_t)(col * 4) : NOWHERE, ub = inb ? (uint32_t)(col * 4 + 4) : NOWHERE;
    auto st_up = [&](uint32_t so, const Two &u) {
        BufIO<float>::st_nt(rup, ua, so, u.a);
        BufIO<float>::st_nt(rup, ub, so, u.b);
    };

    // one cycle of the lane's two nodes of a row
    auto update = [&](Two (&f)[8], auto cell_a, auto cell_b, int k, int y) {
        float fa[8], fb[8], g[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f}, n7, n8, dT;
        Two ux, uy;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            fa[i] = f[i].a;
            fb[i] = f[i].b;
        }
        node_update<false>(d, cell_a(), fa, g, ux.a, uy.a, n7, n8, dT);
        __builtin_amdgcn_sched_barrier(0);
        node_update<false>(d, cell_b(), fb, g, ux.b, uy.b, n7, n8, dT);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = Two{(float)(S)fa[i], (float)(S)fb[i]};
        if (LAST && k == C - 1) {   // u(t - 1) of the residual
            const uint32_t so = (uint32_t)(y * d.pitch * 4);
            st_up(so, ux);
            st_up(so + (uint32_t)(d.plane * 4), uy);
        }
    };
    auto patch = [&](Two &v, const Two &own, bool pulls_right) {
        if (pulls_right) {
            v.a = la ? own.a : v.a;
        } else {
            v.a = ra ? own.a : v.a;
            v.b = rb ? own.b : v.b;
        }
    };

    StripHold H[C - 1];
    Raw w;
    // cycle 0 runs on rows [lo, hi), cycle k on a row less at each end that is no wall
    const int grow = C - 1;
    const int lo = per_y ? y0 - grow : (y0 - grow < 0 ? 0 : y0 - grow);
    const int hi = per_y ? y1 + grow : (y1 + grow > d.ny ? d.ny : y1 + grow);
    int slot = 0;   // of row r in the ring of cells

    // Row r through every cycle. FULL: each cycle has its row, none of them next to
    // a y wall, and there is a next row to fetch: the rows of a strip but the first
    // and last few, without a branch (over a branch the compiler sinks what only
    // the next row needs, as two operands instead of one result: 11 registers more
    // per cycle). EDGE: an edge strip.
    auto advance = [&](auto full, auto edge, int r) {
        constexpr bool FULL = decltype(full)::value, EDGE = decltype(edge)::value;
        Two f[8];
        bool made = FULL || r < hi;   // the cycle before made a row: f holds row r - k + 1
        // cycle 0, row r
        if (made) {
            const bool bot = !FULL && !per_y && r == 0, top = !FULL && !per_y && r == d.ny - 1;
            Two raw[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) raw[i] = IO::get(w.f[i], (uint32_t)col);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool out = (EY[i] > 0 && bot) || (EY[i] < 0 && top);
                f[i] = raw[i];
                if (!out) {
                    if (EX[i] > 0) f[i] = pull_right(raw[i]);
                    if (EX[i] < 0) f[i] = pull_left(raw[i]);
                }
                if (EY[i] < 0 && top) {
                    f[i].a = f[i].a + (float)EX[i] * d.lid6;
                    f[i].b = f[i].b + (float)EX[i] * d.lid6;
                }
            }
            if (EDGE) {
                patch(f[0], raw[2], true);
                patch(f[2], raw[0], false);
                const Two s1{w.s1, w.s1}, s2{w.s2, w.s2};
                if (!bot) {
                    patch(f[4], s1, true);
                    patch(f[5], s1, false);
                }
                if (!top) {
                    patch(f[6], s2, false);
                    patch(f[7], s2, true);
                }
            }
            const Cell ca = med.cell(d, w.ca), cb = med.cell(d, w.cb);
            if (CELLS) {
                float4 *q = cells + ((wv * C + slot) * 2) * 64 + lane;
                q[0] = make_float4(ca.phi, ca.inv_phi, ca.cdh, ca.cfh);
                q[64] = make_float4(cb.phi, cb.inv_phi, cb.cdh, cb.cfh);
            }
            update(f, [&] { return ca; }, [&] { return cb; }, 0, r);
            __builtin_amdgcn_sched_barrier(0);
        }
        // cycles 1 .. C - 1, each on the row behind the last one's
        int back = slot;
#pragma unroll
        for (int k = 1; k < C; ++k) {
            StripHold &h = H[k - 1];
            const int y = r - k;
            back = back == 0 ? C - 1 : back - 1;
            const int a = y0 - (grow - k), b = y1 + (grow - k);
            const bool act = FULL || (y >= (per_y ? a : (a < 0 ? 0 : a)) && y < (per_y ? b : (b > d.ny ? d.ny : b)));
            const bool top = !FULL && !per_y && y == d.ny - 1, bot = !FULL && !per_y && y == -1;
            Two in[8];
            if (act) {
                in[0] = h.g0;
                in[1] = h.g1;
                in[2] = h.g2;
                in[4] = h.g4;
                in[5] = h.g5;
                if (top) {
                    in[3] = h.r1;
                    in[6] = Two{h.r4.a - d.lid6, h.r4.b - d.lid6};
                    in[7] = Two{h.r5.a + d.lid6, h.r5.b + d.lid6};
                } else {
                    in[3] = f[3];
                    in[6] = pull_left(f[6]);
                    in[7] = pull_right(f[7]);
                    if (EDGE) {
                        patch(in[6], h.r4, false);
                        patch(in[7], h.r5, true);
                    }
                }
            }
            if (made) {
                // row y + 1 of the cycle before
                h.g0 = pull_right(f[0]);
                h.g2 = pull_left(f[2]);
                if (bot) {
                    h.g1 = f[3];
                    h.g4 = f[6];
                    h.g5 = f[7];
                } else {
                    h.g1 = h.r1;
                    h.g4 = pull_right(h.r4);
                    h.g5 = pull_left(h.r5);
                }
                if (EDGE) {
                    patch(h.g0, f[2], true);
                    patch(h.g2, f[0], false);
                    patch(h.g4, f[6], true);
                    patch(h.g5, f[7], false);
                }
                h.r1 = f[1];
                h.r4 = f[4];
                h.r5 = f[5];
            }
            made = act;
            if (act) {
                auto kept = [&](int col) -> Cell {
                    if (!CELLS) return med.cell(d, CellRaw{0.0f, 0.0f, 0.0f});
                    const float4 u = cells[((wv * C + back) * 2 + col) * 64 + lane];
                    Cell c;
                    c.phi = u.x;
                    c.inv_phi = u.y;
                    c.cdh = u.z;
                    c.cfh = u.w;
                    c.s_nu = d.s_nu;
                    c.h_nu2 = d.h_nu2;
                    c.h_nu4 = d.h_nu4;
                    return c;
                };
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = in[i];
                update(f, [&] { return kept(0); }, [&] { return kept(1); }, k, y);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // The next row's loads go out before this row's stores (a wait for them waits
        // for no store), and only here: the registers they need are free between the
        // collisions, and the other wavefronts' rows cover their latency.
        if (FULL || r + 1 < hi) fetch(full, edge, r + 1, w);
        if (made) {
            const int y = r - grow;
            const uint32_t so = (uint32_t)y * rowb;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t o = so + (uint32_t)i * pl;
                if (!EDGE) {
                    IO::template st<NT ? CPOL_NT : 0>(rout, va, o, f[i]);
                } else if (NT) {
                    BufIO<S>::st_nt(rout, va, o, f[i].a);
                    BufIO<S>::st_nt(rout, vb, o, f[i].b);
                } else {
                    BufIO<S>::st(rout, va, o, f[i].a);
                    BufIO<S>::st(rout, vb, o, f[i].b);
                }
            }
        }
        slot = slot + 1 == C ? 0 : slot + 1;
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    const int end = y1 + grow;
    int full0 = y0 + grow, full1 = end - 1;   // the rows that are FULL
    if (!per_y && full1 > d.ny - 2) full1 = d.ny - 2;
    int r = lo;
    if (xw || ragged) {
        fetch(no, yes, lo, w);
        for (; r < full0 && r < end; ++r) advance(no, yes, r);
        for (; r + 2 < full1; r += 3) {
            advance(yes, yes, r);
            advance(yes, yes, r + 1);
            advance(yes, yes, r + 2);
        }
        for (; r < end; ++r) advance(no, yes, r);
    } else {
        fetch(no, no, lo, w);
        for (; r < full0 && r < end; ++r) advance(no, no, r);
        // three rows per turn: a link's value moves from register to register with a
        // period of three, so the copies at the end of a turn fall to a third
        for (; r + 2 < full1; r += 3) {
            advance(yes, no, r);
            advance(yes, no, r + 1);
            advance(yes, no, r + 2);
        }
        for (; r < end; ++r) advance(no, no, r);
    }
}

template <typename S, int C, int MK, bool ODD>
static const void *strip_fn_t(bool nt, bool last) {
    if (nt) return last ? (const void *)&k_step4_strip<S, C, MK, ODD, true, true> : (const void *)&k_step4_strip<S, C, MK, ODD, true, false>;
    return last ? (const void *)&k_step4_strip<S, C, MK, ODD, false, true> : (const void *)&k_step4_strip<S, C, MK, ODD, false, false>;
}

template <typename S, int C>
static const void *strip_fn_c(const Dom &d) {
    const bool odd = sizeof(S) == 2 && d.bc_x == BC_PERIODIC && (d.nx & 1), nt = d.nt_store != 0, last = d.uprev != nullptr;
    switch (medium_kind(d)) {
    case MK_ERGUN:
        if constexpr (sizeof(S) == 2)
            if (odd) return strip_fn_t<S, C, MK_ERGUN, true>(nt, last);
        return strip_fn_t<S, C, MK_ERGUN, false>(nt, last);
    case MK_UNIFORM:   // (four cycles go through tiles)
        if constexpr (C == 6) {
            if constexpr (sizeof(S) == 2)
                if (odd) return strip_fn_t<S, C, MK_UNIFORM, true>(nt, last);
            return strip_fn_t<S, C, MK_UNIFORM, false>(nt, last);
        }
        return nullptr;
    default: return nullptr;
    }
}

// Where the strip pass is taken, unless the rolling pass (lbm_roll.h) is (us per step
// in 48-step calls, the tile passes' default against the strip pass, one box): log-normal channels in FP32 from 2^22
// nodes (2048^2 23.5 against 20.1, 3000^2 46.8 against 37.9, 4096^2 81 against 65,
// 8192^2 294 against 224; 1750^2 15.2 against 15.7); binary16 storage, whose tile
// passes move half the bytes, from 9 x 2^20 (channel 3801 x 3001 46.8 against 44.3,
// 8191^2 256 against 212; 3001 x 3000 36.4 against 36.6, 2576 x 2614 27.5 against 28.7,
// 2575 x 2614, whose pairs wrap onto odd columns, 29.1 against 32.3), in uniform media
// from 2^24 (cavity 4096^2 61.2 against 61.0, 8192^2 233 against 213; 3700^2 49.8
// against 51.1, 2575 x 2615 25.2 against 29.0); uniform media in FP32, where
// the tiles load no porosity, from 2^23, where these passes take four cycles too
// (cavity 4096^2 63.4 against 60.9, 8192^2 243 against 227; 2048^2 17.2 against
// 19.9); and where at least three quarters of the strips' lanes are columns of
// the domain. Media with a 1/K or a viscosity plane keep the tiles.
bool strip_domain(const Dom &d, int storage) {
    const int mk = medium_kind(d);
    const bool per_x = d.bc_x == BC_PERIODIC;
    if (d.thermal || mk == MK_ANY || d.bc_x == BC_NEE || d.bc_y == BC_NEE) return false;
    const int64_t M = (int64_t)1 << 20;
    const int64_t least = storage == ST_F16 ? (mk == MK_ERGUN ? 9 : 16) * M : (mk == MK_ERGUN ? 4 : 8) * M;
    if ((int64_t)d.nx * d.ny < least || d.ny < 64 || (per_x && d.nx < 2 * STRIP_COLS)) return false;
    return 4 * (int64_t)d.nx >= 3 * (int64_t)STRIP_COLS * strip_count(d.nx, per_x, 6);
}

// Cycles of the next pass with n left (6: strips; 4: strips or tiles, whichever the caller
// finds faster; 1 to 3: tiles): sixes, and fours and a three where they come out even.
int strip_cycles(int64_t n) {
    static const int next[12] = {0, 1, 2, 3, 4, 3, 6, 4, 4, 6, 6, 4};
    return n >= 12 ? 6 : next[n];
}

// One round of wavefronts, three per SIMD (what 168 registers allow), and from 128
// rows a wavefront more and shorter rounds: 8192^2 in one round 231 us per step, in
// two 224 (2048^2, 4096^2: 20.1 and 65 in one, 25.8 and 67 in two).
static int strip_chunks(const Dom &d, int strips) {
    constexpr int WAVES = 256 * 4 * 3;
    int chunks = WAVES / strips < 1 ? 1 : WAVES / strips;
    while (d.ny / (2 * chunks) >= 64) chunks *= 2;
    return chunks > d.ny ? d.ny : chunks;
}

hipError_t launch_step_strip(const Dom &d, int storage, int cycles, hipStream_t st) {
    const void *fn = nullptr;
    if (cycles == 4) fn = storage == ST_F32 ? strip_fn_c<float, 4>(d) : strip_fn_c<_Float16, 4>(d);
    if (cycles == 6) fn = storage == ST_F32 ? strip_fn_c<float, 6>(d) : strip_fn_c<_Float16, 6>(d);
    if (!fn || !strip_domain(d, storage)) return hipErrorInvalidValue;
    Dom dd = d;
    StripPlan p{strip_count(d.nx, d.bc_x == BC_PERIODIC, cycles), 0};
    p.chunks = strip_chunks(d, p.strips);
    const int wgs = (p.strips * p.chunks + STRIP_WAVES - 1) / STRIP_WAVES;
    void *args[2] = {&dd, &p};
    return hipLaunchKernel(fn, dim3((unsigned)wgs), dim3(64 * STRIP_WAVES), args, 0, st);
}

}  // namespace mrt
