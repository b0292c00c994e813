// Two time steps of a small tile in one launch (FP64 and FP32 storage).
//
// A case too small to fill the device is bound by the launch and by the
// latencies of one step: load, barrier, collide, store.  Here a workgroup
// keeps its tile (OZ x OR nodes) and a halo in LDS, and a launch pays for two
// steps at once:
//   phi(t) on the tile and 5 cells around it, f pulled from memory
//   step 1 on the tile and 3 cells around it, post-collision values to LDS
//   phi(t+1) on the tile and 2 cells around it, f pulled from LDS
//   step 2 on the tile, stored
// Each phase deals its own cells out over the threads, densely.  Every node is
// advanced by the operations of tile_step, in the same order, so the results
// are the same bits.  Nothing branches on a lane: cells outside the grid or
// beyond a phase's last write to a spare cell of the LDS arrays, read any, and
// load from, or drop their stores to, a clamped place (see axi_pair.hpp for
// why).  With one or two wavefronts per SIMD it is the length of the serial
// instruction stream that counts, so the sizes are compile-time constants:
// the same code with sizes known only at run time took 8.0 us a launch on
// 64 x 128 nodes in FP32 (divisions, and an address sum per LDS access).
#pragma once

#include "axi_pair.hpp"

namespace axi {

template <int OZ_, int OR_, int THREADS_>
struct TileShape {
    static constexpr int OZ = OZ_, OR = OR_, THREADS = THREADS_;
    static constexpr int PZ = OZ + 10, PR = OR + 10, NP = PZ * PR;     // phi(t)
    static constexpr int DZ = OZ + 6, DR = OR + 6, ND = DZ * DR;       // step 1
    static constexpr int EZ = OZ + 4, ER = OR + 4, NE = EZ * ER;       // phi(t + 1)
    static constexpr int NO = OZ * OR;
    static constexpr int LDS_VALUES = 18 * (ND + 1) + (NP + 1) + 3 * (NO + 1);
    static_assert(NO <= THREADS, "one node of step 2 per thread");
};

template <typename T, typename R, int MODE, typename S>
__device__ __forceinline__ void tile_two_steps(const Geom &g, const Phys<R> &P0, R gz1, int tz, int tr,
                                               const T *__restrict__ fin, const T *__restrict__ gin,
                                               const T *__restrict__ ain, T *__restrict__ fout, T *__restrict__ gout,
                                               T *__restrict__ aout, R *lds)
{
    constexpr int NT = S::THREADS, QA = (S::NP + NT - 1) / NT, QB = (S::ND + NT - 1) / NT;
    constexpr int DS = S::ND + 1, OS = S::NO + 1;  // values between the planes of `post` and `prev`
    R *const post = lds, *const phi = post + 18 * DS, *const prev = phi + S::NP + 1;
    const int tid = threadIdx.x;
    const int nr = g.nr, nz = g.nz;
    const int k0 = tz * S::OZ, j0 = tr * S::OR;
    // every pull and stencil of the tile is plain (uniform): with periodic z
    // only columns wrap
    const bool plain = j0 >= 6 && j0 + S::OR + 6 <= nr && (g.zper || (k0 >= 6 && k0 + S::OZ + 6 <= nz));
    const bool wraps = g.zper && (k0 < 6 || k0 + S::OZ + 6 > nz);                  // uniform

    const Pitch pt = pitch_of<T>(g);
    const __amdgpu_buffer_rsrc_t fr = raw_rsrc(fin), gr = raw_rsrc(gin), ar = raw_rsrc(ain);
    const __amdgpu_buffer_rsrc_t fo = bound_rsrc(fout, 9 * pt.plane), go = bound_rsrc(gout, 9 * pt.plane),
                                 ao = bound_rsrc(aout, 3 * pt.plane);

    // cell n of a frame of width W that begins h cells before the tile (from
    // NC on, cell 0 again): its place (z, r), its node (kl, jl) and whether
    // that is in the grid
    struct Cell {
        int z, r, kl, jl;
        bool in;
    };
    auto cell = [&](auto width, auto count, int h, int n) {
        constexpr int W = decltype(width)::value, NC = decltype(count)::value;
        Cell e;
        const bool last = n >= NC;
        n = last ? 0 : n;
        e.r = n / W;
        e.z = n - e.r * W;
        e.kl = k0 - h + e.z;
        e.jl = j0 - h + e.r;
        e.in = !last;
        if (!plain) e.in = e.in && e.jl >= 0 && e.jl < nr && (g.zper || (e.kl >= 0 && e.kl < nz));
        return e;
    };
    // the column and row a cell's loads come from
    auto source = [&](const Cell &e, int &c, int &j) {
        j = e.jl;
        c = e.kl;
        if (!plain) {
            j = j < 0 ? 0 : (j >= nr ? nr - 1 : j);
            if (!g.zper) c = c < 0 ? 0 : (c >= nz ? nz - 1 : c);
        }
        if (wraps) {
            c %= nz;
            c = c < 0 ? c + nz : c;
        }
    };
    auto pull = [&](const __amdgpu_buffer_rsrc_t &r, const T *base, int c, int j, R(&v)[9]) {
        const uint32_t off = (uint32_t)(j * nz + c) * (uint32_t)sizeof(T);
        if (!plain)
            pull9_bc<T, R>((const char *)base, g, pt, c, j, v);
        else if (wraps)
            pull9_buf<T, R, 0>(r, pt, col_off<true>(off, c, g, sizeof(T)), v);
        else
            pull9_buf<T, R, 0>(r, pt, col_off<false>(off, c, g, sizeof(T)), v);
    };
    using IntPZ = std::integral_constant<int, S::PZ>;
    using IntNP = std::integral_constant<int, S::NP>;
    using IntDZ = std::integral_constant<int, S::DZ>;
    using IntND = std::integral_constant<int, S::ND>;
    using IntEZ = std::integral_constant<int, S::EZ>;
    using IntNE = std::integral_constant<int, S::NE>;
    using IntOZ = std::integral_constant<int, S::OZ>;
    using IntNO = std::integral_constant<int, S::NO>;

    // ---- loads: f of phi's cells, g and aux of step 1's cells
    R fa[QA][9], gb[QB][9], ab[QB][3], ira[QA];
    int pa[QA], da[QA];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
        const Cell e = cell(IntPZ{}, IntNP{}, 5, tid + q * NT);
        int c, j;
        source(e, c, j);
        ira[q] = inv_radius<R>(j);
        pa[q] = e.in ? e.r * S::PZ + e.z : S::NP;
        da[q] = e.in && e.z >= 2 && e.z < S::PZ - 2 && e.r >= 2 && e.r < S::PR - 2 ? (e.r - 2) * S::DZ + (e.z - 2) : S::ND;
        pull(fr, fin, c, j, fa[q]);
    }
    Cell eb[QB];
    int ib[QB];                                    // their places in `post`
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        eb[q] = cell(IntDZ{}, IntND{}, 3, tid + q * NT);
        ib[q] = eb[q].in ? tid + q * NT : S::ND;
        int c, j;
        source(eb[q], c, j);
        pull(gr, gin, c, j, gb[q]);
        const uint32_t off = (uint32_t)(j * nz + c) * (uint32_t)sizeof(T);
        ab[q][0] = (R)buf_load<T, 0>(ar, off, 0);
        ab[q][1] = (R)buf_load<T, 0>(ar, off, pt.plane);
        ab[q][2] = (R)buf_load<T, 0>(ar, off, 2 * pt.plane);
    }
    // ---- phi(t); f of step 1's cells goes to them through `post`
#pragma unroll
    for (int q = 0; q < QA; ++q) {
        phi[pa[q]] = sum9(fa[q]) * ira[q];
#pragma unroll
        for (int i = 0; i < 9; ++i) post[i * DS + da[q]] = fa[q][i];
    }
    lds_barrier();

    // stencil around a cell at place (z, r) of phi's frame
    auto stencil = [&](const Cell &e, int z, int r, Stencil<R> &s) {
        if (plain) {
            const R *o = phi + r * S::PZ + z;
            s.c = o[0]; s.e = o[1]; s.w = o[-1]; s.ee = o[2]; s.ww = o[-2];
            s.n = o[S::PZ]; s.ne = o[S::PZ + 1]; s.nw = o[S::PZ - 1];
            s.s = o[-S::PZ]; s.se = o[1 - S::PZ]; s.sw = o[-1 - S::PZ];
            s.nn = o[2 * S::PZ]; s.nne = o[2 * S::PZ + 2]; s.nnw = o[2 * S::PZ - 2];
            s.ss = o[-2 * S::PZ]; s.sse = o[2 - 2 * S::PZ]; s.ssw = o[-2 - 2 * S::PZ];
            return;
        }
        // ghost cells (Sec. 2.3); a cell that does not count reads its frame as it is
        int row[5], col[5];
#pragma unroll
        for (int d = -2; d <= 2; ++d) {
            row[d + 2] = (r + (e.in ? ghost_row(e.jl + d, nr) - e.jl : d)) * S::PZ;
            col[d + 2] = z + (e.in && !g.zper ? ghost_col(e.kl + d, nz, 0) - e.kl : d);
        }
        auto at = [&](int b, int a) { return phi[row[b + 2] + col[a + 2]]; };
        s.c = at(0, 0); s.e = at(0, 1); s.w = at(0, -1); s.ee = at(0, 2); s.ww = at(0, -2);
        s.n = at(1, 0); s.ne = at(1, 1); s.nw = at(1, -1);
        s.s = at(-1, 0); s.se = at(-1, 1); s.sw = at(-1, -1);
        s.nn = at(2, 0); s.nne = at(2, 2); s.nnw = at(2, -2);
        s.ss = at(-2, 0); s.sse = at(-2, 2); s.ssw = at(-2, -2);
    };

    // ---- step 1
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        const Cell &e = eb[q];
        R fv[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) fv[i] = post[i * DS + ib[q]];
        Stencil<R> st;
        stencil(e, e.z + 2, e.r + 2, st);
        const int j = plain ? e.jl : (e.jl < 0 ? 0 : e.jl);
        const R r = (R)j + (R)0.5, ir = inv_radius<R>(j);
        Macro<R> m;
        macro_state<MODE>(P0, r, ir, st, gb[q], ab[q][1], ab[q][2], m);
        collide_node<MODE>(P0, r, ir, m, ab[q][0], ab[q][1], ab[q][2], fv, gb[q]);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            post[i * DS + ib[q]] = fv[i];
            post[(9 + i) * DS + ib[q]] = gb[q][i];
        }
        const int z = e.z - 3, rr = e.r - 3;
        const int o = e.in && z >= 0 && z < S::OZ && rr >= 0 && rr < S::OR ? rr * S::OZ + z : S::NO;
        prev[o] = m.phi;
        prev[OS + o] = m.uz;
        prev[2 * OS + o] = m.ur;
    }
    lds_barrier();

    // populations that a node at place d of `post` pulls from there (q: 0 for
    // f, 9 for g; the rules of pull_slot; d is never at the frame's edge)
    auto pull_post = [&](auto group, int d, const Cell &e, R(&v)[9]) {
        constexpr int q = decltype(group)::value;
        auto one = [&](auto link) {
            constexpr int I = decltype(link)::value, CZ = link_z(I), CR = link_r(I);
            if (plain) {
                v[I] = post[d + ((q + I) * DS - CZ - CR * S::DZ)];
                return;
            }
            int n = (q + I) * DS - CZ - CR * S::DZ;
            if (CR > 0) n = e.jl == 0 ? (q + axis_image(I)) * DS - CZ : n;
            bool wall = false;
            if (CZ > 0) wall = !g.zper && e.kl == 0;
            if (CZ < 0) wall = !g.zper && e.kl == nz - 1;
            if (CR < 0) wall = wall || e.jl == nr - 1;
            n = wall ? (q + reverse_link(I)) * DS : n;
            v[I] = post[d + n];
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{});
        one(std::integral_constant<int, 7>{});
        one(std::integral_constant<int, 8>{});
    };
    using F = std::integral_constant<int, 0>;
    using G = std::integral_constant<int, 9>;

    // ---- phi(t + 1); what step 2 pulls
#pragma unroll
    for (int q = 0; q < (S::NE + NT - 1) / NT; ++q) {
        const Cell e = cell(IntEZ{}, IntNE{}, 2, tid + q * NT);
        R v[9];
        pull_post(F{}, (e.r + 1) * S::DZ + e.z + 1, e, v);
        const int j = plain ? e.jl : (e.jl < 0 ? 0 : e.jl);
        phi[e.in ? (e.r + 3) * S::PZ + e.z + 3 : S::NP] = sum9(v) * inv_radius<R>(j);
    }
    const Cell e = cell(IntOZ{}, IntNO{}, 0, tid);
    R fv[9], gv[9];
    {
        const int d = (e.r + 3) * S::DZ + e.z + 3;
        pull_post(F{}, d, e, fv);
        pull_post(G{}, d, e, gv);
    }
    const int o = e.r * S::OZ + e.z;
    const R php = prev[o], uzp = prev[OS + o], urp = prev[2 * OS + o];
    lds_barrier();

    // ---- step 2
    Stencil<R> st;
    stencil(e, e.z + 5, e.r + 5, st);
    Phys<R> P1 = P0;
    P1.g_z = gz1;
    const R r = (R)e.jl + (R)0.5, ir = inv_radius<R>(e.jl);
    Macro<R> m;
    macro_state<MODE>(P1, r, ir, st, gv, uzp, urp, m);
    collide_node<MODE>(P1, r, ir, m, php, uzp, urp, fv, gv);
    const uint32_t so = e.in && e.kl < nz ? (uint32_t)(e.jl * nz + e.kl) * (uint32_t)sizeof(T) : 0xfffffff0u;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        buf_store<0>((T)fv[i], fo, so, (uint32_t)i * pt.plane);
        buf_store<0>((T)gv[i], go, so, (uint32_t)i * pt.plane);
    }
    buf_store<0>((T)m.phi, ao, so, 0);
    buf_store<0>((T)m.uz, ao, so, pt.plane);
    buf_store<0>((T)m.ur, ao, so, 2 * pt.plane);
}

// The shapes there are (two_step_plan picks by size).
using Tile8x4 = TileShape<8, 4, 256>;
using Tile12x8 = TileShape<12, 8, 256>;
using Tile16x16 = TileShape<16, 16, 512>;
using Tile32x16 = TileShape<32, 16, 512>;
constexpr int TILE_SHAPES = 4;

// fn(shape) for shape number t
template <typename F>
inline void with_tile_shape(int t, F &&fn)
{
    switch (t) {
    case 0: fn(Tile8x4{}); break;
    case 1: fn(Tile12x8{}); break;
    case 2: fn(Tile16x16{}); break;
    default: fn(Tile32x16{}); break;
    }
}

} // namespace axi
