// Two time steps in one pass over memory (FP64 and FP32 storage).
//
// One step moves every population and aux value through HBM once each way,
// and that traffic bounds large cases (336 / 168 bytes per node and step, at
// 0.86 of a plain copy's bandwidth).  Two steps fused move it once for both.
// A workgroup owns a strip of columns (one per lane) and marches up a run of
// rows, holding what the second step needs of the last few rows in registers
// and LDS:
//   iteration J: step 1 of row J       phi(t) of rows J-2..J+2 from LDS
//      barrier   row J-1 pulled        its populations at t+1 are complete now
//                phi(t+1) of row J-1   to LDS
//                phi(t) of row J+3     to LDS, from loads an iteration old
//      barrier   step 2 of row J-3     phi(t+1) of rows J-5..J-1 from LDS; stored
// Step 1 leaves populations in registers; they reach the neighbouring lane by
// a DPP shift, and across wavefronts through LDS.  Only phi and those edges
// are shared.  Held back are, per lane, what the collision takes (Pre: 5 + 6
// moments instead of 18 populations where every free rate is 1).
// Reach: phi(t) is pulled from memory on every lane l of L, step 1 is right on
// lanes 2..L-3, the populations at t+1 on 3..L-4, step 2 on 5..L-6
// (PAIR_HALO); a run recomputes 3 rows of step 1 beyond each of its ends.
// Every node is advanced by the operations of tile_step, in the same order,
// so the results are the same bits.
// Nothing here branches on a lane: what only some lanes write, the others
// write to a spare cell.  (With this many live registers the compiler split
// live ranges by copies at the joins of such branches, ahead of the
// instruction that restores the lanes: lanes that had skipped the branch kept
// old values.)
//
// Measured, us per step, one step per launch -> two (best tile each):
//   64 cases 256 x 512 FP32      249.5 -> 154.5 (1.48 GB moved per step at 6.0
//                                TB/s -> per two steps at 4.8)
//   32 cases 256 x 512 FP64      250.6 -> 165.5
//   one case 700 x 2000 FP32      50.7 -> 31.5
// What bounds it now: vector instructions issue two thirds of the time (FP32),
// at a clock that power holds at 2.0 to 2.1 of 2.4 GHz, beside the ~40 memory
// streams; FP64 runs one wavefront per SIMD (LDS, registers).
#pragma once

#include "axi_device.hpp"

namespace axi {

constexpr int PAIR_HALO = 5;         // lanes lost on each side of a strip
// cache policy of the stores: the default, so that L2 puts the halves of a line
// that two strips write together (nt sc1: 40 cases of 200 x 500 FP32 143 us a
// step against 85.6, 32 of 256 x 512 FP64 208 against 165; with one strip to a
// case, 64 of 256 x 512 FP32, 154.8 against 154.5)
constexpr int PAIR_STORE = 0;
// most wavefronts of a workgroup (FP32 by LDS; FP64: four measured slower than two)
template <typename R>
constexpr int PAIR_WAVES = sizeof(R) == 8 ? 2 : 8;

// lane i takes the value of lane i - 1 (from_left) or i + 1 (from_right) of its
// wavefront; the lane at the end takes its own `edge`
__device__ __forceinline__ uint32_t dpp_left(uint32_t v, uint32_t edge)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t dpp_right(uint32_t v, uint32_t edge)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ float from_left(float v, float e)
{
    return __builtin_bit_cast(float, dpp_left(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, e)));
}
__device__ __forceinline__ float from_right(float v, float e)
{
    return __builtin_bit_cast(float, dpp_right(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, e)));
}
__device__ __forceinline__ double from_left(double v, double e)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, v), b = __builtin_bit_cast(uint64_t, e);
    return __builtin_bit_cast(double, ((uint64_t)dpp_left((uint32_t)(a >> 32), (uint32_t)(b >> 32)) << 32) |
                                          dpp_left((uint32_t)a, (uint32_t)b));
}
__device__ __forceinline__ double from_right(double v, double e)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, v), b = __builtin_bit_cast(uint64_t, e);
    return __builtin_bit_cast(double, ((uint64_t)dpp_right((uint32_t)(a >> 32), (uint32_t)(b >> 32)) << 32) |
                                          dpp_right((uint32_t)a, (uint32_t)b));
}

// a wave-uniform value moved to scalar registers
__device__ __forceinline__ float uniform(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ uint32_t scalar(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// raw_rsrc with the record count that bounds the accesses
__device__ __forceinline__ __amdgpu_buffer_rsrc_t bound_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
}

// barrier of the workgroup that orders its LDS accesses (and no other memory)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS of one wavefront: rings of rows that a lane writes and reads back
// itself, and what its end lanes hand to the neighbouring wavefronts
template <typename R, int MODE>
struct PairWave {
    static constexpr int NF = Pre<MODE, R>::NF, NG = Pre<MODE, R>::NG;
    R aux[3][2][64];       // u_z, u_r of step 1, for step 2: row j in slot j % 3
    R fh[2][NF][64];       // Pre of f at t, rows J and J + 1
    R h[2][NF + NG][64];   // Pre of f and g at t + 1, rows J - 3 and J - 2
    R right[2][4], left[2][4];   // f, g: links 1, 5, 8 of lane 63; links 3, 6, 7 of lane 0
    R spare[2][4];               // where the other lanes write
};

// LDS bytes of a workgroup of nw wavefronts: their PairWave, then phi(t) and
// phi(t + 1) of the last five rows (row j in slot j % 5, lane l of the
// workgroup in cell l + 2, two ghost cells at either end and a spare one)
__host__ __device__ constexpr int pair_pitch(int nw) { return 64 * nw + 6; }
template <typename R, int MODE>
__host__ __device__ constexpr int pair_lds_bytes(int nw)
{
    return nw * (int)sizeof(PairWave<R, MODE>) + 2 * 5 * pair_pitch(nw) * (int)sizeof(R);
}

// One strip of a workgroup of nw wavefronts: lane l stands for column kb + l;
// it stores the columns k0 .. k1 - 1 of rows ra .. rb - 1 after two steps.  P0
// holds the rates, gz1 the acceleration of the second step.  ZWALL: the lanes
// reach a z wall.  full: the strip is the whole period, its ends neighbours.
template <typename T, typename R, int MODE, bool ZWALL>
__device__ __forceinline__ void pair_march(const Geom &g, const Phys<R> &P0, R gz1, int nw, int kb, int k0, int k1,
                                           bool full, int ra, int rb, const T *__restrict__ fin,
                                           const T *__restrict__ gin, const T *__restrict__ ain, T *__restrict__ fout,
                                           T *__restrict__ gout, T *__restrict__ aout, char *lds)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    PairWave<R, MODE> *const waves = (PairWave<R, MODE> *)lds;
    PairWave<R, MODE> &S = waves[wv];
    const PairWave<R, MODE> &Sl = waves[wv > 0 ? wv - 1 : (full ? nw - 1 : 0)];
    const PairWave<R, MODE> &Sr = waves[wv < nw - 1 ? wv + 1 : (full ? 0 : wv)];
    const int pitch = pair_pitch(nw);
    R(*const to_right)[4] = lane == 63 ? S.right : S.spare;
    R(*const to_left)[4] = lane == 0 ? S.left : S.spare;
    R *const phi_t = (R *)(lds + nw * sizeof(PairWave<R, MODE>)), *const phi_t1 = phi_t + 5 * pitch;

    const int nr = g.nr, nz = g.nz;
    // the lane's column: wrapped with periodic z, else clamped (lanes beyond a
    // wall stand for nothing: no lane inside reads them)
    const int kl = kb + tid;
    int c;
    if (g.zper) {
        c = kl % nz;
        c = c < 0 ? c + nz : c;
    } else {
        c = kl < 0 ? 0 : (kl >= nz ? nz - 1 : kl);
    }
    const bool at_lo = ZWALL && kl == 0, at_hi = ZWALL && kl == nz - 1;
    // where the lane stores: lanes with no column of their own use an offset
    // beyond the buffers, whose stores the hardware drops (a branch around the
    // stores would make the next wait for loads wait for them as well)
    const uint32_t so = kl >= k0 && kl < k1 ? (uint32_t)c * (uint32_t)sizeof(T) : 0xfffffff0u;

    const Pitch pt = pitch_of<T>(g);
    // the column's byte offset, and with its neighbours' one row further on, so
    // that none is negative: the pulls take one row off their scalar offset
    const uint32_t cb = (uint32_t)c * (uint32_t)sizeof(T);
    const ColOff co = col_off<true>(cb + pt.row, c, g, sizeof(T));
    const __amdgpu_buffer_rsrc_t fr = raw_rsrc(fin), gr = raw_rsrc(gin), ar = raw_rsrc(ain);
    const __amdgpu_buffer_rsrc_t fo = bound_rsrc(fout, 9 * pt.plane), go = bound_rsrc(gout, 9 * pt.plane),
                                 ao = bound_rsrc(aout, 3 * pt.plane);
    // at the z walls, per link: plane, column shift or the node's own reversed
    // population (plane and row shift cannot stay in the scalar offset)
    uint32_t wo[9];
    auto wall_off = [&](auto link) {
        constexpr int I = decltype(link)::value;
        const bool back = link_z(I) > 0 ? at_lo : (link_z(I) < 0 ? at_hi : false);
        return back ? cb + pt.row + (uint32_t)reverse_link(I) * pt.plane : cb + pt.row + link_offset<I, T>(pt);
    };
    if constexpr (ZWALL) {
        wo[1] = wall_off(std::integral_constant<int, 1>{});
        wo[3] = wall_off(std::integral_constant<int, 3>{});
        wo[5] = wall_off(std::integral_constant<int, 5>{});
        wo[6] = wall_off(std::integral_constant<int, 6>{});
        wo[7] = wall_off(std::integral_constant<int, 7>{});
        wo[8] = wall_off(std::integral_constant<int, 8>{});
    }

    const int lo1 = ra - 3 < 0 ? 0 : ra - 3, hi1 = rb + 2 < nr - 1 ? rb + 2 : nr - 1;      // step 1
    const int ilo = ra - 2 < 0 ? 0 : ra - 2, ihi = rb + 1 < nr - 1 ? rb + 1 : nr - 1;      // pulled at t + 1
    const int phi_hi = hi1 + 2 < nr - 1 ? hi1 + 2 : nr - 1;                                // phi(t)

    // the nine pulls of a row; inner: a row known to be clear of the axis and
    // the r-wall (no branch, whose merge would wait for the loads)
    auto pull_row = [&](auto inner, const __amdgpu_buffer_rsrc_t &r, const T *base, int row, R(&v)[9]) {
        if (decltype(inner)::value || (row >= 1 && row <= nr - 2)) {
            const uint32_t ro = scalar((uint32_t)(row - 1) * pt.row);
            auto one = [&](auto link) {
                constexpr int I = decltype(link)::value;
                if constexpr (ZWALL && link_z(I) != 0)
                    v[I] = (R)buf_load<T, 0>(r, wo[I], ro);
                else
                    v[I] = (R)buf_load<T, 0>(r, link_voff<I>(co), ro + link_offset<I, T>(pt));
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
        } else {
            pull9_bc<T, R>((const char *)base, g, pt, c, row, v);
        }
    };
    auto load_aux = [&](int row, R(&v)[3]) {
        const uint32_t ro = scalar((uint32_t)row * pt.row);
        v[0] = (R)buf_load<T, 0>(ar, cb, ro);
        v[1] = (R)buf_load<T, 0>(ar, cb, ro + pt.plane);
        v[2] = (R)buf_load<T, 0>(ar, cb, ro + 2 * pt.plane);
    };
    // where the lane's phi goes in a row of a ring, and where once more: the
    // mirrored ghost cells of a wall (Sec. 2.3), the two columns beyond either
    // end of a whole period, else its own cell again
    int cell = tid + 2, ghost = cell;
    if (ZWALL) {
        if (kl < 0 || kl >= nz) cell = 64 * nw + 4;
        ghost = kl == 0 ? cell - 1 : (kl == 1 && tid > 0 ? cell - 3 : cell);
        ghost = kl == nz - 1 ? cell + 1 : (kl == nz - 2 && tid < 64 * nw - 1 ? cell + 3 : ghost);
    } else if (full) {
        ghost = tid < 2 ? cell + 64 * nw : (tid >= 64 * nw - 2 ? cell - 64 * nw : cell);
    }
    auto put_phi = [&](R *ring, int row, R v) {
        R *slot = ring + (unsigned)row % 5u * pitch;
        slot[cell] = v;
        if (ZWALL || full) slot[ghost] = v;
    };
    auto get_stencil = [&](const R *ring, int row, Stencil<R> &s) {
        const R *own = ring + tid + 2;
        const R *y0 = own + (unsigned)row % 5u * pitch;
        const R *yp = own + (unsigned)ghost_row(row + 1, nr) % 5u * pitch;
        const R *ym = own + (unsigned)ghost_row(row - 1, nr) % 5u * pitch;
        const R *ypp = own + (unsigned)ghost_row(row + 2, nr) % 5u * pitch;
        const R *ymm = own + (unsigned)ghost_row(row - 2, nr) % 5u * pitch;
        s.c = y0[0]; s.e = y0[1]; s.w = y0[-1]; s.ee = y0[2]; s.ww = y0[-2];
        s.n = yp[0]; s.ne = yp[1]; s.nw = yp[-1];
        s.s = ym[0]; s.se = ym[1]; s.sw = ym[-1];
        s.nn = ypp[0]; s.nne = ypp[2]; s.nnw = ypp[-2];
        s.ss = ymm[0]; s.sse = ymm[2]; s.ssw = ymm[-2];
    };

    Phys<R> P1 = P0;
    P1.g_z = gz1;

    // f of the rows lo1 - 2 .. lo1 + 2 (clamped: a repeated row rewrites its own values)
    constexpr int NF = Pre<MODE, R>::NF, NG = Pre<MODE, R>::NG;
    Pre<MODE, R> fp;                             // f of row J + 2
    R fn[9], gn[9], an[3];                       // on their way: f of row J + 3, g and aux of row J
    R ph[4] = {};                                // phi(t) of rows J .. J - 3
    {
        R f5[5][9];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int row = lo1 + q - 2;
            pull_row(std::false_type{}, fr, fin, row < 0 ? 0 : (row > nr - 1 ? nr - 1 : row), f5[q]);
        }
        pull_row(std::false_type{}, gr, gin, lo1, gn);
        load_aux(lo1, an);
        pull_row(std::false_type{}, fr, fin, lo1 + 3 <= phi_hi ? lo1 + 3 : phi_hi, fn);
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int row = lo1 + q - 2;
            if (row >= 0 && row < nr) put_phi(phi_t, row, sum9(f5[q]) * inv_radius<R>(row));
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            fp.take_f(f5[2 + q]);
            if (q < 2)
#pragma unroll
                for (int i = 0; i < NF; ++i) S.fh[(lo1 + q) & 1][i][lane] = fp.f[i];
        }
    }
    // populations at t + 1 on their way (f then g): of links 2, 5, 6 into row J
    // and into row J + 1, of links 0, 1, 3 in row J
    R upA[2][3] = {}, upB[2][3] = {}, mid[2][3] = {};
    // 1 / r of rows J + 2 .. J - 3
    R ir[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const int row = lo1 + 2 - q;
        ir[q] = uniform(inv_radius<R>(row < 0 ? 0 : row));
    }
    lds_barrier();

    auto iteration = [&](int J, auto full_t) {
        constexpr bool FULL = decltype(full_t)::value;     // every stage runs, no row at the edge of the grid
        const bool s1 = FULL || J <= hi1;
        const int I = J - 1, O = J - 3;
        R fv[9], gv[9];
        R uz1 = 0, ur1 = 0;
        if (s1) {
            // ---- step 1 of row J
            Pre<MODE, R> pre;
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                pre.f[i] = S.fh[J & 1][i][lane];
                S.fh[J & 1][i][lane] = fp.f[i];
            }
            pre.take_g(gn);
            const R php = an[0], uzp = an[1], urp = an[2];
            Stencil<R> st;
            get_stencil(phi_t, J, st);
            // the next loads go where the old values were: they are issued only
            // once those are used (else the loop's end would copy, and wait for, them)
            const int rg = FULL || J + 1 <= hi1 ? J + 1 : hi1;
            __builtin_amdgcn_sched_barrier(0);
            pull_row(full_t, gr, gin, rg, gn);
            __builtin_amdgcn_sched_barrier(0);
            const R r = (R)J + (R)0.5;
            Macro<R> m;
            macro_state<MODE>(P0, r, ir[2], st, pre.sums(), uzp, urp, m);
            collide_pre<MODE>(P0, r, ir[2], m, php, uzp, urp, pre, fv, gv);
            ph[3] = ph[2]; ph[2] = ph[1]; ph[1] = ph[0]; ph[0] = m.phi;
            uz1 = m.uz; ur1 = m.ur;
            __builtin_amdgcn_sched_barrier(0);
            load_aux(rg, an);
            to_right[0][0] = fv[1]; to_right[0][1] = fv[5]; to_right[0][2] = fv[8];
            to_right[1][0] = gv[1]; to_right[1][1] = gv[5]; to_right[1][2] = gv[8];
            to_left[0][0] = fv[3]; to_left[0][1] = fv[6]; to_left[0][2] = fv[7];
            to_left[1][0] = gv[3]; to_left[1][1] = gv[6]; to_left[1][2] = gv[7];
        } else {
            ph[3] = ph[2]; ph[2] = ph[1]; ph[1] = ph[0];
        }
        lds_barrier();
        // ---- row J - 1 at t + 1 (Eq. 20 and the boundary rules of pull_slot)
        const bool s2 = FULL || (O >= ra && O < rb);
        Pre<MODE, R> h;
#pragma unroll
        for (int i = 0; i < NF; ++i) h.f[i] = S.h[I & 1][i][lane];
#pragma unroll
        for (int i = 0; i < NG; ++i) h.g[i] = S.h[I & 1][NF + i][lane];
        if (FULL || (I >= ilo && I <= ihi)) {
            R n[2][9];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const R *p = q ? gv : fv;
                n[q][0] = mid[q][0]; n[q][1] = mid[q][1]; n[q][3] = mid[q][2];
                n[q][2] = upA[q][0]; n[q][5] = upA[q][1]; n[q][6] = upA[q][2];
                if (FULL || J < nr) {
                    n[q][4] = p[4];
                    n[q][7] = from_right(p[7], Sr.left[q][2]);
                    n[q][8] = from_left(p[8], Sl.right[q][2]);
                    if (ZWALL) {
                        n[q][8] = at_lo ? upB[q][1] : n[q][8];
                        n[q][7] = at_hi ? upB[q][2] : n[q][7];
                    }
                } else {
                    n[q][4] = upB[q][0]; n[q][7] = upB[q][1]; n[q][8] = upB[q][2];
                }
            }
            Pre<MODE, R> w;
            w.take_f(n[0]);
            w.take_g(n[1]);
            put_phi(phi_t1, I, w.mass() * ir[3]);
#pragma unroll
            for (int i = 0; i < NF; ++i) S.h[I & 1][i][lane] = w.f[i];
#pragma unroll
            for (int i = 0; i < NG; ++i) S.h[I & 1][NF + i][lane] = w.g[i];
        }
        if (s1) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const R *p = q ? gv : fv;
                const R *el = Sl.right[q], *er = Sr.left[q];
                if (!FULL && J == 0) {                     // mirror images across the axis
                    upA[q][0] = p[4]; upA[q][1] = from_left(p[8], el[2]); upA[q][2] = from_right(p[7], er[2]);
                } else {
                    upA[q][0] = upB[q][0]; upA[q][1] = upB[q][1]; upA[q][2] = upB[q][2];
                }
                mid[q][0] = p[0]; mid[q][1] = from_left(p[1], el[0]); mid[q][2] = from_right(p[3], er[0]);
                if (ZWALL) {                               // bounce-back of the node's own
                    upA[q][1] = at_lo ? p[7] : upA[q][1];
                    upA[q][2] = at_hi ? p[8] : upA[q][2];
                    mid[q][1] = at_lo ? p[3] : mid[q][1];
                    mid[q][2] = at_hi ? p[1] : mid[q][2];
                }
                if (!FULL && J == nr - 1) {                // kept for the bounce-back at the r-wall
                    upB[q][0] = p[2]; upB[q][1] = p[5]; upB[q][2] = p[6];
                } else {
                    upB[q][0] = p[2]; upB[q][1] = from_left(p[5], el[1]); upB[q][2] = from_right(p[6], er[1]);
                    if (ZWALL) {
                        // links 5 at the low and 6 at the high wall are bounced
                        // back: their places carry 6 and 5, which the node reads
                        // back as 8 and 7 of this row
                        upB[q][1] = at_lo ? p[6] : upB[q][1];
                        upB[q][2] = at_hi ? p[5] : upB[q][2];
                    }
                }
            }
        }
        // ---- phi(t) of row J + 3, and the loads of the next
        const R ir3 = ir[5];                               // of row J - 3
        ir[5] = ir[4]; ir[4] = ir[3]; ir[3] = ir[2]; ir[2] = ir[1]; ir[1] = ir[0];
        ir[0] = uniform(inv_radius<R>(J + 3));
        if (FULL || J + 3 <= phi_hi) {
            fp.take_f(fn);
            put_phi(phi_t, J + 3, fp.mass() * ir[0]);
            __builtin_amdgcn_sched_barrier(0);
            pull_row(full_t, fr, fin, FULL || J + 4 <= phi_hi ? J + 4 : phi_hi, fn);
        }
        lds_barrier();
        const int slot = (int)((unsigned)J % 3u);          // rows J and J - 3
        const R uz2 = S.aux[slot][0][lane], ur2 = S.aux[slot][1][lane];
        if (s1) {
            S.aux[slot][0][lane] = uz1;
            S.aux[slot][1][lane] = ur1;
        }
        if (s2) {
            // ---- step 2 of row J - 3
            Stencil<R> st;
            get_stencil(phi_t1, O, st);
            const R r = (R)O + (R)0.5;
            Macro<R> m;
            macro_state<MODE>(P1, r, ir3, st, h.sums(), uz2, ur2, m);
            R hf[9], hg[9];
            collide_pre<MODE>(P1, r, ir3, m, ph[3], uz2, ur2, h, hf, hg);
            const uint32_t ro = scalar((uint32_t)O * pt.row);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                buf_store<PAIR_STORE>((T)hf[i], fo, so, ro + (uint32_t)i * pt.plane);
                buf_store<PAIR_STORE>((T)hg[i], go, so, ro + (uint32_t)i * pt.plane);
            }
            buf_store<PAIR_STORE>((T)m.phi, ao, so, ro);
            buf_store<PAIR_STORE>((T)m.uz, ao, so, ro + pt.plane);
            buf_store<PAIR_STORE>((T)m.ur, ao, so, ro + 2 * pt.plane);
        }
    };

    // FULL: step 2 has begun (J >= ra + 3) and the rows loaded (up to J + 4) are
    // wanted and clear of the r-wall
    const int full_lo = ra + 3, last = rb + 2;
    const int full_hi = (phi_hi < nr - 2 ? phi_hi : nr - 2) - 4;
    int J = lo1;
    for (; J < full_lo && J <= last; ++J) iteration(J, std::false_type{});
    // nothing in flight at the loop's entry: else the waits inside would be
    // those of the entry, for everything
    __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
    for (; J <= full_hi; ++J) iteration(J, std::true_type{});
    for (; J <= last; ++J) iteration(J, std::false_type{});
}

// Columns of a strip: what its lanes have beyond the halo, rounded down to
// whole lines of `line` columns where `strips` strips then still cover nz.
// (A strip at a z wall could own up to PAIR_HALO more; one strip of all
// columns between walls needs no halo.)
__host__ __device__ inline int pair_inner(int nz, int z_periodic, int nw, int strips, int line)
{
    const int lanes = 64 * nw;
    if (strips == 1) return nz;
    const int inner = lanes - 2 * PAIR_HALO, whole = inner / line * line;
    return (int64_t)whole * strips >= nz ? whole : inner;
}

// Strip s of a case cut into `strips` workgroups of nw wavefronts.  Beyond a
// strip's own columns its lanes hold a halo of PAIR_HALO on either side,
// except at a z wall and where one strip is the whole period.
template <typename T, typename R, int MODE>
__device__ __forceinline__ void pair_strip(const Geom &g, const Phys<R> &P0, R gz1, int nw, int strips, int s, int ra,
                                           int rb, const T *__restrict__ fin, const T *__restrict__ gin,
                                           const T *__restrict__ ain, T *__restrict__ fout, T *__restrict__ gout,
                                           T *__restrict__ aout, char *lds)
{
    const int lanes = 64 * nw, nz = g.nz;
    const bool full = g.zper && strips == 1 && nz == lanes;
    // strips begin on 64-byte lines where that takes no more of them
    // (pair_strips): the stores of two strips then share no line
    const int inner = pair_inner(nz, g.zper, nw, strips, 64 / (int)sizeof(T));
    const int k0 = full ? 0 : s * inner, k1 = s == strips - 1 ? nz : k0 + inner;
    const int kb = full ? 0 : (g.zper || s > 0 ? k0 - PAIR_HALO : 0);
    if (!g.zper && (kb <= 0 || kb + lanes >= nz))
        pair_march<T, R, MODE, true>(g, P0, gz1, nw, kb, k0, k1, full, ra, rb, fin, gin, ain, fout, gout, aout, lds);
    else
        pair_march<T, R, MODE, false>(g, P0, gz1, nw, kb, k0, k1, full, ra, rb, fin, gin, ain, fout, gout, aout, lds);
}

} // namespace axi
