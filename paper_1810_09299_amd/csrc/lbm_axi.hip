// lbm_axi: C-ABI library for one case of the axisymmetric Allen-Cahn MRT
// lattice Boltzmann method on one MI355X (gfx950).  Declarations and the
// contract of every entry point: include/lbm_axi.h.
//
// Device state of one case (caller-owned block, offsets 256-byte aligned):
//   pop[2][2][9][plane]  ping-pong x {f, g} x populations, storage type T
//   aux[3][plane]        previous-step phi, u_z, u_r (T) of buffer 0
//   fld[5][plane]        doubles: the aux of buffer 1 (T) in the first planes,
//                        the last two for the moments fields of a case that
//                        a graph holds, the last for state transfer; with
//                        FP16-deviation storage (axi_half.hpp) the moments fields
//   red[...]             double scratch for the diagnostics reductions
// plane = nr*nz rounded up to 64 elements, plus 64; SoA, z fastest.
//   diag                 the diagnostics record (lbm_axi_diag) reduced on the device
//
// Two steps of an FP64 or FP32 case are one launch of pair_kernel (large cases,
// axi_pair.hpp) or tile_kernel (small ones, axi_tile.hpp).  A step on its own --
// the odd one out, in a recording, where single steps are ahead, FP16-deviation
// storage -- is one launch of step_kernel: every workgroup owns a 64 x TR tile,
// pulls the f populations of its tile plus a 2-cell ring (the ring's extra
// reads hit L2), forms phi in LDS, and then finishes its own nodes: stencil,
// pressure, velocity, both collisions, store.  No grid-wide synchronisation.

#include "case_internal.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

using namespace axi;

namespace {

constexpr int DIAG_THREADS = 256;  // workgroup of the diagnostics passes (4 waves)
constexpr int DIAG_BLOCKS = 512;   // at most this many moments-pass partials
constexpr int PRS_BLOCKS = 256;    // at most this many pressure-pass partials
constexpr double CS = 0.57735026918962576451;   // lattice sound speed 1/sqrt(3)

inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

} // namespace

namespace axi {
// Elements between population planes: 256-byte aligned, plus PLANE_PAD spare
// elements so that planes and buffers are not a power of two apart (on 16
// cases of 256 x 512 pads of 0..1088 elements measured within 2% of each other).
int64_t plane_elems(int nr, int nz)
{
    return (int64_t)round_up((size_t)nr * nz, 64) + PLANE_PAD;
}
} // namespace axi

namespace {

// ------------------------------------------------------------------ kernels

// t = 0: u = 0, p = 0, g = 0 and the phase-field population at the discrete
// fixed point of a uniform phi: f^eq(phi0, u = 0) of Eq. 11 plus the
// non-equilibrium part h that balances the equilibrium's radial flux M phi.
// With s3..s6 = 1/tau_f and tau_f = 3M + 1/2 (Eq. 18), h_i = -tau_f w_i c_ir phi0,
// so f_i = w_i phi0 (r + 3 M c_ir - tau_f c_ir) = w_i phi0 (r - c_ir / 2).
// Values go into the slots the first step pulls from (the pull map is a bijection).
template <typename T>
__global__ void init_kernel(Geom g, const double *__restrict__ phi0, T *__restrict__ f,
                            T *__restrict__ gp, T *__restrict__ aux)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t nn = (int64_t)g.nr * g.nz;
    if (n >= nn) return;
    int j = (int)(n / g.nz), k = (int)(n - (int64_t)j * g.nz);
    double ph = phi0[n];
    double r = (double)j + 0.5;
    double mid = ph * r, up = ph * (r - 0.5), down = ph * (r + 0.5);
    const double w0 = 4.0 / 9.0, w1 = 1.0 / 9.0, w5 = 1.0 / 36.0;
    f[pull_slot<0>(g, k, j)] = (T)(w0 * mid);
    f[pull_slot<1>(g, k, j)] = (T)(w1 * mid);
    f[pull_slot<2>(g, k, j)] = (T)(w1 * up);
    f[pull_slot<3>(g, k, j)] = (T)(w1 * mid);
    f[pull_slot<4>(g, k, j)] = (T)(w1 * down);
    f[pull_slot<5>(g, k, j)] = (T)(w5 * up);
    f[pull_slot<6>(g, k, j)] = (T)(w5 * up);
    f[pull_slot<7>(g, k, j)] = (T)(w5 * down);
    f[pull_slot<8>(g, k, j)] = (T)(w5 * down);
    for (int i = 0; i < 9; ++i)
        gp[(int64_t)i * g.plane + n] = (T)0;
    aux[n] = (T)ph;
    aux[g.plane + n] = (T)0;
    aux[2 * g.plane + n] = (T)0;
}

// One time step of every node (see the header comment of this file).
template <typename T, typename R, int TR, int MODE>
__global__ __launch_bounds__(TZ *TR) void step_kernel(Geom g, Phys<R> P, const T *__restrict__ fin,
                                                      const T *__restrict__ gin, T *__restrict__ fout,
                                                      T *__restrict__ gout, const T *__restrict__ ain,
                                                      T *__restrict__ aout)
{
    __shared__ R tile[TR + 4][TZ + 4];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    tile_step<T, R, TZ, TR, MODE>(g, P, t % g.tiles_z, t / g.tiles_z, fin, gin, fout, gout, ain, aout, tile);
}

// Two time steps of every node (pair_strip): a workgroup of blockDim / 64
// wavefronts takes one of `strips` strips of columns by a run of `rows` rows.
template <typename T, typename R, int MODE>
__global__ __launch_bounds__(64 * PAIR_WAVES<R>) void pair_kernel(Geom g, Phys<R> P, R gz1, int strips, int rows,
                                                               const T *__restrict__ fin, const T *__restrict__ gin,
                                                               T *__restrict__ fout, T *__restrict__ gout,
                                                               const T *__restrict__ ain, T *__restrict__ aout)
{
    extern __shared__ __align__(16) char lds[];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int s = t % strips, q = t / strips;
    pair_strip<T, R, MODE>(g, P, gz1, (int)(blockDim.x >> 6), strips, s, q * rows,
                           g.nr - q * rows < rows ? g.nr : (q + 1) * rows, fin, gin, ain, fout, gout, aout, lds);
}

// Two time steps of every node of a small case: one tile per workgroup
// (tile_two_steps).
template <typename T, typename R, int MODE, typename S>
__global__ __launch_bounds__(S::THREADS) void tile_kernel(Geom g, Phys<R> P, R gz1, int tiles_z,
                                                          const T *__restrict__ fin, const T *__restrict__ gin,
                                                          T *__restrict__ fout, T *__restrict__ gout,
                                                          const T *__restrict__ ain, T *__restrict__ aout)
{
    extern __shared__ __align__(16) char lds[];
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    tile_two_steps<T, R, MODE, S>(g, P, gz1, b % tiles_z, b / tiles_z, fin, gin, ain, fout, gout, aout, (R *)lds);
}

__device__ __forceinline__ int64_t slot_rt(const Geom &g, int i, int k, int j)
{
    switch (i) {
    case 0: return pull_slot<0>(g, k, j);
    case 1: return pull_slot<1>(g, k, j);
    case 2: return pull_slot<2>(g, k, j);
    case 3: return pull_slot<3>(g, k, j);
    case 4: return pull_slot<4>(g, k, j);
    case 5: return pull_slot<5>(g, k, j);
    case 6: return pull_slot<6>(g, k, j);
    case 7: return pull_slot<7>(g, k, j);
    default: return pull_slot<8>(g, k, j);
    }
}

// post-propagation plane i of a population buffer -> double [nr][nz]
template <typename T>
__global__ void gather_plane_kernel(Geom g, int i, const T *__restrict__ buf, double *__restrict__ out)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)g.nr * g.nz) return;
    int j = (int)(n / g.nz), k = (int)(n - (int64_t)j * g.nz);
    out[n] = (double)buf[slot_rt(g, i, k, j)];
}

// inverse of gather_plane_kernel
template <typename T>
__global__ void scatter_plane_kernel(Geom g, int i, const double *__restrict__ in, T *__restrict__ buf)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)g.nr * g.nz) return;
    int j = (int)(n / g.nz), k = (int)(n - (int64_t)j * g.nz);
    buf[slot_rt(g, i, k, j)] = (T)in[n];
}

template <typename A, typename B>
__global__ void convert_kernel(int64_t count, const A *__restrict__ in, B *__restrict__ out)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n < count) out[n] = (B)in[n];
}

// ------------------------------------------- FP16-deviation storage kernels

// population i arriving at (k, j) from buffer side B (q: 0 for f, 1 for g)
__device__ void slot_of(const Geom &g, int i, int k, int j, int &p, int &ks, int &js)
{
    switch (i) {
    case 0: pull_source<0>(g, k, j, p, ks, js); break;
    case 1: pull_source<1>(g, k, j, p, ks, js); break;
    case 2: pull_source<2>(g, k, j, p, ks, js); break;
    case 3: pull_source<3>(g, k, j, p, ks, js); break;
    case 4: pull_source<4>(g, k, j, p, ks, js); break;
    case 5: pull_source<5>(g, k, j, p, ks, js); break;
    case 6: pull_source<6>(g, k, j, p, ks, js); break;
    case 7: pull_source<7>(g, k, j, p, ks, js); break;
    default: pull_source<8>(g, k, j, p, ks, js); break;
    }
}

// row of the slot that population i (1..8) arriving at (k, j) comes from
__device__ int row_of(const Geom &g, int i, int k, int j)
{
    switch (i) {
    case 1: return slot_row<1>(g, k, j);
    case 2: return slot_row<2>(g, k, j);
    case 3: return slot_row<3>(g, k, j);
    case 4: return slot_row<4>(g, k, j);
    case 5: return slot_row<5>(g, k, j);
    case 6: return slot_row<6>(g, k, j);
    case 7: return slot_row<7>(g, k, j);
    default: return slot_row<8>(g, k, j);
    }
}

// t = 0 as init_kernel: every f_q (q >= 1) a node pulls is the uniform-field
// value phi0 b_q(r) its slot is referenced to, so every stored deviation is 0;
// f_0 on the row's grid.
__global__ void init_kernel_h(Geom g, Codec C, const double *__restrict__ phi0, HalfBuf B, float *__restrict__ uz,
                              float *__restrict__ ur)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t nn = (int64_t)g.nr * g.nz;
    if (n >= nn) return;
    int j = (int)(n / g.nz);
    double ph = phi0[n];
    double r = (double)j + 0.5;
    B.f0[n] = quantize_row((float)(4.0 / 9.0 * (ph * r)), j);
    for (int p = 1; p < 9; ++p)
        B.f[(int64_t)(p - 1) * g.plane + n] = (half_t)0.0f;
    for (int i = 0; i < 9; ++i)
        B.g[(int64_t)i * g.plane + n] = (half_t)0.0f;
    B.phi[n] = (float)ph;
    uz[n] = 0.0f;
    ur[n] = 0.0f;
}

// six waves per SIMD for 64 x 8 and 64 x 16 tiles, as batch_step_kernel_h
template <int TR, int MODE, bool SR>
__global__ __launch_bounds__(TZ *TR) __attribute__((amdgpu_waves_per_eu(
    TR >= 8 ? 6 : 1))) void step_kernel_h(Geom g, Phys<float> P, Codec C, HalfState S)
{
    __shared__ float tile[TR + 4][TZ + 4];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    tile_step_h<TZ, TR, MODE, false, SR>(g, P, C, t % g.tiles_z, t / g.tiles_z, S, Fields{}, tile);
}

__global__ void gather_plane_h(Geom g, Codec C, HalfBuf B, int i, int q, double *__restrict__ out)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)g.nr * g.nz) return;
    int j = (int)(n / g.nz), k = (int)(n - (int64_t)j * g.nz);
    int p, ks, js;
    slot_of(g, i, k, j, p, ks, js);
    int64_t s = (int64_t)js * g.nz + ks;
    float rs = (float)js + 0.5f, rd = (float)j + 0.5f;
    float v;
    if (q == 1)
        v = decode_g(B.g[(int64_t)p * g.plane + s], rs, C);
    else if (p == 0)
        v = B.f0[s];
    else {  // referenced to the reader (k, j), population i
        const int jx = row_of(g, i, k, j);
        v = decode_f(B.f[(int64_t)(p - 1) * g.plane + s], B.phi[n], bulk_factor_rt(i, rd), (float)jx + 0.5f, jx, C);
    }
    out[n] = (double)v;
}

// inverse of gather_plane_h (the phase field of side B must be set first)
__global__ void scatter_plane_h(Geom g, Codec C, HalfBuf B, int i, int q, const double *__restrict__ in)
{
    int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)g.nr * g.nz) return;
    int j = (int)(n / g.nz), k = (int)(n - (int64_t)j * g.nz);
    int p, ks, js;
    slot_of(g, i, k, j, p, ks, js);
    int64_t s = (int64_t)js * g.nz + ks;
    float rs = (float)js + 0.5f, rd = (float)j + 0.5f;
    float v = (float)in[n];
    if (q == 1)
        B.g[(int64_t)p * g.plane + s] = encode_g(v, 1.0f / rs, C);
    else if (p == 0)
        B.f0[s] = quantize_row(v, js);
    else
        B.f[(int64_t)(p - 1) * g.plane + s] =
            encode_f(v, B.phi[n], bulk_factor_rt(i, rd), 1.0f / ((float)row_of(g, i, k, j) + 0.5f), C);
}

// sum of the f that node n pulls in FP16-deviation storage (exact in FP32);
// over all nodes it is the sum of every stored value (a pull is a bijection)
__device__ double node_mass_h(const Geom &g, const Codec &C, const HalfBuf &B, int64_t n, int j)
{
    const int k = (int)(n - (int64_t)j * g.nz);
    const float rd = (float)j + 0.5f;
    double s = (double)B.f0[n];
    const float ph = B.phi[n];
    for (int i = 1; i < 9; ++i) {
        int p, ks, js;
        slot_of(g, i, k, j, p, ks, js);
        const int jx = row_of(g, i, k, j);
        s += (double)decode_f(B.f[(int64_t)(p - 1) * g.plane + (int64_t)js * g.nz + ks], ph, bulk_factor_rt(i, rd),
                              (float)jx + 0.5f, jx, C);
    }
    return s;
}

// ----------------------------------------------------------- diagnostics
//
// The read-back is three launches, the reductions in double:
//   moments_kernel  the fields at time t (the macroscopic prefix of a step),
//                   and on the way the sums over the nodes: phase mass (the f
//                   each node pulls), fluid mass, momentum, max |u|, the
//                   psi-weighted sums, min axis phi and the non-finite count;
//                   at most DIAG_BLOCKS workgroups stride over the tiles, each
//                   leaving one partial
//   diag_pressure   at most PRS_BLOCKS workgroups; each first reduces the
//                   partial psi sums (in the order diag_final reduces them,
//                   so the same centroid and R_eq), then sums the pressure inside and
//                   outside over its nodes and finds its nearest psi = 1/2
//                   crossings around the centroid column (axis row left and
//                   right, the column upwards)
//   diag_final      one workgroup: the remaining reductions and the record
// Within a wave, values are combined by an xor butterfly of lane shuffles;
// the four waves of a workgroup then meet in LDS behind a single barrier.
// The order of every sum is fixed, so the diagnostics are deterministic.
// (Folding the final reduction into the last workgroup of a pass to finish
// measured slower: the device-scope release it needs writes back each XCD's
// L2, fields included, from every workgroup.)
//
// Scratch of one read-back (doubles): DIAG_BLOCKS x NSUM partials, then
// PRS_BLOCKS x NPRS partials; every read-back writes the partials it reads.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

enum { RED_SUM = 0, RED_MAX = 1, RED_MIN = 2 };

// N values per thread reduced over the workgroup (DIAG_THREADS = 4 waves);
// kinds[q] says how value q combines.  Every thread receives the results.
template <int N>
__device__ __forceinline__ void block_reduce(double (&v)[N], const int (&kinds)[N], double (*sh)[N])
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < N; ++q)
        v[q] = kinds[q] == RED_SUM ? wave_sum(v[q]) : (kinds[q] == RED_MAX ? wave_max(v[q]) : wave_min(v[q]));
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < N; ++q) sh[wv][q] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const double a = sh[0][q], b = sh[1][q], c = sh[2][q], d = sh[3][q];
        v[q] = kinds[q] == RED_SUM ? (a + b) + (c + d)
                                   : (kinds[q] == RED_MAX ? fmax(fmax(a, b), fmax(c, d)) : fmin(fmin(a, b), fmin(c, d)));
    }
}

// partial sums of the moments pass, per workgroup
enum { S_MASS, S_FLUID, S_MOMZ, S_UMAX, S_PSI, S_PSIZ, S_PSIU, S_MINAX, S_BAD, NSUM };
constexpr int S_KIND[NSUM] = {RED_SUM, RED_SUM, RED_SUM, RED_MAX, RED_SUM, RED_SUM, RED_SUM, RED_MIN, RED_SUM};
// partials of diag_pressure: pressure sums and counts, and the distances of
// the nearest psi <= 1/2 crossings from the centroid column (see diag_record)
enum { P_IN, P_NIN, P_OUT, P_NOUT, P_LEFT, P_RIGHT, P_UP, NPRS };
constexpr int P_KIND[NPRS] = {RED_SUM, RED_SUM, RED_SUM, RED_SUM, RED_MIN, RED_MIN, RED_MIN};
constexpr double NONE = 2147483647.0;     // no crossing

__device__ __forceinline__ void diag_init(double (&a)[NSUM])
{
#pragma unroll
    for (int q = 0; q < NSUM; ++q) a[q] = 0.0;
    a[S_MINAX] = INFINITY;
}

// one node's share of the first reduction
__device__ __forceinline__ void diag_add(double (&a)[NSUM], int gas, int j, int k, double phi, double rho, double uz,
                                         double ur, double p, double mass)
{
    const double r = j + 0.5;
    const double psi = gas ? 1.0 - phi : phi;
    a[S_MASS] += mass;
    a[S_FLUID] += r * rho;
    a[S_MOMZ] += r * rho * uz;
    a[S_UMAX] = fmax(a[S_UMAX], sqrt(uz * uz + ur * ur));
    // psi-weighted over the dispersed phase's region psi > 1/100: on a large
    // grid a bulk phase field a little off 0 or 1 would otherwise outweigh the
    // drop; the tanh tail left out is ~W/400 of a cell
    const double wt = psi > 0.01 ? r * psi : 0.0;
    a[S_PSI] += wt;
    a[S_PSIZ] += wt * k;
    a[S_PSIU] += wt * uz;
    if (j == 0) a[S_MINAX] = fmin(a[S_MINAX], phi);
    const bool bad = !(isfinite(phi) && isfinite(uz) && isfinite(ur) && isfinite(p));
    a[S_BAD] += bad ? 1.0 : 0.0;
    if (bad) a[S_UMAX] = INFINITY;
}

// workgroups of the moments pass: one per tile, at most DIAG_BLOCKS
inline int moments_blocks(const Geom &g) { return std::min(g.tiles, DIAG_BLOCKS); }

// layout of the read-back scratch
struct DiagScratch {
    double *sums;        // [DIAG_BLOCKS][NSUM]
    double *prs;         // [PRS_BLOCKS][NPRS]
};
constexpr size_t DIAG_SCRATCH_DOUBLES = (size_t)DIAG_BLOCKS * NSUM + (size_t)PRS_BLOCKS * NPRS;

__host__ __device__ inline DiagScratch diag_scratch(double *base)
{
    DiagScratch d;
    d.sums = base;
    d.prs = base + (size_t)DIAG_BLOCKS * NSUM;
    return d;
}

// totals of the first reduction over n partials, in partial order; every
// thread receives them
__device__ __forceinline__ void reduce_sums(int n, const double *__restrict__ part, double (&a)[NSUM],
                                            double (*sh)[NSUM])
{
    diag_init(a);
    for (int b = threadIdx.x; b < n; b += DIAG_THREADS) {
        const double *q = part + (int64_t)b * NSUM;
        a[S_MASS] += q[S_MASS];
        a[S_FLUID] += q[S_FLUID];
        a[S_MOMZ] += q[S_MOMZ];
        a[S_UMAX] = fmax(a[S_UMAX], q[S_UMAX]);
        a[S_PSI] += q[S_PSI];
        a[S_PSIZ] += q[S_PSIZ];
        a[S_PSIU] += q[S_PSIU];
        a[S_MINAX] = fmin(a[S_MINAX], q[S_MINAX]);
        a[S_BAD] += q[S_BAD];
    }
    __syncthreads();                     // sh may still be read by an earlier reduction
    block_reduce<NSUM>(a, S_KIND, sh);
}

// the psi sums of reduce_sums alone: the same partials per lane in the same
// order and the same tree, so the same values
__device__ __forceinline__ void reduce_psi(int n, const double *__restrict__ part, double &spsi, double &spsiz,
                                           double (*sh)[2])
{
    double v[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < n; b += DIAG_THREADS) {
        v[0] += part[(int64_t)b * NSUM + S_PSI];
        v[1] += part[(int64_t)b * NSUM + S_PSIZ];
    }
    const int kinds[2] = {RED_SUM, RED_SUM};
    block_reduce<2>(v, kinds, sh);
    spsi = v[0];
    spsiz = v[1];
}

template <typename T, typename R, int TR>
__global__ __launch_bounds__(TZ *TR) void moments_kernel(Geom g, Phys<R> P, const T *__restrict__ fin,
                                                         const T *__restrict__ gin,
                                                         const T *__restrict__ aux, Fields F, int gas,
                                                         double *__restrict__ scratch)
{
    static_assert(TZ * TR == DIAG_THREADS, "the reductions take four waves");
    __shared__ R tile[TR + 4][TZ + 4];
    __shared__ double sh[4][NSUM];
    double a[NSUM];
    diag_init(a);
    const int tx = threadIdx.x % TZ, ty = threadIdx.x / TZ;
    for (int t = blockIdx.x; t < g.tiles; t += gridDim.x) {
        const int tz = t % g.tiles_z, tr = t / g.tiles_z;
        const int k0 = tz * TZ, j0 = tr * TR;
        const int k = k0 + tx, j = j0 + ty;
        const bool inside = (k < g.nz) && (j < g.nr);
        const int jo = ghost_row(j, g.nr), ko = ghost_col(k, g.nz, g.zper);
        R fv[9], gv[9];
        // every load of the tile before its barrier: one wait on memory (g
        // and aux of a node beyond the grid are read at its ghost cell and
        // not used)
        pull9<T, R>(g, fin, ko, jo, fv);
        pull9<T, R>(g, gin, ko, jo, gv);
        const int64_t n = (int64_t)j * g.nz + k, no = (int64_t)jo * g.nz + ko;
        const R uzp = (R)aux[g.plane + no], urp = (R)aux[2 * g.plane + no];
        tile[ty + 2][tx + 2] = sum9(fv) * inv_radius<R>(jo);
        fill_halo<T, R, TZ, TR>(g, fin, k0, j0, tile);
        __syncthreads();
        if (inside) {
            Stencil<R> st;
            read_stencil<R, TZ>(tile, tx, ty, st);
            R r = (R)j + (R)0.5, ir = inv_radius<R>(j);
            Macro<R> m;
            macro_state<FORM_OF_P>(P, r, ir, st, gv, uzp, urp, m);
            if (F.phi) F.phi[n] = (double)m.phi;
            if (F.rho) F.rho[n] = (double)m.rho;
            if (F.uz) F.uz[n] = (double)m.uz;
            if (F.ur) F.ur[n] = (double)m.ur;
            if (F.p) F.p[n] = (double)m.p;
            double mass = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i) mass += (double)fv[i];
            diag_add(a, gas, j, k, (double)m.phi, (double)m.rho, (double)m.uz, (double)m.ur, (double)m.p, mass);
        }
        __syncthreads();    // the LDS tile is refilled for the next tile
    }
    block_reduce<NSUM>(a, S_KIND, sh);
    if (threadIdx.x < NSUM) diag_scratch(scratch).sums[(int64_t)blockIdx.x * NSUM + threadIdx.x] = a[threadIdx.x];
}

template <int TR>
__global__ __launch_bounds__(TZ *TR) void moments_kernel_h(Geom g, Phys<float> P, Codec C, HalfState S, Fields F,
                                                           int gas, double *__restrict__ scratch)
{
    static_assert(TZ * TR == DIAG_THREADS, "the reductions take four waves");
    __shared__ float tile[TR + 4][TZ + 4];
    __shared__ double sh[4][NSUM];
    double a[NSUM];
    diag_init(a);
    for (int t = blockIdx.x; t < g.tiles; t += gridDim.x) {
        NodeMoments mo;
        tile_step_h<TZ, TR, COLLIDE_MRT, true>(g, P, C, t % g.tiles_z, t / g.tiles_z, S, F, tile, &mo);
        if (mo.valid) diag_add(a, gas, mo.j, mo.k, mo.phi, mo.rho, mo.uz, mo.ur, mo.p, mo.mass);
        __syncthreads();    // the LDS tile is refilled for the next tile
    }
    block_reduce<NSUM>(a, S_KIND, sh);
    if (threadIdx.x < NSUM) diag_scratch(scratch).sums[(int64_t)blockIdx.x * NSUM + threadIdx.x] = a[threadIdx.x];
}

__device__ __forceinline__ double psi_at(const Geom &g, int gas, const double *phi, int j, int k)
{
    const double v = phi[(int64_t)j * g.nz + k];
    return gas ? 1.0 - v : v;
}

__device__ __forceinline__ int wrap_col(int k, int nz) { return k < 0 ? k + nz : (k >= nz ? k - nz : k); }

// the column nearest the centroid
__device__ __forceinline__ int centroid_column(const Geom &g, double zc)
{
    const int kc = (int)floor(zc + 0.5);
    return kc < 0 ? 0 : (kc >= g.nz ? g.nz - 1 : kc);
}

// The diagnostics record from the totals, the reduced pressure partials and
// the phase field (the semi-axes).  The axial semi-axis is half the distance
// between the nearest psi = 1/2 crossings left and right of the centroid
// column kc on the axis row (a wall bounds the walk half a cell beyond the
// last column; with periodic z a walk that finds none ends one period away),
// the radial one the crossing up column kc (nr if none), each linearly
// interpolated between the two nodes around it; both 0 when kc's axis node is
// not in the dispersed phase.
__device__ void diag_record(const Geom &g, int gas, const double *tot, const double (&pp)[NPRS],
                            const double *__restrict__ phi, int64_t t, lbm_axi_diag *__restrict__ out)
{
    const double spsi = tot[S_PSI];
    const double zc = spsi > 0 ? tot[S_PSIZ] / spsi : 0.0;
    lbm_axi_diag d;
    d.t = t;
    d.phase_mass = tot[S_MASS];
    d.fluid_mass = tot[S_FLUID];
    d.mom_z = tot[S_MOMZ];
    d.umax = tot[S_UMAX];
    d.centroid_z = zc;
    d.rise_u = spsi > 0 ? tot[S_PSIU] / spsi : 0.0;
    d.R_eq = spsi > 0 ? cbrt(1.5 * spsi) : 0.0;
    d.min_axis_phi = tot[S_MINAX];
    d.nonfinite = (int64_t)tot[S_BAD];
    d.p_in = pp[P_NIN] > 0 ? pp[P_IN] / pp[P_NIN] : 0.0;
    d.p_out = pp[P_NOUT] > 0 ? pp[P_OUT] / pp[P_NOUT] : 0.0;
    d.dp = d.p_in - d.p_out;
    d.semi_z = 0.0;
    d.semi_r = 0.0;
    const int kc = centroid_column(g, zc);
    if (psi_at(g, gas, phi, 0, kc) > 0.5) {
        double zlo, zhi;
        if (pp[P_LEFT] != NONE) {
            const int mp = kc - (int)pp[P_LEFT];
            const double va = psi_at(g, gas, phi, 0, wrap_col(mp, g.nz));
            const double vb = psi_at(g, gas, phi, 0, wrap_col(mp + 1, g.nz));
            zlo = mp + (0.5 - va) / (vb - va);
        } else {
            zlo = g.zper ? (double)(kc - g.nz) : -0.5;
        }
        if (pp[P_RIGHT] != NONE) {
            const int pk = kc + (int)pp[P_RIGHT];
            const double va = psi_at(g, gas, phi, 0, wrap_col(pk - 1, g.nz));
            const double vb = psi_at(g, gas, phi, 0, wrap_col(pk, g.nz));
            zhi = (pk - 1) + (va - 0.5) / (va - vb);
        } else {
            zhi = g.zper ? (double)(kc + g.nz) : g.nz - 0.5;
        }
        d.semi_z = 0.5 * (zhi - zlo);
        if (pp[P_UP] != NONE) {
            const int jr = (int)pp[P_UP];
            const double va = psi_at(g, gas, phi, jr, kc), vb = psi_at(g, gas, phi, jr + 1, kc);
            d.semi_r = jr + 0.5 + (va - 0.5) / (va - vb);
        } else {
            d.semi_r = g.nr;
        }
    }
    *out = d;
}

// pass 2: pressure inside and outside the dispersed phase, and the crossing
// candidates: on the axis row, a node with psi <= 1/2 at distance m left
// (right) of the centroid column kc, counting around the period with periodic
// z (m = 1..nz), only on its own side with walls; up column kc, a node of row
// j >= 1 with psi <= 1/2 stands for the crossing between rows j - 1 and j.
// nsums: the partials of the moments pass.
__global__ __launch_bounds__(DIAG_THREADS) void diag_pressure(Geom g, int gas, double W, Fields F, int nsums,
                                                               double *__restrict__ scratch)
{
    __shared__ double shs[4][2];
    __shared__ double sh[4][NPRS];
    const DiagScratch D = diag_scratch(scratch);
    double spsi, spsiz;
    reduce_psi(nsums, D.sums, spsi, spsiz, shs);
    const double zc = spsi > 0 ? spsiz / spsi : 0.0, Rq = spsi > 0 ? cbrt(1.5 * spsi) : 0.0;
    const int kc = centroid_column(g, zc);
    const int64_t nn = (int64_t)g.nr * g.nz;
    double a[NPRS] = {0, 0, 0, 0, NONE, NONE, NONE};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < nn; n += stride) {
        // nr*nz <= 2^25: a 32-bit division
        const int j = (int)n / g.nz, k = (int)n - j * g.nz;
        const double dz = k - zc, r = j + 0.5;
        const double dist = sqrt(dz * dz + r * r);
        const double p = F.p[n];
        if (dist < Rq - 2.0 * W) {
            a[P_IN] += p;
            a[P_NIN] += 1.0;
        } else if (dist > Rq + 2.0 * W) {
            const bool near_wall = (j > g.nr - 4) || (!g.zper && (k < 3 || k > g.nz - 4));
            if (!near_wall) {
                a[P_OUT] += p;
                a[P_NOUT] += 1.0;
            }
        }
        if ((j == 0 || k == kc) && psi_at(g, gas, F.phi, j, k) <= 0.5) {
            if (j == 0) {
                int ml = kc - k, mr = k - kc;
                if (g.zper) {
                    ml = ml <= 0 ? ml + g.nz : ml;
                    mr = mr <= 0 ? mr + g.nz : mr;
                }
                if (ml > 0) a[P_LEFT] = fmin(a[P_LEFT], (double)ml);
                if (mr > 0) a[P_RIGHT] = fmin(a[P_RIGHT], (double)mr);
            }
            if (k == kc && j >= 1) a[P_UP] = fmin(a[P_UP], (double)(j - 1));
        }
    }
    block_reduce<NPRS>(a, P_KIND, sh);
    if (threadIdx.x < NPRS) D.prs[(int64_t)blockIdx.x * NPRS + threadIdx.x] = a[threadIdx.x];
}

// pass 3 (one workgroup): the totals of both passes and the record.  The
// totals of the moments pass reduce exactly as in every workgroup of
// diag_pressure, so the centroid is the one it used.
__global__ __launch_bounds__(DIAG_THREADS) void diag_final(Geom g, int gas, int nsums, int nprs,
                                                            const double *__restrict__ scratch,
                                                            const double *__restrict__ phi, int64_t t,
                                                            lbm_axi_diag *__restrict__ out)
{
    __shared__ double shs[4][NSUM];
    __shared__ double sh[4][NPRS];
    const DiagScratch D = diag_scratch((double *)scratch);
    // the pressure partials are read before the first reduction waits
    double pp[NPRS] = {0, 0, 0, 0, NONE, NONE, NONE};
    for (int b = threadIdx.x; b < nprs; b += DIAG_THREADS) {
        const double *w = D.prs + (int64_t)b * NPRS;
        for (int x = 0; x < NPRS; ++x) pp[x] = P_KIND[x] == RED_SUM ? pp[x] + w[x] : fmin(pp[x], w[x]);
    }
    double tot[NSUM];
    reduce_sums(nsums, D.sums, tot, shs);
    block_reduce<NPRS>(pp, P_KIND, sh);
    if (threadIdx.x == 0) diag_record(g, gas, tot, pp, phi, t, out);
}

// Reduction scratch of lbm_axi_moments_noalloc, one copy per device the
// library runs on (held until the process ends).  Its size does not depend on
// the grid: the read-back's passes stride over the nodes with at most
// DIAG_BLOCKS and PRS_BLOCKS workgroups.  Host code never uses this name as an
// address: it takes the device address once per device (noalloc_scratch).
static __device__ __align__(256) double scratch[DIAG_SCRATCH_DOUBLES];

} // namespace

// ------------------------------------------------------------------- host



namespace {

// device addresses of `scratch`, taken once per device with that device current
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_addr[MAX_DEVICES];

int noalloc_scratch(int dev, double **out)
{
    if (dev < 0 || dev >= MAX_DEVICES) return LBM_AXI_EDEVICE;
    std::lock_guard<std::mutex> lk(scratch_mu);
    if (!scratch_addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LBM_AXI_EDEVICE;
        scratch_addr[dev] = ptr;
    }
    *out = (double *)scratch_addr[dev];
    return LBM_AXI_OK;
}

struct Layout {
    int64_t plane;
    size_t esize, fbytes, gbytes, off_pop, off_aux, off_fld, off_part, off_diag, total;
};

bool finite(double x) { return std::isfinite(x); }

int validate(const lbm_axi_params *p)
{
    if (!p) return LBM_AXI_EINVAL;
    if (p->nr < 4 || p->nz < 4) return LBM_AXI_EINVAL;
    // the 9 population planes of a buffer stay below 2^32 bytes (32-bit offsets)
    if ((int64_t)p->nr * p->nz > ((int64_t)1 << 25)) return LBM_AXI_EINVAL;
    if (p->z_periodic != 0 && p->z_periodic != 1) return LBM_AXI_EINVAL;
    if (p->precision != LBM_AXI_FP64 && p->precision != LBM_AXI_FP32 && p->precision != LBM_AXI_FP16D)
        return LBM_AXI_EINVAL;
    if (p->dispersed_gas != 0 && p->dispersed_gas != 1) return LBM_AXI_EINVAL;
    if (p->free_s1 != 0 && p->free_s1 != 1) return LBM_AXI_EINVAL;
    if (p->fp16_rounding != LBM_AXI_ROUND_NEAREST && p->fp16_rounding != LBM_AXI_ROUND_STOCHASTIC)
        return LBM_AXI_EINVAL;
    if (p->fp16_rounding != LBM_AXI_ROUND_NEAREST && p->precision != LBM_AXI_FP16D) return LBM_AXI_EINVAL;
    if (p->free_s1 && p->collision == LBM_AXI_SRT) return LBM_AXI_EINVAL;
    if (p->free_s1 && !(std::isfinite(p->s_g[1]) && p->s_g[1] > 0 && p->s_g[1] < 2)) return LBM_AXI_EINVAL;
    if (!std::isfinite(p->g_ramp) || p->g_ramp < 0) return LBM_AXI_EINVAL;
    if (p->collision != LBM_AXI_MRT && p->collision != LBM_AXI_SRT && p->collision != LBM_AXI_NMRT)
        return LBM_AXI_EINVAL;
    const double vals[] = {p->W, p->mobility, p->sigma, p->rho_l, p->rho_g, p->nu_l, p->nu_g, p->g_z};
    for (double v : vals)
        if (!finite(v)) return LBM_AXI_EINVAL;
    if (!(p->W > 0) || !(p->mobility > 0) || p->sigma < 0) return LBM_AXI_EINVAL;
    if (!(p->rho_l > 0) || !(p->rho_g > 0) || !(p->nu_l > 0) || !(p->nu_g > 0)) return LBM_AXI_EINVAL;
    for (int a = 0; a < 9; ++a) {
        bool fd = (a >= 3 && a <= 6), gd = (a == 1 || a == 7 || a == 8);
        if (!fd && !(finite(p->s_f[a]) && p->s_f[a] >= 0 && p->s_f[a] < 2)) return LBM_AXI_EINVAL;
        if (!gd && !(finite(p->s_g[a]) && p->s_g[a] >= 0 && p->s_g[a] < 2)) return LBM_AXI_EINVAL;
    }
    if (!(p->s_g[2] > 0)) return LBM_AXI_EINVAL;  // s_p of Eq. 33 divides by s_2^g
    return LBM_AXI_OK;
}

Layout layout_of(const lbm_axi_params *p)
{
    Layout L;
    L.plane = plane_elems(p->nr, p->nz);
    const size_t pl = (size_t)L.plane;
    size_t aux_bytes;
    if (p->precision == LBM_AXI_FP16D) {
        // f: the FP32 f_0 plane, then 8 FP16 planes; g: 9 FP16 planes;
        // aux: phase field (two sides), u_z, u_r in FP32
        L.esize = 2;
        L.fbytes = round_up(pl * 4 + 8 * pl * 2, 256);
        L.gbytes = round_up(9 * pl * 2, 256);
        aux_bytes = 4 * pl * 4;
    } else {
        L.esize = p->precision == LBM_AXI_FP64 ? 8 : 4;
        L.fbytes = L.gbytes = 9 * pl * L.esize;
        aux_bytes = 3 * pl * L.esize;
    }
    L.off_pop = 0;
    L.off_aux = round_up(L.off_pop + 2 * (L.fbytes + L.gbytes), 256);
    L.off_fld = round_up(L.off_aux + aux_bytes, 256);
    L.off_part = round_up(L.off_fld + 5 * (size_t)L.plane * 8, 256);
    L.off_diag = round_up(L.off_part + DIAG_SCRATCH_DOUBLES * 8, 256);
    L.total = round_up(L.off_diag + sizeof(lbm_axi_diag), 256);
    return L;
}

template <typename R>
Phys<R> make_phys(const lbm_axi_params *p)
{
    Phys<R> P;
    P.round_key = 0;
    P.rho_l = (R)p->rho_l;
    P.rho_g = (R)p->rho_g;
    P.drho = (R)(p->rho_l - p->rho_g);
    P.nu_g = (R)p->nu_g;
    P.dnu = (R)(p->nu_l - p->nu_g);
    P.mob = (R)p->mobility;
    P.lam4W = (R)(4.0 / p->W);
    P.beta4 = (R)(4.0 * 12.0 * p->sigma / p->W);
    P.kap = (R)(1.5 * p->sigma * p->W);
    P.g_z = (R)p->g_z;
    double s_tau_f = 1.0 / (3.0 * p->mobility + 0.5);        // Eq. 18
    for (int a = 0; a < 9; ++a) {
        P.sf[a] = (R)((a >= 3 && a <= 6) ? s_tau_f : p->s_f[a]);
        P.sg[a] = (R)p->s_g[a];
    }
    P.sg2 = (R)p->s_g[2];
    P.isg2 = (R)(1.0 / p->s_g[2]);
    P.free_s1 = p->free_s1;
    P.isg1 = (R)(p->free_s1 ? 1.0 / p->s_g[1] : 0.0);
    P.g_full = p->g_z;
    P.g_ramp = p->g_ramp;
    bool unit = !p->free_s1;
    for (int a = 0; a < 9; ++a) {
        if (!(a >= 3 && a <= 6) && p->s_f[a] != 1.0) unit = false;
        if (!(a == 1 || a == 7 || a == 8) && p->s_g[a] != 1.0) unit = false;
    }
    P.srt = p->collision == LBM_AXI_SRT;
    if (P.srt)
        for (int a = 0; a < 9; ++a)
            P.sf[a] = (R)s_tau_f;
    P.nmrt = p->collision == LBM_AXI_NMRT;
    P.unit_rates = (unit && p->collision == LBM_AXI_MRT) ? 1 : 0;
    P.mode = P.srt ? COLLIDE_SRT : (P.nmrt ? COLLIDE_NMRT : (P.unit_rates ? COLLIDE_MRT_UNIT : COLLIDE_MRT));
    return P;
}

// FP16 scales (powers of two).  f: deviations of f/r from the bulk form stay
// well below 0.1, stored times 2^10.  g: g/r is of the order of the pressure,
// whose scale is the capillary pressure 4 sigma / W at the smallest resolved
// radius or the hydrostatic range rho_l g_z L; it is stored times 2^4 / that
// scale, which leaves 12 binades above it and 18 normal binades below it.
Codec make_codec(const lbm_axi_params *p)
{
    double gref = std::max(4.0 * p->sigma / p->W,
                           std::max(p->rho_l * std::fabs(p->g_z) * (double)std::max(p->nr, p->nz), 1e-6 * p->rho_l));
    int eg = 4 - (int)std::ceil(std::log2(gref));
    Codec C;
    C.sf = std::ldexp(1.0f, 10);
    C.isf = std::ldexp(1.0f, -10);
    C.sg = std::ldexp(1.0f, eg);
    C.isg = std::ldexp(1.0f, -eg);
    return C;
}

#define HIP_OK(x)                                  \
    do {                                           \
        if ((x) != hipSuccess) return LBM_AXI_EDEVICE; \
    } while (0)

int launch_ok() { return hipGetLastError() == hipSuccess ? LBM_AXI_OK : LBM_AXI_EDEVICE; }

template <typename T, typename R, int TR>
void launch_step(lbm_axi_case *c, const Phys<R> &P)
{
    const T *fin = (const T *)c->pop[c->cur][0];
    const T *gin = (const T *)c->pop[c->cur][1];
    T *fout = (T *)c->pop[c->cur ^ 1][0];
    T *gout = (T *)c->pop[c->cur ^ 1][1];
    if (P.mode == COLLIDE_MRT_UNIT)
        step_kernel<T, R, TR, COLLIDE_MRT_UNIT><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(
            c->geom, P, fin, gin, fout, gout, (const T *)c->aux[c->cur], (T *)c->aux[c->cur ^ 1]);
    else if (P.mode == COLLIDE_SRT)
        step_kernel<T, R, TR, COLLIDE_SRT><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(
            c->geom, P, fin, gin, fout, gout, (const T *)c->aux[c->cur], (T *)c->aux[c->cur ^ 1]);
    else if (P.mode == COLLIDE_NMRT)
        step_kernel<T, R, TR, COLLIDE_NMRT><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(
            c->geom, P, fin, gin, fout, gout, (const T *)c->aux[c->cur], (T *)c->aux[c->cur ^ 1]);
    else
        step_kernel<T, R, TR, COLLIDE_MRT><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(
            c->geom, P, fin, gin, fout, gout, (const T *)c->aux[c->cur], (T *)c->aux[c->cur ^ 1]);
}

template <typename T, typename R>
void launch_step_tr(lbm_axi_case *c, const Phys<R> &P)
{
    switch (c->tile_r) {
    case 2: launch_step<T, R, 2>(c, P); break;
    case 4: launch_step<T, R, 4>(c, P); break;
    case 16: launch_step<T, R, 16>(c, P); break;
    default: launch_step<T, R, 8>(c, P); break;
    }
}

template <typename R>
Phys<R> phys_at(const Phys<R> &P, int64_t t);

template <int TR, bool SR>
void launch_step_h(lbm_axi_case *c)
{
    HalfState S = half_state(c, c->cur);
    const Phys<float> P = phys_at(c->P32, c->t);
    if (P.mode == COLLIDE_MRT_UNIT)
        step_kernel_h<TR, COLLIDE_MRT_UNIT, SR><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(c->geom, P, c->codec, S);
    else if (P.mode == COLLIDE_SRT)
        step_kernel_h<TR, COLLIDE_SRT, SR><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(c->geom, P, c->codec, S);
    else if (P.mode == COLLIDE_NMRT)
        step_kernel_h<TR, COLLIDE_NMRT, SR><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(c->geom, P, c->codec, S);
    else
        step_kernel_h<TR, COLLIDE_MRT, SR><<<c->geom.tiles, TZ * TR, 0, c->stream>>>(c->geom, P, c->codec, S);
}

template <bool SR>
void launch_step_h_sr(lbm_axi_case *c)
{
    switch (c->tile_r) {
    case 2: launch_step_h<2, SR>(c); break;
    case 4: launch_step_h<4, SR>(c); break;
    case 16: launch_step_h<16, SR>(c); break;
    default: launch_step_h<8, SR>(c); break;
    }
}

void launch_step_h_tr(lbm_axi_case *c)
{
    if (c->prm.fp16_rounding == LBM_AXI_ROUND_STOCHASTIC)
        launch_step_h_sr<true>(c);
    else
        launch_step_h_sr<false>(c);
}

// the case's rates with the acceleration of the step from time t
template <typename R>
Phys<R> phys_at(const Phys<R> &P, int64_t t)
{
    Phys<R> Q = P;
    Q.g_z = (R)ramp_accel(P.g_full, P.g_ramp, t);
    Q.round_key = mix32((uint32_t)t);
    return Q;
}

// two time steps in one launch
template <typename T, typename R>
void launch_two(lbm_axi_case *c, const Phys<R> &P)
{
    const T *fin = (const T *)c->pop[c->cur][0], *gin = (const T *)c->pop[c->cur][1];
    T *fout = (T *)c->pop[c->cur ^ 1][0], *gout = (T *)c->pop[c->cur ^ 1][1];
    const T *ain = (const T *)c->aux[c->cur];
    T *aout = (T *)c->aux[c->cur ^ 1];
    const Phys<R> P0 = phys_at(P, c->t);
    const R gz1 = phys_at(P, c->t + 1).g_z;
    const int nr = c->prm.nr, nz = c->prm.nz;
    const TwoStepPlan &w = c->two;
    auto go = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if (w.march) {
            const int strips = pair_strips(nz, c->prm.z_periodic, w.waves), runs = (nr + w.rows - 1) / w.rows;
            pair_kernel<T, R, MODE><<<strips * runs, 64 * w.waves, pair_lds_bytes<R, MODE>(w.waves), c->stream>>>(
                c->geom, P0, gz1, strips, w.rows, fin, gin, fout, gout, ain, aout);
            return;
        }
        with_tile_shape(w.tile, [&](auto shape) {
            using S = decltype(shape);
            const int tiles_z = (nz + S::OZ - 1) / S::OZ, tiles = tiles_z * ((nr + S::OR - 1) / S::OR);
            tile_kernel<T, R, MODE, S><<<tiles, S::THREADS, S::LDS_VALUES * sizeof(R), c->stream>>>(
                c->geom, P0, gz1, tiles_z, fin, gin, fout, gout, ain, aout);
        });
    };
    if (P.mode == COLLIDE_MRT_UNIT)
        go(std::integral_constant<int, COLLIDE_MRT_UNIT>{});
    else if (P.mode == COLLIDE_SRT)
        go(std::integral_constant<int, COLLIDE_SRT>{});
    else if (P.mode == COLLIDE_NMRT)
        go(std::integral_constant<int, COLLIDE_NMRT>{});
    else
        go(std::integral_constant<int, COLLIDE_MRT>{});
}

int do_steps(lbm_axi_case *c, int64_t n)
{
    const bool rec = n > 0 && recording(c->stream);
    c->recorded = c->recorded || rec;
    int64_t pairs = 0;
    if (c->prm.precision != LBM_AXI_FP16D && c->two.tile >= 0) pairs = pairs_of(n, rec, c->recorded);
    for (n -= 2 * pairs; pairs > 0; --pairs) {
        if (c->prm.precision == LBM_AXI_FP64)
            launch_two<double, double>(c, c->P64);
        else
            launch_two<float, float>(c, c->P32);
        c->cur ^= 1;
        c->t += 2;
    }
    for (int64_t s = 0; s < n; ++s) {
        if (c->prm.precision == LBM_AXI_FP64)
            launch_step_tr<double, double>(c, phys_at(c->P64, c->t));
        else if (c->prm.precision == LBM_AXI_FP16D)
            launch_step_h_tr(c);
        else
            launch_step_tr<float, float>(c, phys_at(c->P32, c->t));
        c->cur ^= 1;
        c->t += 1;
    }
    return launch_ok();
}

constexpr int MOM_TR = 4;

// the double planes of the moments fields: the population buffer the next
// step writes (between steps it holds nothing that is still needed; 72 or 144
// bytes per node against 40), with FP16-deviation storage, whose buffers are
// smaller, planes of their own
Fields case_fields(const lbm_axi_case *c)
{
    const int64_t pl = c->geom.plane;
    double *f = c->prm.precision == LBM_AXI_FP16D ? c->xfer - 4 * pl : (double *)c->pop[c->cur ^ 1][0];
    return Fields{f, f + pl, f + 2 * pl, f + 3 * pl, f + 4 * pl};
}

// the macroscopic prefix of the step from time t: the fields that F asks for
// (FP16-deviation storage: all), and the sums' partials
void launch_moments(lbm_axi_case *c, const Geom &g, const Fields &F, double *scratch)
{
    const int nb = moments_blocks(g), gas = c->prm.dispersed_gas;
    if (c->prm.precision == LBM_AXI_FP64)
        moments_kernel<double, double, MOM_TR><<<nb, TZ * MOM_TR, 0, c->stream>>>(
            g, phys_at(c->P64, c->t), (const double *)c->pop[c->cur][0], (const double *)c->pop[c->cur][1],
            (const double *)c->aux[c->cur], F, gas, scratch);
    else if (c->prm.precision == LBM_AXI_FP16D)
        moments_kernel_h<MOM_TR><<<nb, TZ * MOM_TR, 0, c->stream>>>(g, phys_at(c->P32, c->t), c->codec,
                                                                    half_state(c, c->cur), F, gas, scratch);
    else
        moments_kernel<float, float, MOM_TR><<<nb, TZ * MOM_TR, 0, c->stream>>>(
            g, phys_at(c->P32, c->t), (const float *)c->pop[c->cur][0], (const float *)c->pop[c->cur][1],
            (const float *)c->aux[c->cur], F, gas, scratch);
}

// The read-back of a case: fields into F (phi and p at least), the diagnostics
// record into the device record `out`; `scratch` holds the reductions' partials
// (DIAG_SCRATCH_DOUBLES doubles; nothing in it needs to start at zero).
int run_readback(lbm_axi_case *c, const Fields &F, double *scratch, lbm_axi_diag *out)
{
    const Geom g = geom_for(c, MOM_TR);
    const int gas = c->prm.dispersed_gas;
    const int nb = moments_blocks(g);
    launch_moments(c, g, F, scratch);
    const int64_t nn = (int64_t)g.nr * g.nz;
    const int np = (int)std::min<int64_t>(PRS_BLOCKS, (nn + DIAG_THREADS - 1) / DIAG_THREADS);
    diag_pressure<<<np, DIAG_THREADS, 0, c->stream>>>(g, gas, c->prm.W, F, nb, scratch);
    diag_final<<<1, DIAG_THREADS, 0, c->stream>>>(g, gas, nb, np, scratch, F.phi, c->t, out);
    return launch_ok();
}

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

} // namespace

namespace axi {
bool recording(hipStream_t stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    // the null stream cannot be recorded, but asking about it while a blocking
    // stream is recorded is an error, which the next launch check would report
    (void)hipGetLastError();
    return false;
}

int pair_strips(int nz, int z_periodic, int waves)
{
    const int lanes = 64 * waves, inner = lanes - 2 * PAIR_HALO;
    if (z_periodic ? nz == lanes : nz <= lanes) return 1;
    return (nz + inner - 1) / inner;
}

// The march's workgroup is the one with the fewest lanes over all strips (lanes
// that only hold a halo cost what the others do: 64 cases of 512 columns in
// FP32 took 155.8 us a step in one strip of 8 wavefronts, 167 in three of 3, 219
// in ten of 1; strips that share lines cost 3 % more), the smallest of equals;
// then the shortest runs of rows that fill the resident wavefronts of the
// fullest XCD once (or the fewest times), a run costing about 10 rows more than it owns:
// its start and the rows recomputed at its ends (512 x 2048 in FP32: runs of 8
// rows 30.8 us a step, of 12 31.2, of 32 over 35; the 64 cases: 4 runs 155.8, 6
// runs 185, 8 runs 164.8).  Tall and narrow cases have many runs: 19200 x 64
// takes 27.9 us in them, 90 in 256 runs, 44.7 singly; 300000 x 4 194, 1275 and
// 284.  A batch deals whole runs to the XCDs (build_pairs): ten FP64 cases of
// 256 x 512 fill every XCD but two once in 10 runs each, those two and so the
// launch twice (105 us a step, singly 83), and all once in 9.
struct MarchCost {
    float launch, row, full;     // us a step: per row of the longest chain, and more by how full the device is
};
constexpr MarchCost MARCH_COST[2][4] = {                                // [precision][COLLIDE_*], 5 to 9 % rms
    {{-4.8f, 1.45f, 0.55f}, {-2.9f, 1.16f, 0.75f}, {-6.7f, 1.54f, 0.39f}, {-4.8f, 1.45f, 0.55f}},   // FP32
    {{-5.8f, 1.72f, 0.32f}, {-4.5f, 1.48f, 0.27f}, {-5.0f, 1.64f, 0.21f}, {-5.8f, 1.72f, 0.32f}},   // FP64
};

// sets waves and rows; what a step is estimated to take, in us
static float plan_march(const lbm_axi_case *const *cases, int n, bool alone, TwoStepPlan &best)
{
    const bool fp64 = cases[0]->prm.precision == LBM_AXI_FP64, unit = cases[0]->P64.mode == COLLIDE_MRT_UNIT;
    // resident wavefronts per compute unit, by LDS (FP64: more than one per
    // SIMD measured no faster, and unevenly filled SIMDs slower)
    const int resident = fp64 ? 4 : (unit ? 12 : 8), most = fp64 ? PAIR_WAVES<double> : PAIR_WAVES<float>;
    const int line = fp64 ? 8 : 16;
    int64_t best_lanes = 0;
    int max_nr = 0;
    for (int i = 0; i < n; ++i) max_nr = std::max(max_nr, cases[i]->prm.nr);
    for (int w = 1; w <= most; ++w) {
        if (resident % w && w != 8) continue;
        int64_t lanes = 0;
        for (int i = 0; i < n; ++i) {
            const lbm_axi_params &p = cases[i]->prm;
            const int strips = pair_strips(p.nz, p.z_periodic, w);
            const bool whole = strips == 1 || pair_inner(p.nz, p.z_periodic, w, strips, line) % line == 0;
            lanes += (int64_t)p.nr * 64 * w * strips * (whole ? 32 : 33);
        }
        if (!best_lanes || lanes < best_lanes) {
            best_lanes = lanes;
            best.waves = w;
        }
    }
    const int64_t slots = std::max(1, cases[0]->cus * (resident / best.waves) / 8);      // of one XCD
    auto fullest_xcd = [&](int rows) {
        int64_t groups[8] = {};
        int next = 0;
        for (int i = 0; i < n; ++i) {
            const lbm_axi_params &p = cases[i]->prm;
            const int strips = pair_strips(p.nz, p.z_periodic, best.waves), runs = (p.nr + rows - 1) / rows;
            if (alone) return ((int64_t)strips * runs + 7) / 8;                          // xcd_tile
            for (int x = 0; x < 8; ++x) groups[(next + x) % 8] += (int64_t)(runs / 8 + (x < runs % 8)) * strips;
            next = (next + runs) % 8;
        }
        return *std::max_element(groups, groups + 8);
    };
    int64_t best_cost = 0, held = 0;
    // every length that a number of equal runs of the tallest case has, from one run on
    for (int rows = max_nr;;) {
        const int64_t groups = fullest_xcd(rows), cost = (groups + slots - 1) / slots * (rows + 10);
        if (!best_cost || cost < best_cost) {
            best_cost = cost;
            best.rows = rows;
            held = std::min(groups, slots);
        }
        if (rows <= 4) break;
        const int runs = (max_nr + rows - 2) / (rows - 1);
        rows = std::max(4, (max_nr + runs - 1) / runs);
    }
    const MarchCost c = MARCH_COST[fp64][cases[0]->P64.mode];
    return c.launch + (float)best_cost * (c.row + c.full * (float)held / (float)slots);
}

// Marching takes too long to start for what fits the caches: one FP32 case of
// 512 x 1024 21.4 us a step against 15.3 in tiles, of 512 x 2048 30 against 27,
// of 700 x 2000 31.5 against 34.8, 16 cases of 256 x 512 47 against 60; FP64,
// 512 x 1024 30 against 26, 600 x 1500 43 against 50.
// Tiles: the shape whose launch is done first.  A compute unit takes its tiles
// together or in turn; either way a step takes what a launch and the first
// latencies do and a share per tile of the fullest unit (of the XCD that has
// most: three cases of 42 x 896 FP32 are 252 tiles of 32 x 16, but 33 on the first
// XCD's 32 units, 9.2 us a step against 7.1 in 16 x 16), more where many of a
// case's tiles lie at its rim and take the boundary rules (TileCost; fitted, 4 to
// 7 % rms, to some 680 cases and batches of 20 to 1250 thousand nodes: 128 x 512
// FP32 4.4 in 16 x 16, 5.1 in 12 x 8, 5.8 in 32 x 16; 300 x 600 FP32 9.4 in 12 x 8,
// 8.0 in 16 x 16, 8.4 in 32 x 16; 256 x 1024 10.0 and 8.9 in the last two, FP64
// 15.0 and 16.3; eight cases of 63 x 608 general MRT FP64 26.6 in 12 x 8, a fifth
// more per tile than four of 256 x 512).
// The general and the non-orthogonal MRT hold more registers: in FP64 a unit
// takes one 16 x 16 tile of theirs at a time, two of the other forms' (256 x 1024
// non-orthogonal 20.9 us a step in 16 x 16, 17.3 in 32 x 16, 17.5 singly; six cases of
// 256 x 512 64.4, 52.3, 51.8; SRT 42.8, 49.8, 51.0).
struct TileCost {
    float launch, tile, rim;      // us a step; rim: per tile, where all are at the rim
};
constexpr TileCost TILE_COST[2][2][TILE_SHAPES] = {                     // [precision][MRT with free rates, non-orthogonal]
    {{{2.95f, 0.72f, 0.21f}, {2.95f, 0.78f, 0.33f}, {2.75f, 1.77f, 0.46f}, {2.75f, 3.16f, 0.6f}},   // FP32
     {{3.0f, 0.83f, 0.24f}, {2.95f, 0.91f, 0.39f}, {2.8f, 2.03f, 0.48f}, {2.75f, 3.5f, 0.75f}}},
    {{{3.15f, 1.15f, 0.38f}, {2.85f, 1.41f, 0.51f}, {2.4f, 3.23f, 0.45f}, {0.0f, 8.1f, 0.65f}},     // FP64
     {{2.75f, 1.38f, 0.48f}, {2.85f, 1.51f, 0.62f}, {0.9f, 4.87f, 0.65f}, {0.15f, 8.3f, 0.63f}}},
};

// us a step in tiles of a shape
static float tiles_us(const lbm_axi_case *const *cases, int n, int shape, const TileCost &c)
{
    const int64_t cus = std::max(1, cases[0]->cus / 8);           // of one XCD
    int64_t fullest = 0, tiles = 0, plain = 0;                    // each case's are dealt out from the first XCD on
    with_tile_shape(shape, [&](auto t) {
        using S = decltype(t);
        // tiles along an axis of m nodes whose halo stays clear of both ends
        auto clear = [](int m, int size) { return m < 6 ? 0 : std::max(0, (m - 6) / size - (size + 5) / size); };
        for (int i = 0; i < n; ++i) {
            const lbm_axi_params &p = cases[i]->prm;
            const int64_t tz = (p.nz + S::OZ - 1) / S::OZ, all = tz * ((p.nr + S::OR - 1) / S::OR);
            fullest += (all + 7) / 8;
            tiles += all;
            plain += clear(p.nr, S::OR) * (p.z_periodic ? tz : clear(p.nz, S::OZ));
        }
    });
    const float rim = (float)(tiles - plain) / (float)tiles;
    return c.launch + (c.tile + c.rim * rim) * (float)((fullest + cus - 1) / cus);
}

// Single steps take more (5.2 us a step of 64 x 128 FP32, 7.8 of 60 x 286 FP64,
// 11.1 of 128 x 2048 FP32), but while each of their 64 x 8 tiles has a unit to
// itself, and the smaller tiles of two steps, by their ragged edges, need a
// round more, they stay ahead: 69 x 1717 FP32 7.7 against 8.2 in the best shape,
// 200 x 640 6.3 against 7.5, FP64 9.7 against 11.1, 133 x 920 9.7 against 11.2.
// Then a step takes a launch and a share per tile by how its rows lie in memory:
// whole 64-byte lines, half ones, neither (fitted likewise, within 5 %; 256 tiles
// FP32 6.2 us in rows of 512 nodes, 7.3 of 504, 8.0 of 511).  Batches of more
// than eight cases were never ahead singly in one round (14 of 30 x 208 FP32 8.7
// against 7.3).  Of several rounds single steps were ahead only in batches of
// small cases, most of whose tiles lie at a rim (161 of 26 x 96 FP32 24.3 against
// 26.6, eight of 63 x 608 general MRT FP64 24.9 against 26.6).
struct SingleCost {
    float launch, line, half, ragged;                             // one round
    float rounds, round, node, rows;                              // several: also per 100,000 nodes and per 256 ragged tiles
};
constexpr SingleCost SINGLE_COST[2][2] = {
    {{4.6f, 0.0068f, 0.0103f, 0.0125f, 4.6f, 1.16f, 2.25f, 1.37f},
     {4.9f, 0.0065f, 0.0101f, 0.0119f, 4.45f, 1.6f, 2.0f, 1.25f}},
    {{5.9f, 0.0148f, 0.0215f, 0.0244f, 6.3f, 3.05f, 3.56f, 1.7f},
     {6.3f, 0.0135f, 0.0209f, 0.024f, 6.6f, 4.1f, 2.75f, 1.76f}},
};
constexpr int SINGLY_CASES = 8, ROUNDS_CASES = 4;
// cases of different tables in one launch: pairs pay half of it per step
constexpr float SEVERAL_CASES = 0.4f;

// us a step of single steps (64 x 8 tiles in 16 bands a case, the default), or
// infinity where two steps are ahead anyway; one: whether it is one round
static float single_us(const lbm_axi_case *const *cases, int n, const SingleCost &c, bool &one)
{
    const int es = cases[0]->prm.precision == LBM_AXI_FP64 ? 8 : 4, cus = std::max(1, cases[0]->cus / 8);
    int fullest = 0, ragged = 0;                                  // tiles on the first XCD, in rows off whole lines
    int64_t nodes = 0;
    float us = c.launch + (n > 1 ? SEVERAL_CASES : 0.0f);
    for (int i = 0; i < n; ++i) {
        const lbm_axi_params &p = cases[i]->prm;
        const int tiles = geom_for(cases[i], 8).tiles, row = p.nz % 64 * es;
        fullest += n == 1 ? (tiles + 7) / 8 : tiles / 16 * 2 + (tiles % 16 > 0) + (tiles % 16 > 8);
        us += (float)tiles * (row % 64 == 0 ? c.line : (row % 32 == 0 ? c.half : c.ragged));
        nodes += (int64_t)p.nr * p.nz;
        ragged += row % 64 ? tiles : 0;
    }
    one = fullest <= cus;
    if (one) return n > SINGLY_CASES ? INFINITY : us;
    return n < ROUNDS_CASES ? INFINITY
                            : c.rounds + c.round * (float)fullest / (float)cus + c.node * 1e-5f * (float)nodes +
                                  c.rows * (float)ragged / 256.0f;
}

TwoStepPlan two_step_plan(const lbm_axi_case *const *cases, int n, bool alone)
{
    TwoStepPlan plan{false, 1, 4, 0, 0.0f, INFINITY};
    const bool fp64 = cases[0]->prm.precision == LBM_AXI_FP64;
    int64_t nodes = 0;
    for (int i = 0; i < n; ++i) nodes += (int64_t)cases[i]->prm.nr * cases[i]->prm.nz;
    plan.march = nodes >= (fp64 ? 800000 : 1200000);
    if (plan.march) {
        plan_march(cases, n, alone, plan);
        return plan;
    }
    const int mode = cases[0]->P64.mode;
    const bool heavy = mode == COLLIDE_MRT || mode == COLLIDE_NMRT;
    for (int shape = 0; shape < TILE_SHAPES; ++shape) {
        const float us = tiles_us(cases, n, shape, TILE_COST[fp64][heavy][shape]);
        if (shape == 0 || us <= plan.pairs_us) {
            plan.pairs_us = us;
            plan.tile = shape;
        }
    }
    bool one;
    plan.single_us = single_us(cases, n, SINGLE_COST[fp64][heavy], one);
    if (!one && plan.single_us < 1.15f * plan.pairs_us) {
        // tiles hardly pay: then the march may (161 cases of 26 x 96 FP32 21.9 us a step)
        TwoStepPlan march = plan;
        march.march = true;
        march.pairs_us = plan_march(cases, n, alone, march);
        if (march.pairs_us < plan.pairs_us && !singly_ahead(plan.single_us, march.pairs_us)) return march;
    }
    if (alone && singly_ahead(plan.single_us, plan.pairs_us)) plan.tile = -1;
    return plan;
}

// Rows of the single step's tile where the caller names none: 8, or, in
// FP16-deviation storage, 4 while every such tile has a compute unit to itself
// (then it is the time of one tile that counts: 150 x 300 5.6 us a step against
// 6.1, 128 x 256 5.4 against 5.7; beyond, the larger share of ring costs more:
// 256 x 512 6.3 against 6.0).  Not where the last tile column holds a few
// columns only, nearly all of it ghost cells, of which a thread of the smaller
// tile takes two (200 x 65 8.2 us against 7.6, 60 x 321 with walls 8.3 against
// 7.0), nor for the non-orthogonal MRT, whose registers spill (60 x 344 6.5
// against 6.2, 200 x 48 6.3 against 6.1).  FP64 and FP32: 64 x 128 FP32 measured
// the same either way.
int default_tile(const lbm_axi_case *c)
{
    if (c->prm.precision != LBM_AXI_FP16D || c->P64.mode == COLLIDE_NMRT) return 8;
    const int last = c->prm.nz % TZ;
    if (last > 0 && last <= 10) return 8;
    const int64_t tiles = (int64_t)((c->prm.nz + TZ - 1) / TZ) * ((c->prm.nr + 3) / 4);
    return tiles <= c->cus ? 4 : 8;
}

HalfBuf half_buf(const lbm_axi_case *c, int b)
{
    const int64_t pl = c->geom.plane;
    HalfBuf B;
    B.f0 = (float *)c->pop[b][0];
    B.f = (half_t *)((char *)c->pop[b][0] + pl * 4);
    B.g = (half_t *)c->pop[b][1];
    // aux planes: phase field of side 0, u_z, u_r, phase field of side 1
    B.phi = (float *)c->aux[0] + (b ? 3 * pl : 0);
    return B;
}

HalfState half_state(const lbm_axi_case *c, int cur)
{
    HalfBuf in = half_buf(c, cur), out = half_buf(c, cur ^ 1);
    HalfState S;
    S.f0in = in.f0;
    S.fin = in.f;
    S.gin = in.g;
    S.phin = in.phi;
    S.f0out = out.f0;
    S.fout = out.f;
    S.gout = out.g;
    S.phout = out.phi;
    S.uz = (float *)c->aux[0] + c->geom.plane;
    S.ur = (float *)c->aux[0] + 2 * c->geom.plane;
    return S;
}

Geom geom_for(const lbm_axi_case *c, int tile_r)
{
    Geom g;
    g.nr = c->prm.nr;
    g.nz = c->prm.nz;
    g.zper = c->prm.z_periodic;
    g.plane = plane_elems(g.nr, g.nz);
    g.tiles_z = (g.nz + TZ - 1) / TZ;
    g.tiles = g.tiles_z * ((g.nr + tile_r - 1) / tile_r);
    return g;
}
} // namespace axi

namespace {
typedef float copy_vec __attribute__((ext_vector_type(4)));

// one 16-byte element per thread, non-temporal both ways: on this part the
// fastest plain copy measured (against grid-stride loops and unrolled forms)
__global__ __launch_bounds__(256) void device_copy_kernel(const copy_vec *__restrict__ src,
                                                          copy_vec *__restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}
} // namespace

// The planes of a state through the transfer plane, in stream order: the caller
// waits once, for all of them (and on an error for what was enqueued before it).
static int enqueue_get(lbm_axi_case *c, double *f, double *g, double *aux)
{
    Geom G = c->geom;
    int64_t nn = (int64_t)G.nr * G.nz;
    unsigned nb = blocks_for(nn, 256);
    const bool half = c->prm.precision == LBM_AXI_FP16D;
    double *outs[2] = {f, g};
    for (int q = 0; q < 2; ++q) {
        if (!outs[q]) continue;
        for (int i = 0; i < 9; ++i) {
            if (half)
                gather_plane_h<<<nb, 256, 0, c->stream>>>(G, c->codec, half_buf(c, c->cur), i, q, c->xfer);
            else if (c->prm.precision == LBM_AXI_FP64)
                gather_plane_kernel<double><<<nb, 256, 0, c->stream>>>(G, i, (const double *)c->pop[c->cur][q], c->xfer);
            else
                gather_plane_kernel<float><<<nb, 256, 0, c->stream>>>(G, i, (const float *)c->pop[c->cur][q], c->xfer);
            if (launch_ok()) return LBM_AXI_EDEVICE;
            HIP_OK(hipMemcpyAsync(outs[q] + i * nn, c->xfer, nn * sizeof(double), hipMemcpyDeviceToHost, c->stream));
        }
    }
    if (aux) {
        for (int q = 0; q < 3; ++q) {
            if (half)
                convert_kernel<float, double><<<nb, 256, 0, c->stream>>>(
                    nn, q == 0 ? half_buf(c, c->cur).phi : (const float *)c->aux[0] + q * G.plane, c->xfer);
            else if (c->prm.precision == LBM_AXI_FP64)
                convert_kernel<double, double><<<nb, 256, 0, c->stream>>>(nn, (const double *)c->aux[c->cur] + q * G.plane, c->xfer);
            else
                convert_kernel<float, double><<<nb, 256, 0, c->stream>>>(nn, (const float *)c->aux[c->cur] + q * G.plane, c->xfer);
            if (launch_ok()) return LBM_AXI_EDEVICE;
            HIP_OK(hipMemcpyAsync(aux + q * nn, c->xfer, nn * sizeof(double), hipMemcpyDeviceToHost, c->stream));
        }
    }
    return LBM_AXI_OK;
}

static int enqueue_set(lbm_axi_case *c, const double *f, const double *g, const double *aux)
{
    Geom G = c->geom;
    int64_t nn = (int64_t)G.nr * G.nz;
    unsigned nb = blocks_for(nn, 256);
    const bool half = c->prm.precision == LBM_AXI_FP16D;
    if (half) {
        // the stored phase field first: FP16 f values are encoded against it
        for (int q = 0; q < 3; ++q) {
            HIP_OK(hipMemcpyAsync(c->xfer, aux + q * nn, nn * sizeof(double), hipMemcpyHostToDevice, c->stream));
            convert_kernel<double, float><<<nb, 256, 0, c->stream>>>(
                nn, c->xfer, q == 0 ? half_buf(c, c->cur).phi : (float *)c->aux[0] + q * G.plane);
            if (launch_ok()) return LBM_AXI_EDEVICE;
        }
    }
    const double *ins[2] = {f, g};
    for (int q = 0; q < 2; ++q)
        for (int i = 0; i < 9; ++i) {
            HIP_OK(hipMemcpyAsync(c->xfer, ins[q] + i * nn, nn * sizeof(double), hipMemcpyHostToDevice, c->stream));
            if (half)
                scatter_plane_h<<<nb, 256, 0, c->stream>>>(G, c->codec, half_buf(c, c->cur), i, q, c->xfer);
            else if (c->prm.precision == LBM_AXI_FP64)
                scatter_plane_kernel<double><<<nb, 256, 0, c->stream>>>(G, i, c->xfer, (double *)c->pop[c->cur][q]);
            else
                scatter_plane_kernel<float><<<nb, 256, 0, c->stream>>>(G, i, c->xfer, (float *)c->pop[c->cur][q]);
            if (launch_ok()) return LBM_AXI_EDEVICE;
        }
    for (int q = 0; q < 3 && !half; ++q) {
        HIP_OK(hipMemcpyAsync(c->xfer, aux + q * nn, nn * sizeof(double), hipMemcpyHostToDevice, c->stream));
        if (c->prm.precision == LBM_AXI_FP64)
            convert_kernel<double, double><<<nb, 256, 0, c->stream>>>(nn, c->xfer, (double *)c->aux[c->cur] + q * G.plane);
        else
            convert_kernel<double, float><<<nb, 256, 0, c->stream>>>(nn, c->xfer, (float *)c->aux[c->cur] + q * G.plane);
        if (launch_ok()) return LBM_AXI_EDEVICE;
    }
    return LBM_AXI_OK;
}

static int finish(lbm_axi_case *c, int rc)
{
    const hipError_t e = hipStreamSynchronize(c->stream);
    return rc ? rc : (e == hipSuccess ? LBM_AXI_OK : LBM_AXI_EDEVICE);
}

extern "C" {

size_t lbm_axi_state_bytes(const lbm_axi_params *params)
{
    if (validate(params) != LBM_AXI_OK) return 0;
    return layout_of(params).total;
}

int lbm_axi_init(const lbm_axi_params *params, void *dev_state, size_t dev_bytes,
                 const double *phi0_host, void *hip_stream, lbm_axi_case **out)
{
    if (!out) return LBM_AXI_EINVAL;
    *out = nullptr;
    int rc = validate(params);
    if (rc) return rc;
    if (!dev_state || !phi0_host || ((uintptr_t)dev_state & 255)) return LBM_AXI_EINVAL;
    Layout L = layout_of(params);
    if (dev_bytes < L.total) return LBM_AXI_ENOMEM;

    // the allocation-free read-back's scratch address on this device, taken
    // here with the device current
    int dev = 0;
    double *scratch_ptr = nullptr;
    if (hipGetDevice(&dev) != hipSuccess || noalloc_scratch(dev, &scratch_ptr) != LBM_AXI_OK) return LBM_AXI_EDEVICE;
    lbm_axi_case *c = new (std::nothrow) lbm_axi_case;
    if (!c) return LBM_AXI_ENOMEM;
    c->device = dev;
    c->prm = *params;
    c->stream = (hipStream_t)hip_stream;
    c->base = (char *)dev_state;
    c->bytes = dev_bytes;
    c->t = 0;
    c->cur = 0;
    c->recorded = false;
    c->cus = 256;
    (void)hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, dev);
    c->esize = L.esize;
    for (int b = 0; b < 2; ++b)
        for (int q = 0; q < 2; ++q)
            c->pop[b][q] = c->base + L.off_pop + (size_t)b * (L.fbytes + L.gbytes) + (size_t)q * L.fbytes;
    c->aux[0] = c->base + L.off_aux;
    c->aux[1] = params->precision == LBM_AXI_FP16D ? nullptr : (void *)(c->base + L.off_fld);
    c->xfer = (double *)(c->base + L.off_fld) + 4 * L.plane;
    c->part = (double *)(c->base + L.off_part);
    c->diag = (lbm_axi_diag *)(c->base + L.off_diag);
    c->P64 = make_phys<double>(params);
    c->P32 = make_phys<float>(params);
    c->codec = make_codec(params);
    c->tile_r = default_tile(c);
    c->geom = geom_for(c, c->tile_r);
    c->two = two_step_plan(&c, 1, true);

    int64_t nn = (int64_t)params->nr * params->nz;
    if (hipMemcpyAsync(c->xfer, phi0_host, nn * sizeof(double), hipMemcpyHostToDevice, c->stream) != hipSuccess) {
        delete c;
        return LBM_AXI_EDEVICE;
    }
    if (params->precision == LBM_AXI_FP64)
        init_kernel<double><<<blocks_for(nn, 256), 256, 0, c->stream>>>(
            c->geom, c->xfer, (double *)c->pop[0][0], (double *)c->pop[0][1], (double *)c->aux[0]);
    else if (params->precision == LBM_AXI_FP16D)
        init_kernel_h<<<blocks_for(nn, 256), 256, 0, c->stream>>>(c->geom, c->codec, c->xfer, half_buf(c, 0),
                                                                   (float *)c->aux[0] + c->geom.plane,
                                                                   (float *)c->aux[0] + 2 * c->geom.plane);
    else
        init_kernel<float><<<blocks_for(nn, 256), 256, 0, c->stream>>>(
            c->geom, c->xfer, (float *)c->pop[0][0], (float *)c->pop[0][1], (float *)c->aux[0]);
    if (launch_ok() != LBM_AXI_OK || hipStreamSynchronize(c->stream) != hipSuccess) {
        delete c;
        return LBM_AXI_EDEVICE;
    }
    *out = c;
    return LBM_AXI_OK;
}

int lbm_axi_step(lbm_axi_case *c, int64_t nsteps)
{
    if (!c) return LBM_AXI_ESTATE;
    if (nsteps < 0) return LBM_AXI_EINVAL;
    return do_steps(c, nsteps);
}

int lbm_axi_moments(lbm_axi_case *c, double *phi, double *rho, double *uz, double *ur, double *p,
                    lbm_axi_diag *diag)
{
    if (!c) return LBM_AXI_ESTATE;
    const int64_t nn = (int64_t)c->prm.nr * c->prm.nz, pl = c->geom.plane;
    auto copy_out = [&](double *out, const double *plane) {
        return out ? hipMemcpyAsync(out, plane, nn * sizeof(double), hipMemcpyDeviceToHost, c->stream) : hipSuccess;
    };
    if (c->recorded && c->prm.precision != LBM_AXI_FP16D) {
        // a graph may hold a state in either population buffer: the fields go
        // through the two planes that nothing else keeps, two at a time
        double *const a = c->xfer - pl, *const b = c->xfer;
        const Geom g = geom_for(c, MOM_TR);
        int rc = run_readback(c, Fields{a, nullptr, nullptr, nullptr, b}, c->part, c->diag);
        if (rc) return rc;
        HIP_OK(copy_out(phi, a));
        HIP_OK(copy_out(p, b));
        if (rho || uz) {
            launch_moments(c, g, Fields{nullptr, a, b, nullptr, nullptr}, c->part);
            HIP_OK(copy_out(rho, a));
            HIP_OK(copy_out(uz, b));
        }
        if (ur) {
            launch_moments(c, g, Fields{nullptr, nullptr, nullptr, a, nullptr}, c->part);
            HIP_OK(copy_out(ur, a));
        }
        if (launch_ok()) return LBM_AXI_EDEVICE;
    } else {
        const Fields F = case_fields(c);
        int rc = run_readback(c, F, c->part, c->diag);
        if (rc) return rc;
        double *outs[5] = {phi, rho, uz, ur, p};
        const double *planes[5] = {F.phi, F.rho, F.uz, F.ur, F.p};
        for (int q = 0; q < 5; ++q) HIP_OK(copy_out(outs[q], planes[q]));
    }
    lbm_axi_diag d;
    HIP_OK(hipMemcpyAsync(&d, c->diag, sizeof(lbm_axi_diag), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(hipStreamSynchronize(c->stream));
    if (diag) *diag = d;
    if (d.nonfinite > 0 || !(d.umax <= CS)) return LBM_AXI_EUNSTABLE;
    return LBM_AXI_OK;
}

int lbm_axi_moments_noalloc(lbm_axi_case *c, double *phi, double *rho, double *uz, double *ur, double *p,
                            lbm_axi_diag *diag)
{
    if (!c) return LBM_AXI_ESTATE;
    if (!phi || !rho || !uz || !ur || !p || !diag) return LBM_AXI_EINVAL;
    if ((int64_t)c->prm.nr * c->prm.nz > ((int64_t)1 << 25)) return LBM_AXI_EINVAL;
    double *sc = nullptr;
    if (noalloc_scratch(c->device, &sc) != LBM_AXI_OK) return LBM_AXI_EDEVICE;
    c->recorded = c->recorded || recording(c->stream);
    return run_readback(c, Fields{phi, rho, uz, ur, p}, sc, diag);
}

int lbm_axi_get_state(lbm_axi_case *c, double *f, double *g, double *aux, int64_t *t)
{
    if (!c) return LBM_AXI_ESTATE;
    const int rc = finish(c, enqueue_get(c, f, g, aux));
    if (rc) return rc;
    if (t) *t = c->t;
    return LBM_AXI_OK;
}

int lbm_axi_set_state(lbm_axi_case *c, const double *f, const double *g, const double *aux, int64_t t)
{
    if (!c) return LBM_AXI_ESTATE;
    if (!f || !g || !aux || t < 0) return LBM_AXI_EINVAL;
    const int rc = finish(c, enqueue_set(c, f, g, aux));
    if (rc) return rc;
    c->t = t;
    return LBM_AXI_OK;
}

int lbm_axi_time(const lbm_axi_case *c, int64_t *t)
{
    if (!c || !t) return c ? LBM_AXI_EINVAL : LBM_AXI_ESTATE;
    *t = c->t;
    return LBM_AXI_OK;
}

int lbm_axi_set_tile(lbm_axi_case *c, int32_t tile_r)
{
    if (!c) return LBM_AXI_ESTATE;
    if (tile_r == 0) tile_r = default_tile(c);
    if (tile_r != 2 && tile_r != 4 && tile_r != 8 && tile_r != 16) return LBM_AXI_EINVAL;
    c->tile_r = tile_r;
    c->geom = geom_for(c, tile_r);
    return LBM_AXI_OK;
}

int lbm_axi_destroy(lbm_axi_case *c)
{
    delete c;
    return LBM_AXI_OK;
}

int lbm_axi_device_copy(const void *src, void *dst, size_t bytes, void *hip_stream)
{
    if (bytes == 0)
        return LBM_AXI_OK;
    const size_t n = bytes / 16, blocks = (n + 255) / 256;
    if (!src || !dst || bytes % 16 || ((uintptr_t)src | (uintptr_t)dst) % 16 || blocks > (size_t)INT32_MAX)
        return LBM_AXI_EINVAL;
    const uintptr_t s0 = (uintptr_t)src, d0 = (uintptr_t)dst;
    if (s0 < d0 + bytes && d0 < s0 + bytes)
        return LBM_AXI_EINVAL;
    device_copy_kernel<<<(unsigned)blocks, 256, 0, (hipStream_t)hip_stream>>>((const copy_vec *)src, (copy_vec *)dst, n);
    return hipGetLastError() == hipSuccess ? LBM_AXI_OK : LBM_AXI_EDEVICE;
}

const char *lbm_axi_strerror(int code)
{
    switch (code) {
    case LBM_AXI_OK: return "ok";
    case LBM_AXI_EINVAL: return "invalid argument or parameter";
    case LBM_AXI_ENOMEM: return "device block smaller than lbm_axi_state_bytes()";
    case LBM_AXI_EDEVICE: return "HIP runtime error";
    case LBM_AXI_EUNSTABLE: return "non-finite field or |u| above the lattice sound speed";
    case LBM_AXI_EBUSY: return "no free slot or memory";
    case LBM_AXI_ESTATE: return "invalid handle or slot";
    default: return "unknown error";
    }
}

} // extern "C"
