// Internal definitions shared by the translation units of liblbm_axi.so.
#pragma once

#include "axi_device.hpp"
#include "axi_half.hpp"
#include "axi_pair.hpp"
#include "axi_tile.hpp"
#include "../../include/lbm_axi.h"

#include <stddef.h>

struct lbm_axi_case;

namespace axi {

constexpr int TZ = 64;          // tile width along z: one wave per tile row
#ifndef AXI_PLANE_PAD
#define AXI_PLANE_PAD 64
#endif
constexpr int PLANE_PAD = AXI_PLANE_PAD;   // spare elements per population plane

// How the cases of one launch advance two steps at once (FP64 and FP32).
struct TwoStepPlan {
    bool march;            // strips marching up the rows (axi_pair.hpp), else tiles (axi_tile.hpp)
    int waves, rows;       // march: wavefronts of a workgroup, rows of a run
    int tile;              // tiles: the shape (with_tile_shape); -1: steps go singly
    float pairs_us;        // what a step is estimated to take so, and what a
    float single_us;       // single one is (infinite where it is no choice)
};
// single steps are chosen within the estimates' error of 4 %
inline bool singly_ahead(float single_us, float pairs_us) { return single_us < 1.04f * pairs_us; }

} // namespace axi

// One case: its geometry, rates and the pointers into its device block.
struct lbm_axi_case {
    lbm_axi_params prm;
    hipStream_t stream;
    char *base;
    size_t bytes;
    int64_t t;
    int cur;               // ping-pong buffer holding the current state
    int tile_r;
    int cus;               // compute units of the device
    axi::TwoStepPlan two;  // of the case's own launches
    bool recorded;         // a caller's graph holds steps or a read-back of it (pairs_of)
    int device;            // HIP device the case was initialised on
    axi::Geom geom;             // geometry of the step launch (tiles for tile_r)
    axi::Phys<double> P64;
    axi::Phys<float> P32;
    axi::Codec codec;      // FP16-deviation storage scales
    size_t esize;          // bytes per stored value (FP16-deviation: 2)
    void *pop[2][2];       // [buffer][f or g]
    void *aux[2];          // [buffer]; FP16-deviation storage: all its aux planes at [0]
    double *xfer;          // one double plane: state transfer, initial phase field
    double *part;          // per-workgroup partials of the diagnostics reductions
    lbm_axi_diag *diag;    // the diagnostics record, reduced on the device
};

namespace axi {
// geometry of the step launch for a given tile height
Geom geom_for(const lbm_axi_case *c, int tile_r);
// elements between population planes of an nr x nz case
int64_t plane_elems(int nr, int nz);
// how many strips `waves` wavefronts cut nz columns into (axi_pair.hpp)
int pair_strips(int nz, int z_periodic, int waves);
// two steps per launch for the n cases of one launch: the plan that suits them
// (alone: the one case's own launch, which then may also be to step singly;
// else a batch's, which decides for all its launches)
TwoStepPlan two_step_plan(const lbm_axi_case *const *cases, int n, bool alone);
// rows of the single step's tile where the caller names none
int default_tile(const lbm_axi_case *c);
// whether what is enqueued on the stream now is being recorded into a graph
bool recording(hipStream_t stream);
// how many of n steps go in pairs.  A graph holds the addresses of the buffer
// that was current when it was recorded, and a replay starts there: what is
// recorded (rec) goes singly, so that 2 m steps end in the buffer they began
// in, and from then on (recorded) n steps enqueued live leave the buffer where
// n single steps would, which an even number of pairs does.
inline int64_t pairs_of(int64_t n, bool rec, bool recorded) { return rec ? 0 : (recorded ? n / 4 * 2 : n / 2); }
// FP16-deviation storage: buffers of ping-pong side b, and the step from side cur
struct HalfBuf {
    float *f0;       // f_0 plane (FP32)
    half_t *f;       // f_1..f_8 planes (FP16), plane p at f + (p - 1) * plane
    half_t *g;       // g_0..g_8 planes (FP16)
    float *phi;      // stored phase field of side b
};
HalfBuf half_buf(const lbm_axi_case *c, int b);
HalfState half_state(const lbm_axi_case *c, int cur);
} // namespace axi
