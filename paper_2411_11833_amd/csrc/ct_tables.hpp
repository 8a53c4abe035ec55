// Device-resident description of one skeleton's constraint problem.
//
// Built once on the host from the C-ABI descriptors and uploaded to HBM; every
// kernel reads it through a __restrict__ const pointer with wave-uniform
// indices, so the compiler serves it from the scalar cache (SGPR operands)
// rather than spending VGPRs, LDS or vector memory instructions on it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cutamp.h"

namespace ct {

// what a particle-kernel launch produces
enum Mode { MODE_COST = 0, MODE_GRAD = 1, MODE_STEP = 2 };

// lanes per workgroup of the particle kernel (four wave64s)
constexpr int WG = 256;

// Iterations of one launch of the fused step at most: bounds a launch's time
// (an iteration of 200,000 particles takes about a millisecond) at a staging
// cost of a few microseconds every 64 iterations.
constexpr int MAX_LAUNCH_ITERS = 64;

// One joint and its link's spheres, read as one block of scalars: the
// Denavit-Hartenberg constants, the link's robot spheres rs[s0 .. s0 + ns),
// and the sphere holding all of them (as lbs).  Entry 7 is the tool (no joint).
struct alignas(64) Joint {
    float ca, sa, a, d, th0;
    int s0, ns, pad0;
    float4 lb;
    float pad1[4];
};

// A yaw-only oriented box: centre, cos/sin of its yaw, half extents.
struct Box {
    float cx, cy, cz, c, s, hx, hy, hz;
};

// A box that never moves, stored for the point-in-box-frame transform
// p = R^T (x - t) = (c x + s y + u0, c y - s x + u1, z - tz) with
// u0 = -(c tx + s ty), u1 = s tx - c ty (two FMAs per horizontal axis).
struct SBox {
    float c, s, u0, u1, tz, hx, hy, hz;
};

// A box for the bounding-sphere culling tests, an upright cylinder around it:
// for a static box m2x, m2y = -2 (cx, cy) and kc = -(cx^2 + cy^2) + a margin
// for the rounding of the test; for a moved object m2x, m2y = (cx, cy) of its
// initial pose.  z, hz: centre height and half height; r: footprint circle.
struct CullBox {
    float m2x, m2y, z, hz, r, kc, pad0, pad1;
};

// weight slots
enum { W_KPOS, W_KROT, W_GRASP, W_PLACE, W_JLIM, W_COLL, W_GOAL, W_TRAJ, W_MCOLL, W_SELF, W_N };
// tolerance slots
enum { E_KPOS, E_KROT, E_GRASP, E_PLACE, E_JLIM, E_COLL, E_MCOLL, E_SELF, E_N };

// term index of each kind inside one step's block of CT_TERMS_PER_STEP
enum {
    T_PICK_POS = 0, T_PICK_ROT, T_PLACE_POS, T_PLACE_ROT, T_GRASP, T_PLACE,
    T_JLIM_G, T_JLIM_P, T_COLL_G, T_COLL_P, T_COLL_OBJ
};

struct Tables {
    int K;             // pick-place steps
    int D;             // particle dimension = 21 K
    int n_terms;       // all terms
    int n_constraint;  // terms that enter the mask
    int n_static;      // boxes that never move (table, obstacles, unmoved objects)
    int n_os;          // spheres per object
    int goal;          // pairwise placed-object distance cost on/off
    int W;             // interior waypoints per transition (0 = no motion cost)
    int goal_term;     // index of the goal term (or -1)
    int traj_term;     // index of the TrajLength term (or -1)
    int self_on;       // robot self-collision constraint at the key configurations on/off
    int self_term;     // index of the first self-collision term (slot s adds s), or -1
    Joint jk[CT_N_JOINTS + 1];
    int link_start[10];  // robot spheres of link L (1..8) are rs[link_start[L] .. link_start[L+1])
    float q_lo[CT_N_JOINTS], q_hi[CT_N_JOINTS];
    float tool_d;
    float q0[CT_N_JOINTS];
    float w[W_N];
    float eps[E_N];
    float region_lo[2], region_hi[2];
    float4 rs[CT_MAX_ROBOT_SPHERES];           // (x, y, z, r) in the parent frame, grouped by link
    float4 lbs[10];                            // per link L: sphere (centre in the link frame, radius) holding
                                               // all of L's robot spheres, radius grown by a margin; w < 0: none
    SBox sbox[CT_MAX_STATIC_BOXES];
    CullBox cbx[CT_MAX_STATIC_BOXES + CT_MAX_STEPS];   // the n_static static boxes, then the K moved objects
    float2 ck[8 * (CT_MAX_STATIC_BOXES + CT_MAX_STEPS)];   // [8][n_static + K]: thresholds of link L's bounding
                                               // sphere against each (xy as in the culling test, z)
    Box obj0[CT_MAX_STEPS];                    // moved object of step k at its initial pose
    float p0_yaw[CT_MAX_STEPS];                // its initial yaw
    float place_z[CT_MAX_STEPS];               // centre height when placed on the table
    float grasp_lo[CT_MAX_STEPS][3], grasp_hi[CT_MAX_STEPS][3];
    float4 os[CT_MAX_STEPS][CT_MAX_OBJ_SPHERES];  // object spheres (object frame) of step k's object
    float4 obs[CT_MAX_STEPS];                  // sphere holding all of step k's object spheres (as lbs)
    float lo[CT_MAX_STEPS * CT_STEP_DIM];      // uniform-initialization box
    float hi[CT_MAX_STEPS * CT_STEP_DIM];
};

// particles per workgroup tile for a K-step skeleton and SPLIT lanes per slot
__host__ __device__ constexpr int tile_particles(int K, int SPLIT) { return WG / (2 * K * SPLIT); }

// A tile may hold fewer particles, `per`, than its P columns: they are spread
// evenly (particle j in column ceil(j P / per)) and the lanes of the empty
// columns only help with the sphere-box tests of their wave.

// Byte offsets of a tile's LDS for a K-step skeleton (mode MODE_*, W
// waypoints, n_static static boxes, n_rs robot spheres).  Arrays whose size
// the skeleton length alone decides come first.
struct TileLayout {
    int xs, ms, vs, plc, cpart, flg, okp, wave, osl, ob0, frz, ctl, bc, sbx, cbx, tpart, hpart, rs, ck, part, total;
    // floats of one lane's gradient partials, and of a particle's: both odd, so
    // that neighbouring lanes and particles start in different banks
    int np, pp;
};

__host__ __device__ inline TileLayout tile_layout(int K, int split, int mode, int W, int n_static, int n_rs) {
    const int P = tile_particles(K, split), slots = P * 2 * K, state = CT_STEP_DIM * K * P * 4;
    const int mv = mode == MODE_STEP && W == 0 ? state : 0;
    TileLayout o{};
    int at = 0;
    auto take = [&](int bytes) {
        const int here = at;
        at += (bytes + 15) & ~15;
        return here;
    };
    o.xs = take(state);
    o.plc = take(K * P * 16);
    o.cpart = take(slots * 4);
    o.flg = take(slots * 4);
    o.okp = take(P * 4);
    o.wave = take(WG / 64 * 2048);
    o.osl = take(K * CT_MAX_OBJ_SPHERES * 16);
    o.ob0 = take(K * (int)sizeof(Box));
    o.frz = take(CT_STEP_DIM * K);
    o.ctl = take(16);
    o.bc = take(mode == MODE_STEP ? MAX_LAUNCH_ITERS * 8 : 0);
    o.ms = take(mv);
    o.vs = take(mv);
    o.sbx = take(n_static * (int)sizeof(SBox));
    o.cbx = take((n_static + K) * (int)sizeof(CullBox));
    o.tpart = take(W > 0 ? slots * 4 : 0);
    o.hpart = take(mode == MODE_COST ? slots * 4 : 0);
    o.rs = take(n_rs * 16);
    o.ck = take(8 * (n_static + K) * 8);
    o.np = (11 + 3 * K + (W > 0 ? CT_N_JOINTS : 0)) | 1;
    o.pp = (2 * K * split * o.np) | 1;
    o.part = take(mode == MODE_COST ? 0 : P * o.pp * 4);
    o.total = at;
    return o;
}

// Stop-at-first of the fused step: on = leave after the first iteration that
// finds a satisfying particle; with several iterations per launch, the copies
// [D][ld] of the state the launch started from, the iterations each workgroup
// ran (0: it found the solve stopped), and whether this is the second launch
// that brings every tile to the iteration of the stop.  own: that iteration, a
// word which nobody but a launch and its second launch reads or writes
// (STOP_NONE before the launch, which clears own_next for the one after it).
constexpr int32_t STOP_NONE = 0x7FFFFFFF;
struct StopArgs {
    int32_t on, redo;
    float *Xb, *Mb, *Vb;
    int32_t *ran, *own, *own_next;
};

// One skeleton of a batch, as the persistent kernel sees it.
struct BatchSkel {
    const Tables* T;
    float *X, *M, *V, *cost;
    uint8_t* mask;
    int32_t* first_sat;
    const uint8_t* frozen;
    int64_t n, ld;
    float gscale;
    int per;   // particles of a tile
};

}  // namespace ct
