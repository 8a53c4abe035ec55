// Fused particle cost / gradient / mask / Adam kernel for gfx950.
//
// What it computes (per particle x of a K-step pick-place skeleton):
//   the terms J_c of every constraint and soft cost (Sec. IV-A, App. "Cost
//   Weights"), the weighted cost J(x) of Eq. (2), the satisfaction bit of
//   Eq. (3), dJ/dx, and optionally Adam update number t on the batch-mean
//   objective of Eq. (4) (Sec. IV-B).
//
// Work decomposition (one workgroup = 256 lanes = 4 wave64s):
//   * a particle owns 2K "slots", one per robot configuration (q_grasp and
//     q_place of each step); each slot is served by SPLIT adjacent lanes that
//     share its spheres, culling tests and joint sines.  A workgroup's tile has
//     P = 256 / (2K SPLIT) particle columns (a launch may fill fewer of them);
//     lanes are slot-major, so a wave holds the same slot of many particles.
//   * phase 0 stages the particles' columns of the dimension-major X (and the
//     fused step's moments) and the problem's tables in LDS; the fused step
//     then runs every iteration of the launch on them.
//   * phase 1 runs every lane's configuration: forward kinematics link by
//     link, each link's bounding sphere against every box, then the spheres of
//     the configurations that touch something, spread over the wave's lanes;
//     pose / bound terms; gradients leave the lane as world-frame wrenches
//     folded onto the joint axes.
//   * slots of a particle meet in LDS; phase 2 sums each coordinate's partials
//     in a fixed order (bit-reproducible, whatever the tile's filling) and
//     writes G or applies Adam in place.
//
// What bounds it (packing, 8192 particles, K = 4, SPLIT 2; one iteration 55.8
// us with a launch each, 41 now): 50% of the wave time is issue, 44% waits on
// LDS and scalar loads; 230 registers keep two waves per SIMD.  Link tables
// are scalar loads, boxes and spheres LDS reads.
#pragma once

#include "ct_tables.hpp"

namespace ct {


__device__ __forceinline__ float fast_rsq(float x) { return __builtin_amdgcn_rsqf(x); }

// Squared distance from a point to a box, given the point in the box frame
// (p) and the half extents: ||max(|p| - h, 0)||^2, zero inside the box.
__device__ __forceinline__ float box_d2(float px, float py, float pz, float hx, float hy, float hz) {
    const float mx = fmaxf(fabsf(px) - hx, 0.f);
    const float my = fmaxf(fabsf(py) - hy, 0.f);
    const float mz = fmaxf(fabsf(pz) - hz, 0.f);
    return fmaf(mz, mz, fmaf(mx, mx, my * my));
}

// Penetration of a sphere that touches the box (its squared outside distance
// is below r^2), from the centre p in the box frame: pen = r - sdf with
// sdf = ||max(u, 0)|| + min(max_i u_i, 0), u = |p| - h (App. "Collision
// Representation": spheres against oriented boxes), and v = d sdf / d centre
// = -d pen / d centre in world coordinates (box yaw cos c, sin s).
// Tie conventions: sign(0) = +1; among equal interior depths the lowest axis.
__device__ __forceinline__ void pair_hit(float px, float py, float pz, float r, float c, float s, float hx,
                                         float hy, float hz, float& pen, float& vx, float& vy, float& vz) {
    const float ux = fabsf(px) - hx, uy = fabsf(py) - hy, uz = fabsf(pz) - hz;
    const float mx = fmaxf(ux, 0.f), my = fmaxf(uy, 0.f), mz = fmaxf(uz, 0.f);
    const float d2 = fmaf(mz, mz, fmaf(mx, mx, my * my));
    float sdf, ax, ay, az;  // sdf and d sdf / d p
    if (d2 > 0.f) {
        const float inv = fast_rsq(d2);
        sdf = d2 * inv;
        ax = copysignf(mx * inv, px);
        ay = copysignf(my * inv, py);
        az = copysignf(mz * inv, pz);
    } else {
        const float sx = px >= 0.f ? 1.f : -1.f;
        const float sy = py >= 0.f ? 1.f : -1.f;
        const float sz = pz >= 0.f ? 1.f : -1.f;
        if (ux >= uy && ux >= uz) {
            sdf = ux; ax = sx; ay = 0.f; az = 0.f;
        } else if (uy >= uz) {
            sdf = uy; ax = 0.f; ay = sy; az = 0.f;
        } else {
            sdf = uz; ax = 0.f; ay = 0.f; az = sz;
        }
    }
    pen = r - sdf;
    // d pen / d centre = -R d sdf / d p
    vx = fmaf(c, ax, -(s * ay));
    vy = fmaf(c, ay, s * ax);
    vz = az;
}

// The centres of the moved objects as one lane's step k sees them, for the
// culling tests: object j was placed by an earlier step (at P(rho_j), a
// particle variable) or is still at its initial pose.  The SPLIT lanes of a
// slot share the objects out, lane si holds si, si + SPLIT, ... in registers
// (past the last: the last again).
template <int KT, int SPLIT>
struct MoveCtx {
    static constexpr int U = (KT + SPLIT - 1) / SPLIT;
    float x[U], y[U];
    int k, p;   // step, column of the tile
    // nans: a NaN centre counts as touching, so that the penetrations it is in
    // come out non-finite; live: the column has a particle (both compile-time
    // constants in the fused step, see lane_slot)
    bool nans, live;
};

// Bijection from the launch index to a tile index that keeps each XCD's
// workgroups (b = x, x + 8, x + 16, ...) on a contiguous tile range.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t G) {
    constexpr int NX = 8;
    const int64_t x = b % NX, q = G / NX, rem = G % NX;
    return x * q + (x < rem ? x : rem) + b / NX;
}

template <int SPLIT>
__device__ __forceinline__ float split_sum(float v) {
    if (SPLIT >= 2) v += __shfl_xor(v, 1);
    if (SPLIT >= 4) v += __shfl_xor(v, 2);
    return v;
}

// v of the SPLIT lanes of a slot to all of them: out[j0 + u] = v of lane u.
template <int SPLIT>
__device__ __forceinline__ void split_bcast(float v, int j0, float out[CT_N_JOINTS]) {
    const int b = __float_as_int(v);
    if (SPLIT == 1) {
        out[j0] = v;
    } else if (SPLIT == 2) {
        out[j0] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xA0, 0xF, 0xF, true));
        if (j0 + 1 < CT_N_JOINTS) out[j0 + 1] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xF5, 0xF, 0xF, true));
    } else {
        out[j0] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x00, 0xF, 0xF, true));
        if (j0 + 1 < CT_N_JOINTS) out[j0 + 1] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x55, 0xF, 0xF, true));
        if (j0 + 2 < CT_N_JOINTS) out[j0 + 2] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xAA, 0xF, 0xF, true));
        if (j0 + 3 < CT_N_JOINTS) out[j0 + 3] = __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xFF, 0xF, 0xF, true));
    }
}

__device__ __forceinline__ void cross3(const float a[3], const float b[3], float o[3]) {
    o[0] = fmaf(a[1], b[2], -(a[2] * b[1]));
    o[1] = fmaf(a[2], b[0], -(a[0] * b[2]));
    o[2] = fmaf(a[0], b[1], -(a[1] * b[0]));
}

// z . tq + m . f of a joint axis (z, m) and a wrench (force f, moment tq).
__device__ __forceinline__ float axis_wrench(const float z[3], const float m[3], const float f[3], const float tq[3]) {
    return fmaf(m[2], f[2], fmaf(m[1], f[1], fmaf(m[0], f[0], fmaf(z[2], tq[2], fmaf(z[0], tq[0], z[1] * tq[1])))));
}

// One standard-DH joint: (R, t) <- (R, t) Rz(theta_i) Tz(d_i) Tx(a_i) Rx(alpha_i)
// for joint i (0-based) with the sine and cosine of theta_i = q_i + theta0_i.
__device__ __forceinline__ void joint_advance(const Joint& J, float sn, float cs, float R[9], float t[3]) {
    const float ca = J.ca, sa = J.sa, a = J.a, d = J.d;
    const float lx = a * cs, ly = a * sn;
#pragma unroll
    for (int rr = 0; rr < 3; ++rr) {
        const float r0 = R[3 * rr], r1 = R[3 * rr + 1], r2 = R[3 * rr + 2];
        t[rr] += fmaf(r2, d, fmaf(r0, lx, r1 * ly));
        const float w = fmaf(r1, cs, -(r0 * sn));
        R[3 * rr] = fmaf(r0, cs, r1 * sn);
        R[3 * rr + 1] = fmaf(r2, sa, ca * w);
        R[3 * rr + 2] = fmaf(r2, ca, -(sa * w));
    }
}

// ---------------------------------------------------------------------------
// Spheres against boxes.
//
// Of the ~880 sphere-box pairs of a packing configuration 2.6 penetrate, and
// a link's bounding sphere touches 0.2 boxes on average; but over the 32 or 64
// configurations of a wave some lane needs almost every (link, box) pair.  So
// the lanes do not walk their own spheres: per link, the configurations whose
// bounding sphere touches a box ("owners") are compacted, and the whole wave
// tests their spheres, one (owner, sphere) per lane, each lane walking only
// its owner's boxes.  The penetrations found go back through LDS to the
// owner's lanes, which add them in the order in which a lane walking its own
// spheres would: spheres ascending, and within a sphere the static boxes and
// then the moved objects ascending; with SPLIT lanes per configuration lane si
// adds the spheres si, si + SPLIT, ...  Sums are therefore the same whatever
// the mapping of tests to lanes.

// LDS of one workgroup's tile (see tile_layout for the sizes).
struct TileLds {
    float *xs, *ms, *vs;   // staged particles [D][P]; Adam moments (fused step without waypoints)
    float* part;           // gradient partials, np per lane
    float4* plc;           // [K][P] placements (x, y, cos yaw, sin yaw)
    float4* rs;            // robot spheres
    float4* osl;           // [K][CT_MAX_OBJ_SPHERES] object spheres
    SBox* sbx;             // static boxes
    CullBox* cbx;          // culling constants of the static boxes, then of the K moved objects
    float2* ck;            // [8][n_static + K] thresholds (xy^2, z) of link L's bounding sphere
    Box* ob0;              // [K] moved objects at their initial poses
    float *cpart, *tpart;  // [P][2K] slot costs, transition lengths
    int *flg, *hpart;      // [P][2K] slot flags, touching pairs
    int* okp;              // [P] update permission
    uint8_t* frz;          // [D] frozen dimensions
    int* ctl;              // any_sat, halt
    float2* bc;            // [MAX_LAUNCH_ITERS] 1 - beta1^t, 1 - beta2^t of the launch's updates (fused step)
    float4* wave;          // WAVE_F4 per wave: owner records, then test results
    int np, pp, P;   // floats of a lane's, of a particle's partials; columns
};

// Orders a wave's LDS accesses for the compiler: the lanes of a wave run in
// step and its LDS operations complete in order, so no wait is needed.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Per wave: up to OWNERS owner records of 5 float4 (one of padding: the 16
// records of a pass start in different banks), overwritten by the results of
// the wave's 64 tests, 2 float4 each.
constexpr int OWNERS = 16;
constexpr int WAVE_F4 = 128;

// Boxes that a bounding sphere (world centre w, radius rb) may touch: bit b of
// smask for static box b, bit j of omask for moved object j.  A box is tested
// as an upright cylinder (its footprint's circle, its height), 6 vector
// instructions where the exact box distance takes 18 and lets 30% fewer pairs
// through: the circle's squared test |w - c|^2 < (rb + r)^2 is taken as
// |w|^2 - 2 w.c < K with K = (rb + r)^2 - |c|^2 and a margin for its rounding
// from the host.  The bounding sphere holds its set with a margin, so a box
// left out touches no sphere of the set and every sum is unchanged; with
// mc.nans only a centre known to be too far leaves a box out.  The SPLIT
// lanes of a slot hold the same bounding sphere and share the static boxes
// out: lane si tests boxes si, si + SPLIT, ...
template <int SPLIT>
__device__ __forceinline__ uint32_t split_or(uint32_t v) {
    if (SPLIT >= 2) v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);   // lanes ^ 1
    if (SPLIT >= 4) v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // lanes ^ 2
    return v;
}

// L >= 0: robot link L (thresholds from the table); L < 0: an object's sphere
// of radius rb (thresholds formed here).
template <int KT, int SPLIT, bool LINK>
__device__ __forceinline__ void touched_boxes(const TileLds& S, int nsb, int si, const MoveCtx<KT, SPLIT>& mc,
                                              const float2* __restrict__ ck, float wx, float wy, float wz, float rb,
                                              uint32_t& smask, uint32_t& omask) {
    const float q = wx * wx + wy * wy;
    smask = 0u;
    omask = 0u;
    uint32_t bit = 1u << si;
    for (int b0 = 0; b0 < nsb; b0 += SPLIT) {
        const int b = min(b0 + si, nsb - 1);
        const CullBox C = S.cbx[b];
        float2 th;
        if (LINK) {
            th = ck[b];
        } else {
            const float e = rb + C.r;
            th = make_float2(fmaf(e, e, C.kc), rb + C.hz);
        }
        const float t = fmaf(C.m2x, wx, fmaf(C.m2y, wy, q));
        const float z = fabsf(wz - C.z);
        const bool hit = mc.nans ? !(t >= th.x) && !(z >= th.y) : t < th.x && z < th.y;
        smask |= hit ? bit : 0u;
        bit <<= SPLIT;
    }
    // a box past the last one repeats it at a bit of its own
    smask = split_or<SPLIT>(smask) & (nsb < 32 ? (1u << nsb) - 1u : ~0u);
    if (KT == 1) return;   // the only moved object is the one in the hand
#pragma unroll
    for (int u = 0; u < MoveCtx<KT, SPLIT>::U; ++u) {
        const int j = min(u * SPLIT + si, KT - 1);
        const CullBox C = S.cbx[nsb + j];
        float2 th;
        if (LINK) {
            th = ck[nsb + j];
        } else {
            const float e = rb + C.r;
            th = make_float2(e * e * 1.000001f, rb + C.hz);
        }
        const float dx = wx - mc.x[u], dy = wy - mc.y[u], t = dx * dx + dy * dy, z = fabsf(wz - C.z);
        const bool hit = mc.nans ? !(t >= th.x) && !(z >= th.y) : t < th.x && z < th.y;
        omask |= hit ? 1u << j : 0u;
    }
    omask = split_or<SPLIT>(omask);
    omask &= ~(1u << mc.k);   // the step's own object is held, not an obstacle
}

// One set of ns spheres per configuration (a link's, an object's) in the frame
// (R, t) against the boxes of smask and omask.  tab: the set's sphere table
// in LDS, or (OBJ) the table of step 0 (an owner's step selects its own).
// Adds the penetrations of this lane's spheres to coll, their weighted
// gradients to the wrench (f, tq about the world origin) and to the placement
// partials gr.  The active lanes of the wave are its first lanes (at least
// 48: tiles leave at most the tail of the last wave idle).
template <int KT, int SPLIT, bool GRAD, bool OBJ>
__device__ __forceinline__ void sphere_set(const TileLds& S, const float4* __restrict__ tab, int ns, int si,
                                           const float R[9], const float t[3], const MoveCtx<KT, SPLIT>& mc, uint32_t smask,
                                           uint32_t omask, float lam, float& coll, float f[3], float tq[3],
                                           float* __restrict__ gr, int& nhit) {
    const bool mine = (smask | omask) != 0u && mc.live;
    const uint64_t owners = __ballot(mine);
    if (!owners) return;   // wave-uniform: no configuration of the wave touches a box
    const int lane = threadIdx.x & 63;
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(owners >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)owners, 0u)) / SPLIT;
    const int na = __popcll(owners) / SPLIT, nact = __popcll(__ballot(true));
    float4* rec = S.wave + (threadIdx.x >> 6) * WAVE_F4;
    constexpr uint32_t CLASS = SPLIT == 1 ? ~0u : SPLIT == 2 ? 0x55555555u : 0x11111111u;
    for (int c0 = 0; c0 < ns; c0 += 32) {
        const int nc = min(ns - c0, 32);
        const float inv = __builtin_amdgcn_rcpf((float)nc);
        const int per = __builtin_amdgcn_readfirstlane(min((int)(((float)nact + 0.5f) * inv), OWNERS));
        const int g = (int)(((float)lane + 0.5f) * inv), e = lane - g * nc;   // owner of the pass, sphere
        for (int a0 = 0; a0 < na; a0 += per) {
            const bool here = mine && (uint32_t)(rank - a0) < (uint32_t)per;
            const int rel = rank - a0;
            if (here && si == 0) {
                float4* w = rec + rel * 5;
                w[0] = make_float4(R[0], R[1], R[2], R[3]);
                w[1] = make_float4(R[4], R[5], R[6], R[7]);
                w[2] = make_float4(R[8], t[0], t[1], t[2]);
                w[3] = make_float4(__uint_as_float(smask), __uint_as_float(omask | (uint32_t)mc.k << 8 | (uint32_t)mc.p << 16),
                                   lam, 0.f);
            }
            wave_sync();
            const bool on = g < per && a0 + g < na;
            const float4* w = rec + (on ? g : 0) * 5;
            const float4 w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
            uint32_t sm = on ? __float_as_uint(w3.x) : 0u;
            const uint32_t ow = __float_as_uint(w3.y);
            uint32_t om = on ? ow & 0xFFu : 0u;
            const int kk = (int)(ow >> 8 & 0xFFu), pp = (int)(ow >> 16);
            const float wl = w3.z;
            const float4 sp = tab[(OBJ ? kk * CT_MAX_OBJ_SPHERES : 0) + c0 + e];
            const float cx = fmaf(w0.z, sp.z, fmaf(w0.x, sp.x, w0.y * sp.y)) + w2.y;
            const float cy = fmaf(w1.y, sp.z, fmaf(w0.w, sp.x, w1.x * sp.y)) + w2.z;
            const float cz = fmaf(w2.x, sp.z, fmaf(w1.z, sp.x, w1.w * sp.y)) + w2.w;
            const float r = sp.w, r2 = r * r;
            float pen = 0.f, gx = 0.f, gy = 0.f, gz = 0.f;
            int hits = 0;
            while (sm) {   // this lane's owner's static boxes
                const int b = __builtin_ctz(sm);
                sm &= sm - 1u;
                const SBox B = S.sbx[b];
                const float px = fmaf(B.c, cx, fmaf(B.s, cy, B.u0));
                const float py = fmaf(B.c, cy, fmaf(-B.s, cx, B.u1));
                const float pz = cz - B.tz;
                if (box_d2(px, py, pz, B.hx, B.hy, B.hz) < r2) {
                    float pn, vx, vy, vz;
                    pair_hit(px, py, pz, r, B.c, B.s, B.hx, B.hy, B.hz, pn, vx, vy, vz);
                    pen += pn;
                    ++hits;
                    if (GRAD) { gx = fmaf(-wl, vx, gx); gy = fmaf(-wl, vy, gy); gz = fmaf(-wl, vz, gz); }
                }
            }
            if (KT != 1) {
                // the objects of the lane's owner, lowest first: the lanes of one
                // owner take the same object, others another; `own` follows in
                // the owner's own lanes
                uint32_t own = omask;
                while (__ballot(om != 0u)) {
                    const bool cand = om != 0u;
                    const int j = cand ? __builtin_ctz(om) : 0;
                    om &= om - 1u;
                    const int jo = own ? __builtin_ctz(own) : 0;
                    own &= own - 1u;
                    const Box O = S.ob0[j];
                    const float4 pl = S.plc[j * S.P + pp];
                    const bool placed = j < kk;
                    const float bx = placed ? pl.x : O.cx, by = placed ? pl.y : O.cy;
                    const float bc = placed ? pl.z : O.c, bs = placed ? pl.w : O.s;
                    const float dx = cx - bx, dy = cy - by;
                    const float px = fmaf(bc, dx, bs * dy), py = fmaf(bc, dy, -(bs * dx)), pz = cz - O.cz;
                    const bool act = cand && box_d2(px, py, pz, O.hx, O.hy, O.hz) < r2;
                    float vx = 0.f, vy = 0.f, vz;
                    if (act) {
                        float pn;
                        pair_hit(px, py, pz, r, bc, bs, O.hx, O.hy, O.hz, pn, vx, vy, vz);
                        pen += pn;
                        ++hits;
                        if (GRAD) { gx = fmaf(-wl, vx, gx); gy = fmaf(-wl, vy, gy); gz = fmaf(-wl, vz, gz); }
                    }
                    if (GRAD) {
                        // moving the box by d equals moving the sphere by -d; turning it
                        // about its own vertical axis equals turning the sphere back
                        const uint64_t moved = __ballot(act && placed);
                        if (moved) {
                            if (act && placed) {
                                const float ax = -wl * vx, ay = -wl * vy;
                                rec[lane] = make_float4(ax, ay, fmaf(dx, ay, -(dy * ax)), 0.f);
                            }
                            wave_sync();
                            if (here) {
                                uint32_t bits = (uint32_t)(moved >> (rel * nc)) & (CLASS << si);
                                if (nc < 32) bits &= (1u << nc) - 1u;
                                while (bits) {
                                    const float4 v = rec[rel * nc + __builtin_ctz(bits)];
                                    bits &= bits - 1u;
                                    gr[3 * jo] -= v.x;
                                    gr[3 * jo + 1] -= v.y;
                                    gr[3 * jo + 2] -= v.z;
                                }
                            }
                            wave_sync();
                        }
                    }
                }
            }
            const uint64_t any = __ballot(hits != 0);
            if (any) {
                if (hits != 0) {
                    rec[lane] = make_float4(pen, gx, gy, gz);
                    rec[64 + lane] = make_float4(fmaf(cy, gz, -(cz * gy)), fmaf(cz, gx, -(cx * gz)), fmaf(cx, gy, -(cy * gx)),
                                                    __int_as_float(hits));
                }
                wave_sync();
                if (here) {
                    uint32_t bits = (uint32_t)(any >> (rel * nc)) & (CLASS << si);
                    if (nc < 32) bits &= (1u << nc) - 1u;
                    while (bits) {
                        const float4* v = rec + (rel * nc + __builtin_ctz(bits));
                        bits &= bits - 1u;
                        const float4 u = v[0], m = v[64];
                        coll += u.x;
                        if (GRAD) {
                            f[0] += u.y; f[1] += u.z; f[2] += u.w;
                            tq[0] += m.x; tq[1] += m.y; tq[2] += m.z;
                        } else {
                            nhit += __float_as_int(m.w);
                        }
                    }
                }
                wave_sync();
            }
        }
    }
}

// All robot spheres of link L (frame (R, t)).
template <int KT, int SPLIT, bool GRAD>
__device__ __forceinline__ void link_spheres(const Tables* __restrict__ T, const Joint& J, const TileLds& S, int L, int si,
                                             const float R[9], const float t[3], const MoveCtx<KT, SPLIT>& mc, float lam,
                                             float& coll, float f[3], float tq[3], float* __restrict__ gr, int& nhit) {
    const int s0 = J.s0, ns = J.ns;
    if (ns == 0) return;
    const float4 lb = J.lb;
    uint32_t smask, omask;
    touched_boxes<KT, SPLIT, true>(S, T->n_static, si, mc, S.ck + (L - 1) * (T->n_static + KT),
                                   R[0] * lb.x + R[1] * lb.y + R[2] * lb.z + t[0],
                                   R[3] * lb.x + R[4] * lb.y + R[5] * lb.z + t[1],
                                   R[6] * lb.x + R[7] * lb.y + R[8] * lb.z + t[2], lb.w, smask, omask);
    sphere_set<KT, SPLIT, GRAD, false>(S, S.rs + s0, ns, si, R, t, mc, smask, omask, lam, coll, f, tq, gr,
                                       nhit);
}

// The object spheres of this lane's step (frame (R, t)); use = false: this
// lane has none here (every lane of the wave calls, so that all of them can
// take tests).
template <int KT, int SPLIT, bool GRAD>
__device__ __forceinline__ void object_spheres(const Tables* __restrict__ T, const TileLds& S, bool use,
                                               float4 ob, int si, const float R[9], const float t[3],
                                               const MoveCtx<KT, SPLIT>& mc, float lam, float& coll, float f[3], float tq[3],
                                               float* __restrict__ gr, int& nhit) {
    if (T->n_os <= 0) return;
    uint32_t smask, omask;
    touched_boxes<KT, SPLIT, false>(S, T->n_static, si, mc, nullptr,
                                    R[0] * ob.x + R[1] * ob.y + R[2] * ob.z + t[0],
                                    R[3] * ob.x + R[4] * ob.y + R[5] * ob.z + t[1],
                                    R[6] * ob.x + R[7] * ob.y + R[8] * ob.z + t[2], ob.w, smask, omask);
    if (!use) smask = omask = 0u;
    sphere_set<KT, SPLIT, GRAD, true>(S, S.osl, T->n_os, si, R, t, mc, smask, omask, lam, coll, f, tq, gr, nhit);
}

// dist_from_bounds of v against [lo, hi] and its gradient (scaled by lam).
template <int N>
__device__ __forceinline__ float bounds_dist(const float v[N], const float* lo, const float* hi, float lam,
                                             float g[N]) {
    float m[N], ss = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const float below = lo[j] - v[j], above = v[j] - hi[j];
        const float e = fmaxf(fmaxf(below, above), 0.f);
        m[j] = below > above ? -e : e;   // signed: d e / d v = -1 below, +1 above
        ss += e * e;
    }
    const float dist = sqrtf(ss);
    const float inv = dist > 0.f ? lam / dist : 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) g[j] = m[j] * inv;
    return dist;
}

// Robot self-collision of one configuration: pairs of robot spheres on links
// La < Lb with Lb >= La + 2, penalty max(0, r_a + r_b - |c_a - c_b|).  The
// work is done in the frame of La: the frame of every later link relative to
// it is a product of joint transforms (the stored joint sines and cosines),
// so no world frame is formed and nothing is staged.
//
// Gradient: a pair pushes its b sphere with g_b = lam (c_a - c_b) / |c_a - c_b|
// and its a sphere with -g_b along the same line, so a joint that moves both
// spheres (joints up to La) feels nothing; joint j in La+1 .. Lb (0-based
// index La .. Lb-1) feels the wrench (g_b, c_b x g_b) through its axis S_j.
// Per La, the b-side wrenches are summed by link and folded onto the axes as
// in the world pass: dJ/dq_j = <S_j, W_total> - <S_j, W of links <= j>.

// The joint of joint_advance, its products left to the compiler to fuse.
__device__ __forceinline__ void self_advance(const Joint& J, float sn, float cs, float R[9], float t[3]) {
    const float ca = J.ca, sa = J.sa, a = J.a, d = J.d;
    const float lx = a * cs, ly = a * sn;
#pragma unroll
    for (int rr = 0; rr < 3; ++rr) {
        const float r0 = R[3 * rr], r1 = R[3 * rr + 1], r2 = R[3 * rr + 2];
        t[rr] += r0 * lx + r1 * ly + r2 * d;
        const float w = r1 * cs - r0 * sn;
        R[3 * rr] = r0 * cs + r1 * sn;
        R[3 * rr + 1] = ca * w + r2 * sa;
        R[3 * rr + 2] = r2 * ca - sa * w;
    }
}

// NB consecutive spheres of link Lb of one lane (entries b0 + si + SPLIT j,
// j = j0 .. j0+NB-1, in a frame (Q, o) relative to link La's frame) against
// every sphere of La (in La's own frame; uniform loads, one per NB pairs).
// Skipped when no lane's run meets La's bounding sphere (it would add zeros).
template <int SPLIT, int NB, bool GRAD>
__device__ __forceinline__ void self_run(const Tables* __restrict__ T, int a0, int a1, float4 ba, int b0, int b1,
                                         int j0, int si, const float Q[9], const float o[3], float lam, float& pen,
                                         float F[3], float Mo[3]) {
    float cx[NB], cy[NB], cz[NB], rb[NB];
    bool valid[NB];
    bool near = false;
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        const int base = b0 + SPLIT * (j0 + m);   // uniform
        float4 sb = T->rs[min(base, b1 - 1)];
        if (SPLIT > 1) {
#pragma unroll
            for (int u = 1; u < SPLIT; ++u) {
                const float4 alt = T->rs[min(base + u, b1 - 1)];
                if (si == u) sb = alt;
            }
        }
        valid[m] = base + si < b1;
        rb[m] = sb.w;
        cx[m] = Q[0] * sb.x + Q[1] * sb.y + Q[2] * sb.z + o[0];
        cy[m] = Q[3] * sb.x + Q[4] * sb.y + Q[5] * sb.z + o[1];
        cz[m] = Q[6] * sb.x + Q[7] * sb.y + Q[8] * sb.z + o[2];
        const float ux = cx[m] - ba.x, uy = cy[m] - ba.y, uz = cz[m] - ba.z, ur = ba.w + sb.w;
        near |= valid[m] && ux * ux + uy * uy + uz * uz < ur * ur;
    }
    if (!__ballot(near)) return;   // wave-uniform
    float p[NB], gx[NB], gy[NB], gz[NB];
#pragma unroll
    for (int m = 0; m < NB; ++m) p[m] = gx[m] = gy[m] = gz[m] = 0.f;
    for (int a = a0; a < a1; ++a) {
        const float4 sa = T->rs[a];
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            const float dx = sa.x - cx[m], dy = sa.y - cy[m], dz = sa.z - cz[m];
            const float d2 = dx * dx + dy * dy + dz * dz;
            const float rsum = sa.w + rb[m];
            if (valid[m] && d2 < rsum * rsum) {
                const float dist = sqrtf(d2);
                p[m] += rsum - dist;
                if (GRAD && dist > 0.f) {
                    const float sc = lam / dist;
                    gx[m] += dx * sc; gy[m] += dy * sc; gz[m] += dz * sc;
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < NB; ++m) {
        pen += p[m];
        if (GRAD) {
            F[0] += gx[m]; F[1] += gy[m]; F[2] += gz[m];
            Mo[0] += cy[m] * gz[m] - cz[m] * gy[m];
            Mo[1] += cz[m] * gx[m] - cx[m] * gz[m];
            Mo[2] += cx[m] * gy[m] - cy[m] * gx[m];
        }
    }
}

// All sphere pairs of links La and Lb (frame (Q, o) of Lb relative to La):
// runs of 2, then 1 over the entries each lane of the slot takes;
// skipped as a whole when no lane's bounding spheres of the two links meet.
template <int SPLIT, bool GRAD>
__device__ __forceinline__ void self_block(const Tables* __restrict__ T, int La, int Lb, int si, const float Q[9],
                                           const float o[3], float lam, float& pen, float F[3], float Mo[3]) {
    const int a0 = T->link_start[La], a1 = T->link_start[La + 1];
    const int b0 = T->link_start[Lb], b1 = T->link_start[Lb + 1];
    if (b0 == b1) return;
    const float4 ba = T->lbs[La], bb = T->lbs[Lb];
    const float ex = Q[0] * bb.x + Q[1] * bb.y + Q[2] * bb.z + o[0] - ba.x;
    const float ey = Q[3] * bb.x + Q[4] * bb.y + Q[5] * bb.z + o[1] - ba.y;
    const float ez = Q[6] * bb.x + Q[7] * bb.y + Q[8] * bb.z + o[2] - ba.z;
    const float rs = ba.w + bb.w;
    if (!__ballot(ex * ex + ey * ey + ez * ez < rs * rs)) return;   // wave-uniform
    const int per_lane = (b1 - b0 + SPLIT - 1) / SPLIT;
    int j = 0;
    for (; j + 2 <= per_lane; j += 2)
        self_run<SPLIT, 2, GRAD>(T, a0, a1, ba, b0, b1, j, si, Q, o, lam, pen, F, Mo);
    if (j < per_lane) self_run<SPLIT, 1, GRAD>(T, a0, a1, ba, b0, b1, j, si, Q, o, lam, pen, F, Mo);
}

// <S_j, (F, Mo)> for the axis of a frame (R, t): z . Mo + (t x z) . F
__device__ __forceinline__ float axis_dot(const float R[9], const float t[3], const float F[3], const float Mo[3]) {
    const float z[3] = {R[2], R[5], R[8]};
    float mz[3];
    cross3(t, z, mz);
    return z[0] * Mo[0] + z[1] * Mo[1] + z[2] * Mo[2] + mz[0] * F[0] + mz[1] * F[1] + mz[2] * F[2];
}

template <int SPLIT, bool GRAD>
__device__ __forceinline__ void self_pass(const Tables* __restrict__ T, int si, const float jsn[CT_N_JOINTS],
                                          const float jcs[CT_N_JOINTS], float lam, float& pen,
                                          float gq[CT_N_JOINTS]) {
#pragma unroll 1
    for (int La = 1; La <= 6; ++La) {   // wave-uniform
        if (T->link_start[La] == T->link_start[La + 1]) continue;
        float Q[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
        float o[3] = {0.f, 0.f, 0.f};
        float F[3] = {0.f, 0.f, 0.f}, Mo[3] = {0.f, 0.f, 0.f};   // b-side wrench, La's frame and origin
#pragma unroll
        for (int j = 1; j < CT_N_JOINTS; ++j) {   // (Q, o) is frame j: joint j's axis (0-based)
            if (j < La) continue;                  // wave-uniform
            if (GRAD && j > La) gq[j] -= axis_dot(Q, o, F, Mo);
            self_advance(T->jk[j], jsn[j], jcs[j], Q, o);
            if (j + 1 >= La + 2) self_block<SPLIT, GRAD>(T, La, j + 1, si, Q, o, lam, pen, F, Mo);
        }
        // the tool: frame 7 moved along its z-axis
        const float ot[3] = {o[0] + Q[2] * T->tool_d, o[1] + Q[5] * T->tool_d, o[2] + Q[8] * T->tool_d};
        self_block<SPLIT, GRAD>(T, La, 8, si, Q, ot, lam, pen, F, Mo);
        if (GRAD) {
            float R[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
            float t[3] = {0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 1; j < CT_N_JOINTS; ++j) {
                if (j < La) continue;
                gq[j] += axis_dot(R, t, F, Mo);
                if (j + 1 < CT_N_JOINTS) self_advance(T->jk[j], jsn[j], jcs[j], R, t);
            }
        }
    }
}

// Weights of the terms one slot evaluates: the problem's lambda of Eq. (2)
// (uniform), or the particle's own row of a per-particle weight table
// [n_terms][ld] (the multiplier-adjusted weights of the augmented-Lagrangian
// mode; extended kernels only).  Fields a slot kind does not own stay unused.
struct SlotW {
    float kpos, krot, jlim, coll, mcoll, self, grasp, cobj, place, goal, traj;
};

__device__ __forceinline__ SlotW slot_weights(const Tables* __restrict__ T, const float* __restrict__ wts,
                                              int64_t ld, int64_t i, int K, int slot, bool self_on) {
    const float* w = T->w;
    SlotW sw{w[W_KPOS], w[W_KROT], w[W_JLIM], w[W_COLL], w[W_MCOLL], w[W_SELF],
             w[W_GRASP], w[W_COLL], w[W_PLACE], w[W_GOAL], w[W_TRAJ]};
    if (wts) {
        const int tb = CT_TERMS_PER_STEP * (slot >> 1);
        const bool placing = slot & 1;
        auto at = [&](int c) { return wts[(int64_t)c * ld + i]; };
        sw.kpos = at(tb + (placing ? T_PLACE_POS : T_PICK_POS));
        sw.krot = at(tb + (placing ? T_PLACE_ROT : T_PICK_ROT));
        sw.jlim = at(tb + (placing ? T_JLIM_P : T_JLIM_G));
        sw.coll = at(tb + (placing ? T_COLL_P : T_COLL_G));
        if (!placing) {
            sw.grasp = at(tb + T_GRASP);
            sw.cobj = at(tb + T_COLL_OBJ);
        } else {
            sw.place = at(tb + T_PLACE);
        }
        if (T->W > 0) {
            sw.mcoll = at(CT_TERMS_PER_STEP * K + slot);
            sw.traj = at(T->traj_term);
        }
        if (self_on) sw.self = at(T->self_term + slot);
        if (T->goal) sw.goal = at(T->goal_term);
    }
    return sw;
}

struct LaneOut {
    float cost;   // weighted sum of this slot's terms
    float traj;   // this slot's transition length (TrajLength share), 0 without motion
    int flags;    // bit 0: all of the slot's constraints hold; bit 1: finite
    int hits;     // touching sphere-box pairs of the slot (cost mode), summed over its lanes
};

// The per-configuration part of a slot's work: forward kinematics link by
// link with each link's robot spheres, the held object (optional) and the
// kinematic constraint (optional).  Accumulates the penetration sum `coll`,
// dJ/dq of this configuration into gq (folded onto the joint axes from
// world-frame wrenches: dJ/dq_j = z_j . tau + (o_j x z_j) . f for the wrench
// of everything beyond joint j), and the grasp / placement partials gg, gr.
template <int KT, int SPLIT, bool GRAD, int JU>
__device__ __forceinline__ void config_pass(const Tables* __restrict__ T, const TileLds& S, int si,
                                            const float jsn[CT_N_JOINTS], const float jcs[CT_N_JOINTS], bool held,
                                            bool kin, bool placing,
                                            float lam, const MoveCtx<KT, SPLIT>& mc, float gx, float gy, float gz,
                                            float g_c, float g_s, float rho_x, float rho_y, float rho_c,
                                            float rho_s, float& coll, float gq[CT_N_JOINTS], float gg[4],
                                            float* __restrict__ gr, float& kin_pos, float& kin_rot,
                                            const SlotW* slw, bool self, float& self_pen, int& nhit) {
    const int k = mc.k;
    // Joint axis S_j = (z_j, o_j x z_j) of joint j+1 (z of frame j through its
    // origin).  dJ/dq_j = <S_j, wrench of links j+1..8>
    //                   = <S_j, total wrench> - <S_j, wrench of links 1..j>;
    // the second product (c_j) is taken on the way out, when S_j is formed
    // and links 1..j are done; the first after the tip, by a second sweep
    // over the chain that re-forms the axes from the stored joint sines and
    // cosines.  (Cancellation is bounded: an element that matters is >= 1%
    // of the largest, and the subtracted products are of that size.)
    float R[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
    float t[3] = {0.f, 0.f, 0.f};
    float cj[CT_N_JOINTS];
    float f[3] = {0.f, 0.f, 0.f}, tq[3] = {0.f, 0.f, 0.f};   // wrench of the links done so far
    // links 1..7, then the tool (spheres of the tool frame, t = its origin)
#pragma unroll JU
    for (int i = 0; i <= CT_N_JOINTS; ++i) {
        const Joint J = T->jk[i];
        if (i < CT_N_JOINTS) {
            if (GRAD) {
                const float z[3] = {R[2], R[5], R[8]};
                float m[3];
                cross3(t, z, m);
                cj[i] = axis_wrench(z, m, f, tq);
            }
            joint_advance(J, jsn[i], jcs[i], R, t);
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j) t[j] = fmaf(R[3 * j + 2], T->tool_d, t[j]);
        }
        link_spheres<KT, SPLIT, GRAD>(T, J, S, i + 1, si, R, t, mc, lam, coll, f, tq, gr, nhit);
    }
    const float* te = t;

    if (__ballot(held)) {
        // held object frame O = F_ee G^-1, G = Trans(g) Rz(gyaw) Rx(pi); the
        // rotation H = Rz(gyaw) Rx(pi) is symmetric and its own inverse
        const float H[9] = {g_c, g_s, 0.f, g_s, -g_c, 0.f, 0.f, 0.f, -1.f};
        float RO[9];
#pragma unroll
        for (int rr = 0; rr < 3; ++rr)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                RO[3 * rr + cc] = R[3 * rr] * H[cc] + R[3 * rr + 1] * H[3 + cc] + R[3 * rr + 2] * H[6 + cc];
        const float tO[3] = {te[0] - (RO[0] * gx + RO[1] * gy + RO[2] * gz),
                             te[1] - (RO[3] * gx + RO[4] * gy + RO[5] * gz),
                             te[2] - (RO[6] * gx + RO[7] * gy + RO[8] * gz)};
        float fo[3] = {0.f, 0.f, 0.f}, to[3] = {0.f, 0.f, 0.f};
        object_spheres<KT, SPLIT, GRAD>(T, S, held, T->obs[k], si, RO, tO, mc, lam, coll, fo, to, gr, nhit);
        if (GRAD && held) {
            // d/dg: every held point moves by -R_O dg;  d/dgyaw: the held
            // object turns about the tool z-axis through the tool origin
            gg[0] -= RO[0] * fo[0] + RO[3] * fo[1] + RO[6] * fo[2];
            gg[1] -= RO[1] * fo[0] + RO[4] * fo[1] + RO[7] * fo[2];
            gg[2] -= RO[2] * fo[0] + RO[5] * fo[1] + RO[8] * fo[2];
            float txf[3];
            cross3(te, fo, txf);
            gg[3] += R[2] * (to[0] - txf[0]) + R[5] * (to[1] - txf[1]) + R[8] * (to[2] - txf[2]);
#pragma unroll
            for (int j = 0; j < 3; ++j) { f[j] += fo[j]; tq[j] += to[j]; }
        }
    }

    // kinematic constraint FK(q) = P G at the pick (P = initial pose) or the
    // place (P = P(rho_k)): position and rotation error
    if (kin && si == 0) {
        float Px, Py, Pz, Pc, Ps;
        if (placing) {
            Px = rho_x; Py = rho_y; Pz = T->place_z[k]; Pc = rho_c; Ps = rho_s;
        } else {
            Px = T->obj0[k].cx; Py = T->obj0[k].cy; Pz = T->obj0[k].cz; Pc = T->obj0[k].c; Ps = T->obj0[k].s;
        }
        const float Rgx = Pc * gx - Ps * gy, Rgy = Ps * gx + Pc * gy;
        const float ex = te[0] - (Px + Rgx), ey = te[1] - (Py + Rgy), ez = te[2] - (Pz + gz);
        kin_pos = sqrtf(ex * ex + ey * ey + ez * ez);
        const float cphi = Pc * g_c - Ps * g_s, sphi = Ps * g_c + Pc * g_s;
        // R_err = R_ee^T R_t with R_t columns (cphi, sphi, 0), (sphi, -cphi, 0), (0, 0, -1)
        const float E00 = R[0] * cphi + R[3] * sphi, E01 = R[0] * sphi - R[3] * cphi, E02 = -R[6];
        const float E10 = R[1] * cphi + R[4] * sphi, E11 = R[1] * sphi - R[4] * cphi, E12 = -R[7];
        const float E20 = R[2] * cphi + R[5] * sphi, E21 = R[2] * sphi - R[5] * cphi, E22 = -R[8];
        const float w0 = 0.5f * (E21 - E12), w1 = 0.5f * (E02 - E20), w2 = 0.5f * (E10 - E01);
        const float sw = sqrtf(w0 * w0 + w1 * w1 + w2 * w2);
        kin_rot = atan2f(sw, 0.5f * (E00 + E11 + E22 - 1.f));
        if (GRAD) {
            const float lp = slw ? slw->kpos : T->w[W_KPOS], lr = slw ? slw->krot : T->w[W_KROT];
            if (kin_pos > 0.f) {
                const float sc = lp / kin_pos;
                const float nx = ex * sc, ny = ey * sc, nz = ez * sc;
                f[0] += nx; f[1] += ny; f[2] += nz;
                tq[0] += te[1] * nz - te[2] * ny;
                tq[1] += te[2] * nx - te[0] * nz;
                tq[2] += te[0] * ny - te[1] * nx;
                // the target moves with the grasp offset (and the placement)
                gg[0] -= Pc * nx + Ps * ny;
                gg[1] -= -Ps * nx + Pc * ny;
                gg[2] -= nz;
                if (placing) {
                    gr[3 * k] -= nx;
                    gr[3 * k + 1] -= ny;
                    gr[3 * k + 2] -= -Rgy * nx + Rgx * ny;
                }
            }
            if (sw > 0.f) {
                const float inv = 1.f / sw;
                const float u0 = w0 * inv, u1 = w1 * inv, u2 = w2 * inv;
                const float uw0 = R[0] * u0 + R[1] * u1 + R[2] * u2;
                const float uw1 = R[3] * u0 + R[4] * u1 + R[5] * u2;
                const float uw2 = R[6] * u0 + R[7] * u1 + R[8] * u2;
                // turning the tool by w lowers the angle by u_w . w; turning the
                // target about world z raises it by u_w . z
                tq[0] -= lr * uw0; tq[1] -= lr * uw1; tq[2] -= lr * uw2;
                gg[3] += lr * uw2;
                if (placing) gr[3 * k + 2] += lr * uw2;
            }
        }
    }
    if (GRAD) {
        // second sweep: re-form each axis and take it against the total wrench
        float Q[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
        float o[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < CT_N_JOINTS; ++i) {
            const float z[3] = {Q[2], Q[5], Q[8]};
            float m[3];
            cross3(o, z, m);
            gq[i] += fmaf(m[2], f[2], fmaf(m[1], f[1], fmaf(m[0], f[0], fmaf(z[2], tq[2], fmaf(z[1], tq[1], z[0] * tq[0]))))) -
                     cj[i];
            if (i + 1 < CT_N_JOINTS) joint_advance(T->jk[i], jsn[i], jcs[i], Q, o);
        }
    }
    if (self) self_pass<SPLIT, GRAD>(T, si, jsn, jcs, slw ? slw->self : T->w[W_SELF], self_pen, gq);
}

// ---------------------------------------------------------------------------
// One slot of one particle.  Slot 2k owns q_grasp of step k and the free
// transition into it (from q_place of step k-1, or q0); slot 2k+1 owns
// q_place of step k and the holding transition q_grasp -> q_place.  Terms:
//   grasp slot: Kin at the pick, Grasp, joint limits of q_grasp, CFreeHold at
//               q_grasp, CFreePlace of the object at its placement
//   place slot: Kin at the place, StablePlace containment, joint limits of
//               q_place, CFreeHold at q_place, the goal cost (slot 1 only)
//   with waypoints: the transition's collision term over its interior
//               waypoints a + s (b - a), s = w / (W + 1), and its length.
// A waypoint's gradient goes to the transition's end (share s, this slot's
// own configuration) and start (share 1 - s, the previous slot's
// configuration, returned as the "foreign" partial).
// Every lane writes its own gradient partials (no cross-lane reduction) to
// part[0 .. 18+3K): [0,7) own q, [7,11) grasp, [11, 11+3K) placements
// (accumulated in place), [11+3K, 18+3K) foreign q.
template <int KT, int SPLIT, int MODE, bool EXT>
__device__ __forceinline__ LaneOut lane_slot(const Tables* __restrict__ T, const TileLds& S, int p,
                                             int slot, int si, float* __restrict__ part, float* __restrict__ terms,
                                             int64_t term_ld, int64_t i_glob, bool write_terms,
                                             const float* __restrict__ wts, bool live) {
    constexpr bool GRAD = MODE != MODE_COST;
    constexpr int K = KT;
    // how far config_pass unrolls its loop over the 8 links: fully where that is
    // faster, as a link's tables are loaded while the one before is tested
    // (16384 waypoint gradients 1.21 -> 1.14 ms, 100 steps of 256 one-step
    // particles 1.39 -> 1.31), though some of these spill (gradients 12 to 52
    // bytes a lane at split 1 from 3 steps on and at split 2 with 3, 5 and 6;
    // the one-step fused step 80 and 88 at splits 2 and 4); the longer fused
    // steps and the extended kernels would spill more (64 skeletons 37.1 -> 39.3
    // ms, an augmented-Lagrangian round 2.16 -> 2.32) and take pairs (36.7,
    // 2.13), as do the cost kernels past 4 steps, which would pass the 168
    // registers of three waves (65536 x 6 steps 243 -> 326 us)
    constexpr int JU = !EXT && (MODE == MODE_GRAD || (MODE == MODE_COST && KT <= 4) || KT == 1) ? 8 : 2;
    const bool self_on = EXT && T->self_on;   // wave-uniform; compiled out without EXT
    // per-particle weights only in extended kernels; plain kernels read lambda
    // from the tables where each term needs it
    SlotW swv;
    if (EXT) swv = slot_weights(T, wts, term_ld, i_glob, K, slot, self_on);
    const SlotW* sw = EXT ? &swv : nullptr;
    // When a step's slots fill whole waves (the tile layout at K = 1, 2, 4)
    // the step, and at K = 1, 2 also the slot kind, is the same for every
    // lane of a wave: say so, so that step-indexed tables are scalar loads
    // and the kind's branches are uniform.
    constexpr int LANES_PER_SLOT = tile_particles(KT, SPLIT) * SPLIT;
    constexpr bool STEP_UNIFORM = (2 * LANES_PER_SLOT) % 64 == 0;
    constexpr bool KIND_UNIFORM = LANES_PER_SLOT % 64 == 0;
    const int k = STEP_UNIFORM ? __builtin_amdgcn_readfirstlane(slot >> 1) : slot >> 1;
    const bool placing = KIND_UNIFORM ? (__builtin_amdgcn_readfirstlane(slot) & 1) : (slot & 1);
    const int xs_stride = S.P;
    const float* xs = S.xs + p;
    const float4* plc = S.plc + p;
    auto X = [&](int d) { return xs[d * xs_stride]; };
    const int b0 = CT_STEP_DIM * k;
    float* gr = part + 11;   // placement partials, this lane's own

    const float gx = X(b0 + 14), gy = X(b0 + 15), gz = X(b0 + 16), gyaw = X(b0 + 17);
    float g_s, g_c;
    sincosf(gyaw, &g_s, &g_c);
    const float4 own = plc[k * xs_stride];
    // a column without a particle is evaluated at NaN sines and placement: its
    // centres are NaN and join no test
    const float none = __builtin_nanf("");
    const float rho_x = live ? own.x : none, rho_y = own.y, rho_c = own.z, rho_s = own.w;
    MoveCtx<KT, SPLIT> mc;
    // cost and gradient kernels let a NaN coordinate reach every penetration it
    // enters (a term of 0 would count as satisfied); in the fused step the pose
    // errors alone make its particle's cost non-finite and its mask 0, and the
    // tests of NaN would cost it up to 3% (1501 x 6 steps 580 us without, 601
    // with; 64 skeletons 32.7 and 33.2 ms)
    mc.nans = MODE != MODE_STEP;
    mc.live = !mc.nans || live;
#pragma unroll
    for (int u = 0; u < MoveCtx<KT, SPLIT>::U; ++u) {
        const int j = min(u * SPLIT + si, KT - 1);
        const float4 pl = plc[j * xs_stride];
        const Box& O = S.ob0[j];
        mc.x[u] = j < k ? (mc.nans ? fmaf(0.f, pl.z, pl.x) : pl.x) : O.cx;   // NaN with the yaw, too
        mc.y[u] = j < k ? pl.y : O.cy;
    }
    mc.k = k;
    mc.p = p;
    if (GRAD) {
        for (int j = 0; j < 3 * K; ++j) gr[j] = 0.f;
    }

    // this slot's configuration (the transition's end b, row qb_row of the
    // staged particle) and the transition's start a (row qa_row, or q0)
    const int W = T->W;
    const int qb_row = b0 + (placing ? 7 : 0);
    const bool start_is_var = placing || k > 0;
    const int qa_row = placing ? b0 : b0 - CT_STEP_DIM + 7;
    auto qb = [&](int j) { return X(qb_row + j); };
    auto qa = [&](int j) { return start_is_var ? X(qa_row + j) : T->q0[j]; };

    float gq[CT_N_JOINTS], gqa[CT_N_JOINTS];
#pragma unroll
    for (int j = 0; j < CT_N_JOINTS; ++j) gq[j] = gqa[j] = 0.f;
    float gg[4] = {0.f, 0.f, 0.f, 0.f};
    float coll = 0.f, coll_m = 0.f, kin_pos = 0.f, kin_rot = 0.f, selfc = 0.f;
    int nhit = 0;   // touching sphere-box pairs (cost mode only; the adjoint's work)

    // waypoints w = 1..W of the transition, then the configuration itself
    for (int w = 1; w <= W + 1; ++w) {
        const bool key = w == W + 1;   // wave-uniform
        const float s = key ? 1.f : (float)w / (float)(W + 1);
        // sines and cosines of the configuration's joint angles: the SPLIT
        // lanes of the slot take every SPLIT-th joint and exchange them
        float jsn[CT_N_JOINTS], jcs[CT_N_JOINTS], gw[CT_N_JOINTS];
#pragma unroll
        for (int j0 = 0; j0 < CT_N_JOINTS; j0 += SPLIT) {
            const int j = min(j0 + si, CT_N_JOINTS - 1);
            float th0 = T->jk[j0].th0;
#pragma unroll
            for (int u = 1; u < SPLIT; ++u)
                if (j0 + u < CT_N_JOINTS && si == u) th0 = T->jk[j0 + u].th0;
            const float b = qb(j);
            float q = b;
            if (!key) {
                const float a = start_is_var ? X(qa_row + j) : T->q0[j];
                q = a + s * (b - a);
            }
            float sn, cs;
            sincosf(q + th0, &sn, &cs);
            sn = live ? sn : none;
            split_bcast<SPLIT>(sn, j0, jsn);
            split_bcast<SPLIT>(cs, j0, jcs);
        }
#pragma unroll
        for (int j = 0; j < CT_N_JOINTS; ++j) gw[j] = 0.f;
        float cw = 0.f;
        // the object is in the hand at both configurations of its step and
        // along the holding transition
        const bool held = key || placing;
        const float lam = key ? (sw ? sw->coll : T->w[W_COLL]) : (sw ? sw->mcoll : T->w[W_MCOLL]);
        config_pass<KT, SPLIT, GRAD, JU>(T, S, si, jsn, jcs, held, key, placing, lam, mc, gx, gy, gz, g_c, g_s, rho_x, rho_y,
                                     rho_c, rho_s, cw, gw, gg, gr, kin_pos, kin_rot, sw, key && self_on, selfc, nhit);
        if (key) coll += cw; else coll_m += cw;
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < CT_N_JOINTS; ++j) {
                gq[j] += s * gw[j];
                gqa[j] += (1.f - s) * gw[j];
            }
        }
    }
    if (!start_is_var) {
#pragma unroll
        for (int j = 0; j < CT_N_JOINTS; ++j) gqa[j] = 0.f;
    }

    // joint limits of this configuration; the transition's length
    float jlim = 0.f, traj = 0.f;
    if (si == 0) {
        float gj[CT_N_JOINTS], qk[CT_N_JOINTS];
#pragma unroll
        for (int j = 0; j < CT_N_JOINTS; ++j) qk[j] = qb(j);
        jlim = bounds_dist<CT_N_JOINTS>(qk, T->q_lo, T->q_hi, sw ? sw->jlim : T->w[W_JLIM], gj);
        if (GRAD) {
#pragma unroll
            for (int j = 0; j < CT_N_JOINTS; ++j) gq[j] += gj[j];
        }
        if (W > 0) {
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < CT_N_JOINTS; ++j) ss += (qb(j) - qa(j)) * (qb(j) - qa(j));
            traj = sqrtf(ss);
            if (GRAD && traj > 0.f) {
                const float sc = (sw ? sw->traj : T->w[W_TRAJ]) / traj;
#pragma unroll
                for (int j = 0; j < CT_N_JOINTS; ++j) {
                    gq[j] += sc * (qb(j) - qa(j));
                    if (start_is_var) gqa[j] -= sc * (qb(j) - qa(j));
                }
            }
        }
    }

    float grasp = 0.f, coll_obj = 0.f, place = 0.f, goal = 0.f;
    const float lc = sw ? sw->cobj : T->w[W_COLL];
    if (!placing) {
        if (si == 0) {
            const float gv[3] = {gx, gy, gz};
            float gb[3];
            grasp = bounds_dist<3>(gv, T->grasp_lo[k], T->grasp_hi[k], sw ? sw->grasp : T->w[W_GRASP], gb);
            if (GRAD) { gg[0] += gb[0]; gg[1] += gb[1]; gg[2] += gb[2]; }
        }
    }
    if (__ballot(!placing)) {
        // CFreePlace: the object's spheres at its placement P(rho_k); the
        // object frame's force and moment give the placement gradient
        const float Rp[9] = {rho_c, -rho_s, 0.f, rho_s, rho_c, 0.f, 0.f, 0.f, 1.f};
        const float tp[3] = {rho_x, rho_y, T->place_z[k]};
        float fp[3] = {0.f, 0.f, 0.f}, mp[3] = {0.f, 0.f, 0.f};
        object_spheres<KT, SPLIT, GRAD>(T, S, !placing, T->obs[k], si, Rp, tp, mc, lc, coll_obj, fp, mp, gr, nhit);
        if (GRAD && !placing) {
            // translation: the force; turning about the vertical through the
            // placement origin: z of the moment about that point
            gr[3 * k] += fp[0];
            gr[3 * k + 1] += fp[1];
            gr[3 * k + 2] += mp[2] - (tp[0] * fp[1] - tp[1] * fp[0]);
        }
    }
    if (placing && si == 0) {
        // StablePlace containment: footprint corners inside the region
        const float hx = T->obj0[k].hx, hy = T->obj0[k].hy, lpl = sw ? sw->place : T->w[W_PLACE];
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            const float sx = (cc & 1) ? hx : -hx, sy = (cc & 2) ? hy : -hy;
            const float vx = rho_c * sx - rho_s * sy, vy = rho_s * sx + rho_c * sy;
            const float cv[2] = {rho_x + vx, rho_y + vy};
            float gcr[2];
            place += bounds_dist<2>(cv, T->region_lo, T->region_hi, lpl, gcr);
            if (GRAD) {
                gr[3 * k] += gcr[0];
                gr[3 * k + 1] += gcr[1];
                gr[3 * k + 2] += -vy * gcr[0] + vx * gcr[1];
            }
        }
        if (slot == 1 && T->goal) {
            // MinimizeObjDist: sum of pairwise distances of the placements
            const float lg = sw ? sw->goal : T->w[W_GOAL];
            for (int a = 0; a < K; ++a)
                for (int b = a + 1; b < K; ++b) {
                    const float dx = plc[a * xs_stride].x - plc[b * xs_stride].x;
                    const float dy = plc[a * xs_stride].y - plc[b * xs_stride].y;
                    const float dz = T->place_z[a] - T->place_z[b];
                    const float dist = sqrtf(dx * dx + dy * dy + dz * dz);
                    goal += dist;
                    if (GRAD && dist > 0.f) {
                        const float sc = lg / dist;
                        gr[3 * a] += dx * sc; gr[3 * a + 1] += dy * sc;
                        gr[3 * b] -= dx * sc; gr[3 * b + 1] -= dy * sc;
                    }
                }
        }
    }

    // ---- penetration sums of the slot (all SPLIT lanes contribute)
    coll = split_sum<SPLIT>(coll);
    coll_m = split_sum<SPLIT>(coll_m);
    coll_obj = split_sum<SPLIT>(coll_obj);
    if (self_on) selfc = split_sum<SPLIT>(selfc);

    LaneOut out;
    const float* e = T->eps;
    float gsum = 0.f;
    if (GRAD) {
#pragma unroll
        for (int j = 0; j < CT_N_JOINTS; ++j) {
            part[j] = gq[j];
            if (W > 0) part[11 + 3 * K + j] = gqa[j];
            gsum += gq[j] + gqa[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) { part[7 + j] = gg[j]; gsum += gg[j]; }
        for (int j = 0; j < 3 * K; ++j) gsum += gr[j];
    }
    const SlotW swc = sw ? *sw : SlotW{T->w[W_KPOS], T->w[W_KROT], T->w[W_JLIM], T->w[W_COLL], T->w[W_MCOLL],
                                       T->w[W_SELF], T->w[W_GRASP], T->w[W_COLL], T->w[W_PLACE], T->w[W_GOAL],
                                       T->w[W_TRAJ]};
    float kw = swc.kpos * kin_pos + swc.krot * kin_rot + swc.jlim * jlim + swc.coll * coll + swc.mcoll * coll_m +
               swc.traj * traj;
    bool ok = kin_pos <= e[E_KPOS] && kin_rot <= e[E_KROT] && jlim <= e[E_JLIM] && coll <= e[E_COLL] &&
              coll_m <= e[E_MCOLL];
    if (self_on) {
        kw += swc.self * selfc;
        ok = ok && selfc <= e[E_SELF];
    }
    if (!placing) {
        out.cost = kw + swc.grasp * grasp + swc.cobj * coll_obj;
        ok = ok && grasp <= e[E_GRASP] && coll_obj <= e[E_COLL];
    } else {
        out.cost = kw + swc.place * place + swc.goal * goal;
        ok = ok && place <= e[E_PLACE];
    }
    out.traj = traj;
    out.hits = 0;
    if (!GRAD) out.hits = (int)split_sum<SPLIT>((float)nhit);   // exact: small integers
    // a slot is finite when its own cost and every lane's partials are
    const float gtot = split_sum<SPLIT>(gsum);
    const bool fin = __builtin_isfinite(out.cost) && __builtin_isfinite(gtot);
    out.flags = (ok ? 1 : 0) | (fin ? 2 : 0);

    if (write_terms && si == 0) {
        const int tb = CT_TERMS_PER_STEP * k;
        auto put = [&](int idx, float v) { terms[(int64_t)idx * term_ld + i_glob] = v; };
        if (!placing) {
            put(tb + T_PICK_POS, kin_pos);
            put(tb + T_PICK_ROT, kin_rot);
            put(tb + T_GRASP, grasp);
            put(tb + T_JLIM_G, jlim);
            put(tb + T_COLL_G, coll);
            put(tb + T_COLL_OBJ, coll_obj);
        } else {
            put(tb + T_PLACE_POS, kin_pos);
            put(tb + T_PLACE_ROT, kin_rot);
            put(tb + T_PLACE, place);
            put(tb + T_JLIM_P, jlim);
            put(tb + T_COLL_P, coll);
            if (slot == 1 && T->goal) put(T->goal_term, goal);
        }
        if (W > 0) put(CT_TERMS_PER_STEP * K + slot, coll_m);
        if (self_on) put(T->self_term + slot, selfc);
    }
    return out;
}

// ---------------------------------------------------------------------------
// Workgroup-level tile: P particles x 2K slots x SPLIT lanes.

// LDS of a tile (dynamic; the host passes tile_layout(...).total).  At K = 4,
// 60 robot spheres and 9 static boxes a fused step without waypoints takes
// 72,624 bytes at SPLIT 1 and 54,320 at SPLIT 2: two workgroups per compute unit.
__device__ __forceinline__ TileLds tile_lds(char* base, const TileLayout& o, int P) {
    TileLds S;
    S.xs = (float*)(base + o.xs);
    S.ms = (float*)(base + o.ms);
    S.vs = (float*)(base + o.vs);
    S.part = (float*)(base + o.part);
    S.plc = (float4*)(base + o.plc);
    S.rs = (float4*)(base + o.rs);
    S.osl = (float4*)(base + o.osl);
    S.sbx = (SBox*)(base + o.sbx);
    S.cbx = (CullBox*)(base + o.cbx);
    S.ck = (float2*)(base + o.ck);
    S.ob0 = (Box*)(base + o.ob0);
    S.cpart = (float*)(base + o.cpart);
    S.tpart = (float*)(base + o.tpart);
    S.flg = (int*)(base + o.flg);
    S.hpart = (int*)(base + o.hpart);
    S.okp = (int*)(base + o.okp);
    S.frz = (uint8_t*)(base + o.frz);
    S.ctl = (int*)(base + o.ctl);
    S.bc = (float2*)(base + o.bc);
    S.wave = (float4*)(base + o.wave);
    S.np = o.np;
    S.pp = o.pp;
    S.P = P;
    return S;
}

// What one tile reads and writes (one skeleton's buffers).
struct TileIO {
    const Tables* T;
    float *X, *M, *V, *G, *cost, *terms;
    uint8_t* mask;
    int32_t* first_sat;
    const uint8_t* frozen;
    const float* gw;
    int64_t n, ld;
    float gscale;
    const float* wts;   // per-particle term weights [n_terms][ld] (extended kernels), or null
    // stop-at-first: a satisfying particle is not updated, so X keeps it, and a
    // tile leaves its iteration loop after a step that found one
    int stop = 0;
    float *Xb = nullptr, *Mb = nullptr, *Vb = nullptr;   // copies of the state the launch started from, or null
    int32_t* own = nullptr;   // the iteration of the launch's stop, or null (a launch of one iteration)
    int redo = 0;   // start from those copies (or, null, from X), run every iteration, report nothing
    int32_t* hits = nullptr;   // cost mode: touching sphere-box pairs per particle, or null
    int per = 0;               // particles of a tile (1 .. P)
};


// The fused step runs `iters` updates t, t + 1, ... of the tile: particles are
// independent of each other (Eq. 4 is a mean, Adam is per coordinate), so X,
// M and V stay in LDS from the first update to the last and cross HBM once
// per launch, and no tile waits for another between iterations.  One launch
// per iteration paid the staging, the store, a launch gap and the slowest
// tile's tail every time.  cost and mask are those of the last iteration.
// Returns the number of iterations run (stop-at-first may leave early).
template <int KT, int SPLIT, int MODE, bool EXT>
__device__ __forceinline__ int run_tile(const TileIO& io, int64_t p0, char* lds, float lr, float b1,
                                        float b2, float eps, int32_t t, int iters) {
    const Tables* __restrict__ T = io.T;
    constexpr int K = KT;
    constexpr int SLOTS = 2 * K;
    constexpr int P = tile_particles(K, SPLIT);
    constexpr int D = CT_STEP_DIM * K;
    const int64_t n = io.n, ld = io.ld;
    const int tid = threadIdx.x;
    const int W = T->W, nsb = T->n_static;
    const TileLayout lay = tile_layout(K, SPLIT, MODE, W, nsb, T->link_start[9]);
    const TileLds S = tile_lds(lds, lay, P);
    const int NP = S.np;
    // the particle of column p (n: none): floor(p per / P) in the first column
    // that gives it
    const int per = io.per;
    auto particle = [&](int p) -> int64_t {
        const uint32_t at = (uint32_t)(p * per), j = at / P;
        return at - j * P < (uint32_t)per ? p0 + j : n;
    };
    // moments in LDS, or (waypoints: the partials leave no room) read and
    // written in place by every iteration
    constexpr bool MV = MODE == MODE_STEP;
    const bool mv_lds = MV && W == 0;

    // phase 0: stage this tile's particles (coalesced along particles) and,
    // for the fused step, their Adam moments and the frozen flags, and the
    // problem's tables.  A lane issues all of its loads before the first wait
    // (NST is an upper bound on its share), so the tile pays one memory latency here and none
    // in phase 2.
    {
        constexpr int NST = (D * P + WG - 1) / WG;
        float xv[NST], mv[NST], vv[NST];
#pragma unroll
        for (int u = 0; u < NST; ++u) {
            const int idx = tid + u * WG;
            const int d = idx / P, p = idx - d * P;
            const int64_t i = particle(p);
            xv[u] = mv[u] = vv[u] = 0.f;
            if (idx < D * P && i < n) {
                const int64_t a = d * ld + i;
                if (MV && io.redo && io.Xb) {
                    xv[u] = io.Xb[a]; mv[u] = io.Mb[a]; vv[u] = io.Vb[a];
                    if (!mv_lds) { io.M[a] = mv[u]; io.V[a] = vv[u]; }
                } else {
                    xv[u] = io.X[a];
                    if (MV && (mv_lds || io.Xb)) { mv[u] = io.M[a]; vv[u] = io.V[a]; }
                    if (MV && io.Xb) { io.Xb[a] = xv[u]; io.Mb[a] = mv[u]; io.Vb[a] = vv[u]; }
                }
            }
        }
        if (MV && tid < D) S.frz[tid] = io.frozen ? io.frozen[tid] : 0;
#pragma unroll
        for (int u = 0; u < NST; ++u) {
            const int idx = tid + u * WG;
            if (idx < D * P) {
                S.xs[idx] = xv[u];
                if (mv_lds) { S.ms[idx] = mv[u]; S.vs[idx] = vv[u]; }
            }
        }
    }
    for (int idx = tid; idx < K * CT_MAX_OBJ_SPHERES; idx += WG)
        S.osl[idx] = T->os[idx / CT_MAX_OBJ_SPHERES][idx % CT_MAX_OBJ_SPHERES];
    for (int idx = tid; idx < T->link_start[9]; idx += WG) S.rs[idx] = T->rs[idx];
    for (int idx = tid; idx < 8 * (nsb + K); idx += WG) S.ck[idx] = T->ck[idx];
    if (tid < nsb + K) S.cbx[tid] = T->cbx[tid];
    if (tid < nsb) S.sbx[tid] = T->sbox[tid];
    if (tid < K) S.ob0[tid] = T->obj0[tid];
    if (MV && tid >= WG - MAX_LAUNCH_ITERS) {
        const int u = tid - (WG - MAX_LAUNCH_ITERS);
        if (u < iters) S.bc[u] = make_float2(1.f - powf(b1, (float)(t + u)), 1.f - powf(b2, (float)(t + u)));
    }
    if (tid == 0) {
        S.ctl[0] = 0;   // some particle of the tile satisfies
        S.ctl[1] = 0;   // leave the loop
    }
    __syncthreads();

    int done = 0;
    bool reported = false;
    float J = 0.f;   // cost and mask of the iteration (lanes tid < P)
    int m = 0;
    for (;;) {
        const int32_t iter = t + done - 1;   // 0-based index of this iteration
        const bool last = MODE != MODE_STEP || done + 1 == iters;
        // stop-at-first: an earlier iteration of another tile found a particle
        // (never at the first, so an iteration always ran before the loop ends)
        if (MODE == MODE_STEP && io.own && tid == 0)
            S.ctl[1] = __hip_atomic_load(io.own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < iter ? 1 : 0;
        for (int idx = tid; idx < K * P; idx += WG) {
            const int j = idx / P, p = idx - j * P;
            const float* col = S.xs + p;
            float sj, cj;
            sincosf(col[(CT_STEP_DIM * j + 20) * P], &sj, &cj);
            S.plc[idx] = make_float4(col[(CT_STEP_DIM * j + 18) * P], col[(CT_STEP_DIM * j + 19) * P], cj, sj);
        }
        __syncthreads();
        if (MODE == MODE_STEP && S.ctl[1]) break;   // workgroup-uniform

        // phase 1: every lane evaluates its slot.  Lanes are slot-major (the SPLIT
        // lanes of a slot adjacent, then the tile's particles, then the slots), so
        // a wave serves one or two slots of many particles: the same step and kind
        // of configuration, hence uniform branches and coherent box masks.
        {
            const int si = tid % SPLIT, rest = tid / SPLIT;
            const int slot = rest / P, p = rest - slot * P;
            if (slot < SLOTS) {
                const int64_t i = particle(p);
                const bool wt = (MODE == MODE_COST) && io.terms != nullptr && i < n;
                // the table pointer is made opaque per iteration: hoisted out of
                // the loop, the tables' values would not fit the registers
                // (constant address space: they are read with scalar loads)
                uint64_t Ta = (uint64_t)T;
                asm volatile("" : "+s"(Ta));
                const Tables* Ti = (const Tables*)(const __attribute__((address_space(4))) Tables*)Ta;
                const LaneOut o = lane_slot<KT, SPLIT, MODE, EXT>(Ti, S, p, slot, si,
                                                                  S.part + p * S.pp + (slot * SPLIT + si) * NP,
                                                                  io.terms, ld, i, wt, i < n ? io.wts : nullptr, i < n);
                if (si == 0) {
                    S.cpart[p * SLOTS + slot] = o.cost;
                    if (W > 0) S.tpart[p * SLOTS + slot] = o.traj;
                    S.flg[p * SLOTS + slot] = o.flags;
                    if (MODE == MODE_COST) S.hpart[p * SLOTS + slot] = o.hits;
                }
            }
        }
        __syncthreads();

        // phase 1.5: per-particle cost, mask, update permission
        if (tid < P) {
            const int64_t i = particle(tid);
            int ok = 1;
            J = 0.f;
            m = 1;
            for (int s = 0; s < SLOTS; ++s) {
                J += S.cpart[tid * SLOTS + s];
                m &= S.flg[tid * SLOTS + s] & 1;
                ok &= (S.flg[tid * SLOTS + s] >> 1) & 1;
            }
            ok &= __builtin_isfinite(J) ? 1 : 0;
            m &= __builtin_isfinite(J) ? 1 : 0;
            // the solution returned on stop is the satisfying iterate itself
            // (the pre-update x the mask describes), so it keeps its value
            S.okp[tid] = ok & (io.stop ? 1 - m : 1);
            if (i < n) {
                if (MODE == MODE_COST && io.terms && T->traj_term >= 0) {
                    float tl = 0.f;
                    for (int s = 0; s < SLOTS; ++s) tl += S.tpart[tid * SLOTS + s];
                    io.terms[(int64_t)T->traj_term * ld + i] = tl;
                }
                if (MODE == MODE_COST && io.hits) {
                    int h = 0;
                    for (int s = 0; s < SLOTS; ++s) h += S.hpart[tid * SLOTS + s];
                    io.hits[i] = h;
                }
                if (m) S.ctl[0] = 1;
            }
        }
        __syncthreads();
        const bool sat = S.ctl[0];   // workgroup-uniform; stays set: only the first iteration counts
        if (sat && !reported && io.first_sat && !io.redo && tid == 0) {
            atomicMin(io.first_sat, iter);
            if (io.own) atomicMin(io.own, iter);
        }
        reported = reported || sat;

        if (MODE != MODE_COST) {
            // phase 2: sum each coordinate's partials over slots and split lanes
            // in a fixed order, then write G or apply Adam in place
            const float2 bc = MODE == MODE_STEP ? S.bc[done] : make_float2(1.f, 1.f);
            const float bc1 = bc.x, bc2 = bc.y;
            const int FQ = 11 + 3 * K;   // foreign-configuration partials
            for (int idx = tid; idx < D * P; idx += WG) {
                const int d = idx / P, p = idx - d * P;
                const int64_t i = particle(p);
                if (i >= n) continue;
                const int k = d / CT_STEP_DIM, r = d - CT_STEP_DIM * k;
                const float* pp = S.part + p * S.pp;
                auto lane = [&](int slot, int si) { return pp + (slot * SPLIT + si) * NP; };
                float g = 0.f;
#pragma unroll
                for (int si = 0; si < SPLIT; ++si) {
                    if (r < 7) {
                        // q_grasp of step k: its slot, plus (waypoints) the start of the holding transition
                        g += lane(2 * k, si)[r] + (W > 0 ? lane(2 * k + 1, si)[FQ + r] : 0.f);
                    } else if (r < 14) {
                        // q_place of step k: its slot, plus (waypoints) the start of the next free transition
                        g += lane(2 * k + 1, si)[r - 7];
                        if (W > 0 && k + 1 < K) g += lane(2 * k + 2, si)[FQ + (r - 7)];
                    } else if (r < 18) {
                        g += lane(2 * k, si)[7 + (r - 14)] + lane(2 * k + 1, si)[7 + (r - 14)];
                    } else {
                        for (int s = 0; s < SLOTS; ++s) g += lane(s, si)[11 + 3 * k + (r - 18)];
                    }
                }
                if (MODE == MODE_GRAD) {
                    const int64_t a = d * ld + i;
                    io.G[a] = io.gw ? io.gw[i] * g : g;
                } else if (!S.frz[d]) {
                    if (!S.okp[p]) continue;
                    const int64_t a = d * ld + i;
                    const float gs = io.gscale * g;
                    const float m1 = b1 * (mv_lds ? S.ms[idx] : io.M[a]) + (1.f - b1) * gs;
                    const float v1 = b2 * (mv_lds ? S.vs[idx] : io.V[a]) + (1.f - b2) * gs * gs;
                    const float mh = m1 / bc1, vh = v1 / bc2;
                    S.xs[idx] = S.xs[idx] - lr * mh / (sqrtf(vh) + eps);
                    if (mv_lds) {
                        S.ms[idx] = m1;
                        S.vs[idx] = v1;
                    } else {
                        io.M[a] = m1;
                        io.V[a] = v1;
                    }
                }
            }
        }
        ++done;
        if (last || (io.stop && sat && !io.redo)) break;   // workgroup-uniform
        __syncthreads();
    }

    if (tid < P && particle(tid) < n) {
        if (io.cost) io.cost[particle(tid)] = J;
        if (io.mask) io.mask[particle(tid)] = (uint8_t)m;
    }
    if (MODE == MODE_STEP) {
        // every entry by the lane that updated it in phase 2
        for (int idx = tid; idx < D * P; idx += WG) {
            const int d = idx / P, p = idx - d * P;
            const int64_t i = particle(p);
            if (i >= n || S.frz[d]) continue;
            const int64_t a = d * ld + i;
            io.X[a] = S.xs[idx];
            if (mv_lds) {
                io.M[a] = S.ms[idx];
                io.V[a] = S.vs[idx];
            }
        }
    }
    return done;
}

// ---------------------------------------------------------------------------
// One skeleton of KT steps: one workgroup per tile (XCD-aware tile order).
// Stop-at-first over several iterations: tiles do not wait for each other, so
// a tile may run past the iteration at which another found the first
// satisfying particle.  The launch therefore keeps a copy of the state it
// started from, and a second launch (redo) runs the tiles that went past that
// iteration again, from the copy, up to it.  A launch of one iteration needs
// no copy.  first_sat may be shared with other solves and drop at any time: a
// workgroup reads it once, at entry.  Should some workgroups of a launch have
// found the solve stopped and others not, the second launch runs the former
// forward to where the latter are.
template <int SPLIT, int MODE, int KT, bool EXT>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2))) void particle_kernel(
    const Tables* __restrict__ T, float* __restrict__ X, float* __restrict__ M, float* __restrict__ V,
    float* __restrict__ G, float* __restrict__ cost, float* __restrict__ terms, uint8_t* __restrict__ mask,
    int32_t* __restrict__ first_sat, const uint8_t* __restrict__ frozen, int64_t n, int64_t ld, float lr,
    float b1, float b2, float eps, float gscale, int32_t t, int32_t iters, int32_t per, StopArgs stop, const float* __restrict__ gw,
    const float* __restrict__ wts, int32_t* __restrict__ hits) {
    extern __shared__ __attribute__((aligned(16))) char tile_mem[];
    int run = iters;
    bool fresh = false;   // redo of a workgroup that has not run
    if (MODE == MODE_STEP && stop.on) {
        int32_t* word = (int32_t*)tile_mem;
        if (stop.redo) {
            // everything read here was written by the launch before
            const int32_t ran = stop.ran[blockIdx.x], f = *stop.own;
            if (f != STOP_NONE) run = f - t + 2;
            if (ran == run) return;
            if (ran == 0) {   // run now if any other workgroup did
                if (threadIdx.x == 0) *word = 0;
                __syncthreads();
                for (uint32_t b = threadIdx.x; b < gridDim.x; b += WG)
                    if (stop.ran[b]) *word = 1;
                __syncthreads();
                fresh = *word;
                __syncthreads();
                if (!fresh) return;
            }
        } else {
            if (threadIdx.x == 0) *word = __hip_atomic_load(first_sat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int32_t f = *word;
            __syncthreads();
            if (stop.own && threadIdx.x == 0) {
                if (blockIdx.x == 0) *stop.own_next = STOP_NONE;
                if (f < t - 1)
                    stop.ran[blockIdx.x] = 0;
                else if (f <= t - 2 + iters)
                    atomicMin(stop.own, f);   // stopped inside the launch
            }
            if (f < t - 1) return;   // stopped before this launch
        }
    }
    // XCD-aware tile order: consecutive workgroups are dealt round-robin to the
    // 8 XCDs, so give each XCD a contiguous range of particle tiles; tiles
    // that share cache lines of X, M and V then share one L2
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    TileIO io{T, X, M, V, G, cost, terms, mask, first_sat, frozen, gw, n, ld, gscale, EXT ? wts : nullptr};
    io.per = per;
    if (MODE == MODE_COST) io.hits = hits;
    if (MODE == MODE_STEP) {
        io.stop = stop.on;
        io.Xb = fresh ? nullptr : stop.Xb;
        io.Mb = stop.Mb;
        io.Vb = stop.Vb;
        io.redo = stop.redo;
        io.own = stop.redo ? nullptr : stop.own;
    }
    const int ran = run_tile<KT, SPLIT, MODE, EXT>(io, tile * per, tile_mem, lr, b1, b2, eps, t, run);
    if (MODE == MODE_STEP && stop.ran && !stop.redo && threadIdx.x == 0) stop.ran[blockIdx.x] = ran;
}


__device__ __forceinline__ float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// One tile of a skeleton of KT steps for the many-skeleton kernel.  The length
// is compiled in: with the length at run time the kernel kept 336 bytes of
// spills per lane and read the moved objects from LDS (64 skeletons of 1 to 6
// steps: 41.4 ms per 50 iterations, 36.9 with it compiled in).  It is a
// function of its own, not inlined, since six inlined copies share no stack
// and keep 2.1 KB (39.4 ms).  A function's arguments arrive in vector
// registers; all of them are the same for the whole workgroup and are made
// uniform again, so the tables stay scalar loads.
template <int KT, int SPLIT, bool EXT>
__device__ __attribute__((noinline)) void batch_tile(uint64_t skel, uint32_t lds, int32_t tile, float lr, float b1,
                                                     float b2, float eps, int32_t t, int32_t iters) {
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)skel);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(skel >> 32));
    const BatchSkel& b = *(const BatchSkel*)(const __attribute__((address_space(4))) BatchSkel*)(hi << 32 | lo);
    TileIO io{b.T, b.X, b.M, b.V, nullptr, b.cost, nullptr, b.mask, b.first_sat, b.frozen, nullptr,
                    b.n, b.ld, b.gscale};
    io.per = b.per;
    char* mem = (char*)(__attribute__((address_space(3))) char*)__builtin_amdgcn_readfirstlane(lds);
    run_tile<KT, SPLIT, MODE_STEP, EXT>(io, (int64_t)__builtin_amdgcn_readfirstlane(tile) * b.per,
                                        mem, uniform(lr), uniform(b1), uniform(b2), uniform(eps),
                                        __builtin_amdgcn_readfirstlane(t), __builtin_amdgcn_readfirstlane(iters));
}

// Many skeletons of different lengths and sizes, `iters` iterations in one
// launch: a fixed number of workgroups pull (skeleton, tile) items from a
// device queue (items ordered by cost, largest first) until it is empty, and
// run every iteration of an item before they take the next; the last
// workgroup to leave resets the queue for the next launch.
template <int SPLIT, bool EXT>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2))) void batch_kernel(const BatchSkel* __restrict__ skels,
                                                   const int2* __restrict__ items, int32_t n_items,
                                                   int32_t* __restrict__ queue, float lr, float b1, float b2,
                                                   float eps, int32_t t, int32_t iters) {
    extern __shared__ __attribute__((aligned(16))) char tile_mem[];
    int& item_s = *(int*)tile_mem;   // ahead of the tile's own LDS
    for (;;) {
        if (threadIdx.x == 0) item_s = atomicAdd(&queue[0], 1);
        __syncthreads();
        // the item is the same for the whole workgroup: make it wave-uniform
        // so the skeleton's tables are read through the scalar cache
        const int it = __builtin_amdgcn_readfirstlane(item_s);
        __syncthreads();
        if (it >= n_items) break;
        const int2 w = items[it];
        const uint64_t sk = (uint64_t)&skels[w.x];
        const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(tile_mem + 16);
        switch (skels[w.x].T->K) {
            case 1: batch_tile<1, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
            case 2: batch_tile<2, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
            case 3: batch_tile<3, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
            case 4: batch_tile<4, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
            case 5: batch_tile<5, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
            default: batch_tile<6, SPLIT, EXT>(sk, lds, w.y, lr, b1, b2, eps, t, iters); break;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&queue[1], 1) == (int)gridDim.x - 1) {
            atomicExch(&queue[0], 0);
            atomicExch(&queue[1], 0);
        }
    }
}

}  // namespace ct
