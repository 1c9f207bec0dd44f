// k_walk.hip -- Barnes-Hut tree walks: the forward walk (g, j, T at the
// active targets) and the adjoint walk (gradient of L = sum_k w_k . g_k).
//
// Work decomposition: the active targets, in key (Morton) order, are cut
// into groups of at most 64 consecutive targets of one system; one wave64,
// or a team of waves where groups are few, walks the tree once for the whole
// group, and waves left without a group take tiles of the others.  Every lane owns
// one target; in a group of fewer than 64 targets each target is given
// several lanes, which share out the interaction list and add their parts
// at the end, so the wave stays full.  The opening test is applied to the group's bounding box
// (conservative: a node is accepted only if it would be for every point of
// the box), so the whole wave follows one traversal with no divergence in
// the interaction loops.
//
// Traversal: nodes are numbered in depth-first pre-order with a "skip" link
// past each subtree, so any range [a, b) of sibling subtrees can be walked
// by one cursor without a stack (test a; accept or leaf -> a = skip[a];
// open -> a = a + 1).  The 64 lanes hold 64 such cursors and test 64 nodes
// per step; a lane that opens a node hands the rest of its range to an LDS
// stack of ranges that idle lanes pop (load balancing).  Accepted nodes and
// the particles of opened leaves are appended (ballot prefix sums) to LDS
// lists; every 64 entries the wave stages them as FP32 data relative to the
// group centre in LDS and all lanes evaluate the tile (LDS broadcast reads),
// folding the FP32 tile sums into FP64 accumulators.
#include <float.h>

#include <algorithm>
#include <climits>

#include "ag_internal.h"
#include "pair.h"

namespace {

constexpr int kW = 64;          // lanes per wave = targets per group = tile size
constexpr int kPCap = 256;      // pending particle indices
constexpr int kListSlack = 64;  // room behind them for what list_run writes past the end
constexpr int kNCap = 128;      // pending accepted nodes
constexpr int kSCap = 128;      // stacked cursor ranges
constexpr int kMaxSub = 32;     // most lanes given to one target of a small group
// boundary modes of a walk instance
constexpr int kOpen = 0;        // open boundaries
constexpr int kNear = 1;        // periodic, every pair at its nearest image
constexpr int kEwald = 2;       // periodic with Ewald sums: g and T at the images about the group
                                // centre (the correction walk uses the same ones), j at the nearest

// algorithmic operation count of one particle-particle interaction as written
// in ForwardPolicy::particles (outside the softening kernel; every add,
// subtract and multiply = 1, reciprocal square root = 1):
//   d and nu 6, r2 5, rsqrt 1, ri2 1, mf 2, mD 2, g 6, d.nu 5, s 1, j 12,
//   t 3, m f I 1, S 12                                                 = 57
constexpr int AG_WALK_PP_FLOPS = 57;
// algorithmic operation count of one particle-node interaction as written in
// node_interact (monopole + quadrupole g and T, mean-velocity + quadrupole-rate
// jerk; every add, subtract and multiply = 1, reciprocal square root = 1):
//   d and nu 6, r2 5, rsqrt 1, powers 4, P = Q d 15, d.P 5, h e hq 3, ca 2,
//   beta 4, g 12, e P 3, w 6, ca I 1, S diagonal 15, S off-diagonal 18,
//   V = Q nu + Qd d 33, d.nu 5, P.nu 5, d.Qd.d 6, cd 5, cp 1, j 24     = 179
constexpr int AG_PN_FLOPS = 179;

struct Tree {
    const NodeRec* __restrict__ rec;
    const int4* __restrict__ link;     // skip, start, count, level | leaf
    const float4* __restrict__ mp;     // 4 per node
    const double4* __restrict__ spos;  // sorted x, y, z, m
    const float4* __restrict__ svf;    // sorted vx, vy, vz, m
    const int32_t* __restrict__ perm;
    const int32_t* __restrict__ sys_root;
    const double4* __restrict__ ws;    // adjoint: sorted weights (w, 1 if charged)
    const float4* __restrict__ wf;     // adjoint: node charges, 4 per node
    const float* __restrict__ sh;      // sorted per-particle softening lengths, or null
};

struct Groups {
    const int32_t* __restrict__ act_pos;
    const int4* __restrict__ grp;      // start, count, system
    const int32_t* __restrict__ hdr;   // [0] = number of groups, [1] = targets in them
    const int32_t* __restrict__ ord;   // the order in which teams of kMinTeam walk them (open boundaries)
};

// Numbers of groups that are walked in an order of their own (k_group_order): above
// `least`, the teams of a walk, which start that many at once in any order; up to
// `most`, above which single waves walk them, and no more than kOrderMax, which one
// workgroup orders in 9 us (a larger AG_OPT_WALK_WAVES_PER_CU has teams walk more:
// those go in the list's order).
constexpr int kOrderMax = 16384;
struct OrderRange {
    int least, most;
    __device__ __forceinline__ bool holds(int n_groups) const { return n_groups > least && n_groups <= most; }
};

struct WalkOut {
    double* acc;
    double* jerk;
    double* tidal;
    unsigned long long* stats;
    double G;
    int32_t* flags;
    unsigned iter_cap;  // > nodes + particles: every group finishes well within it
    int small_node;     // accepted nodes this small are summed pairwise
    bool mac_offset;    // opening test adds the centre-of-mass offset to the extent
    const float* rel_a; // relative opening test: |a| of the last evaluation per row (null: off)
    float rel_alpha;
    float rel_g;        // |G| of the relative test
    double box, box_inv;        // periodic cube side and inverse (periodic walks only)
    float boxf, boxf_inv, box_half;
    // Ewald correction table: (NE + 1)^3 points of spacing h over [0, NE h]^3,
    // 5 float4 each (dg 3, dT 6, H 10, pad), and the correction walk's limits
    const float4* etab;
    float etab_h, etab_hinv, etab_range;
    int etab_ne;
    float ewald_theta;  // correction walk: opening angle against the nearest image point
    float ewald_grp;    // groups of at most this half extent sum the correction once
    double* dldx;       // adjoint outputs
    double* dldm;
    const double* tin;  // adjoint: tidal tensor rows of the charged targets
};

// group geometry shared by every lane (uniform values)
struct GroupBox {
    double cx, cy, cz;          // centre (FP64)
    double ox, oy, oz;          // origin of the source images (periodic walks; else the centre)
    float hx, hy, hz;           // half extents (rounded up)
    float lox, loy, loz, hix, hiy, hiz;   // absolute box, rounded outward
    float amin;                 // relative opening test: smallest |a| of the group's targets
};

// d rounded to float towards minus or plus infinity (kept within the finite
// floats): the nearest float, or where that lies on the wrong side its
// neighbour, by counting the bits.
__device__ __forceinline__ float f_dn(double d) {
    const float f = (float)d;
    const int b = __float_as_int(f);
    const float g = f == 0.f ? -FLT_TRUE_MIN : __int_as_float(b + (b < 0 ? 1 : -1));
    return (double)f > d ? fmaxf(g, -FLT_MAX) : f;
}
__device__ __forceinline__ float f_upr(double d) { return -f_dn(-d); }

__device__ __forceinline__ GroupBox group_box(double x, double y, double z) {
    double mnx = x, mny = y, mnz = z;
    double mxx = x, mxy = y, mxz = z;
    mnx = ag_wave_min_f64(mnx); mny = ag_wave_min_f64(mny); mnz = ag_wave_min_f64(mnz);
    mxx = ag_wave_max_f64(mxx); mxy = ag_wave_max_f64(mxy); mxz = ag_wave_max_f64(mxz);
    GroupBox g;
    g.cx = 0.5 * (mnx + mxx); g.cy = 0.5 * (mny + mxy); g.cz = 0.5 * (mnz + mxz);
    g.ox = g.cx; g.oy = g.cy; g.oz = g.cz;
    g.hx = f_upr(0.5 * (mxx - mnx)); g.hy = f_upr(0.5 * (mxy - mny)); g.hz = f_upr(0.5 * (mxz - mnz));
    g.lox = f_dn(mnx); g.loy = f_dn(mny); g.loz = f_dn(mnz);
    g.hix = f_upr(mxx); g.hiy = f_upr(mxy); g.hiz = f_upr(mxz);
    return g;
}

// nearest periodic image of a separation: d - L rint(d / L)
__device__ __forceinline__ double near_img(double d, const WalkOut& O) { return d - O.box * rint(d * O.box_inv); }
__device__ __forceinline__ float near_imgf(float d, const WalkOut& O) {
    return __builtin_fmaf(-O.boxf, rintf(d * O.boxf_inv), d);
}

// Opening test for a node's record against the group box.
// Accept iff  L' <= theta * r_min  (r_min: distance from the node's centre of
// mass to the nearest point of the group box; L' the node's extent L, plus,
// with mac_offset set, the distance from its centre of mass to the centre of
// its box, which opens lopsided nodes sooner)  and the node's box is at least
// eps away from the group box (so only Newtonian pairs are approximated).
// Periodic (kPer != 0): distances are taken at the nearest image of the node, and
// a node is accepted only if, along every axis, all of its box lies within
// half a box side of all of the group box -- then every particle-target pair
// of the node has that same nearest image, and the multipole stands for it.
template <int kPer>
__device__ __forceinline__ bool mac_accept(const GroupBox& g, const NodeRec& c, float theta2, float eps2, const WalkOut& O) {
    const float4 lo = c.lo, hi = c.hi;
    double cdx = c.x - g.cx, cdy = c.y - g.cy, cdz = c.z - g.cz;
    if (kPer) {   // the node's image about the image origin, seen from the group centre
        cdx = near_img(c.x - g.ox, O) + (g.ox - g.cx);
        cdy = near_img(c.y - g.oy, O) + (g.oy - g.cy);
        cdz = near_img(c.z - g.oz, O) + (g.oz - g.cz);
    }
    const float rx = fmaxf(fabsf((float)cdx) - g.hx, 0.f);
    const float ry = fmaxf(fabsf((float)cdy) - g.hy, 0.f);
    const float rz = fmaxf(fabsf((float)cdz) - g.hz, 0.f);
    // (the order of these sums is written out: left to the compiler it changes with
    // the code around it, and a node on the edge of the test with it)
    const float r2 = __builtin_fmaf(rz, rz, __builtin_fmaf(rx, rx, ry * ry));
    const float L = O.mac_offset ? c.mac : c.len;
    float gx, gy, gz;
    float bx, by, bz;   // box centre offset from the group centre (at its nearest image)
    if (!kPer) {
        gx = fmaxf(fmaxf(lo.x - g.hix, g.lox - hi.x), 0.f);
        gy = fmaxf(fmaxf(lo.y - g.hiy, g.loy - hi.y), 0.f);
        gz = fmaxf(fmaxf(lo.z - g.hiz, g.loz - hi.z), 0.f);
    } else {
        // box centre offset at its nearest image, and the half extents
        bx = fabsf((float)(near_img(0.5 * ((double)lo.x + (double)hi.x) - g.ox, O) + (g.ox - g.cx)));
        by = fabsf((float)(near_img(0.5 * ((double)lo.y + (double)hi.y) - g.oy, O) + (g.oy - g.cy)));
        bz = fabsf((float)(near_img(0.5 * ((double)lo.z + (double)hi.z) - g.oz, O) + (g.oz - g.cz)));
        const float ex = 0.5f * (hi.x - lo.x) + g.hx;
        const float ey = 0.5f * (hi.y - lo.y) + g.hy;
        const float ez = 0.5f * (hi.z - lo.z) + g.hz;
        // nearest images only: one image for the whole node (the nearest-image
        // field jumps at half a box from each target, so a node across that
        // cut is opened); with Ewald sums the field of all images is smooth
        // there, and every source stands at its image about the image origin,
        // whose cut (half a box away, on a boundary of the root's children)
        // no node below the root crosses
        if (kPer == kNear && (bx + ex >= O.box_half || by + ey >= O.box_half || bz + ez >= O.box_half))
            return false;
        gx = fmaxf(bx - ex, 0.f);
        gy = fmaxf(by - ey, 0.f);
        gz = fmaxf(bz - ez, 0.f);
    }
    const float sep2 = __builtin_fmaf(gz, gz, __builtin_fmaf(gx, gx, gy * gy));
    if (!(r2 > 0.f && L * L <= theta2 * r2 && sep2 >= eps2)) return false;
    if (!O.rel_a) return true;
    // Relative test (Springel 2005) on top of the geometric one: a node of
    // mass M (hi.w) and extent Ln at distance r is used only if
    // G M Ln^2 / r^4 <= alpha |a_old|, the size its truncation error scales
    // with against a fraction of the target's last acceleration, and only if
    // the target lies outside the cube of side 1.2 Ln about the node's box
    // centre.  For a group, r is the distance from the centre of mass to the
    // group's box (r2 above) and |a_old| the smallest of its targets, so
    // every target passes; the cube must miss the whole group box.
    const float Ln = c.len;
    if (!(O.rel_g * hi.w * Ln * Ln <= O.rel_alpha * g.amin * (r2 * r2))) return false;
    if (!kPer) {
        bx = fabsf((float)(0.5 * ((double)lo.x + (double)hi.x) - g.cx));
        by = fabsf((float)(0.5 * ((double)lo.y + (double)hi.y) - g.cy));
        bz = fabsf((float)(0.5 * ((double)lo.z + (double)hi.z) - g.cz));
    }
    {
        // (x with one rounding, y and z with two, written out: that is how the compiler
        // contracted these sums when the test's results were first taken, and a target
        // on the cube's face would change sides with another choice)
#pragma clang fp contract(off)
        const float e = 0.6f * Ln;
        return !(bx < __builtin_fmaf(0.6f, Ln, g.hx) && by < e + g.hy && bz < e + g.hz);
    }
}

// particle-node interaction at quadrupole order.  d = node centre - target,
// nu = node velocity - target velocity, P = Q d, q = d.P:
//   g = ca d - ri5 P,                 ca = M ri3 + 2.5 q ri7
//   S = ca I - beta d d^T - ri5 Q + e (P d^T + d P^T),
//                                     beta = 3 M ri5 + 17.5 q ri9, e = 5 ri7
//   j = S nu - ri5 Qd d + 2.5 (d.Qd.d) ri7 d
//     = ca nu + cd d + cp P - ri5 V,  V = Q nu + Qd d,
//       cd = e P.nu - beta d.nu + 2.5 ri7 (d.Qd.d),  cp = e d.nu,
// with d.Qd.d = d.V - P.nu (Q is symmetric).  Accumulates g, j and S = -T
// (pair.h's convention); the ca I part of S is summed into
// `sca` and added to the diagonal once per tile.
template <bool kTidal>
__device__ __forceinline__ void node_interact(float dx, float dy, float dz, float nx, float ny, float nz,
                                              float M, const float* Q, const float* Qd, PairAcc<float>& A,
                                              float& sca) {
    // written as explicit multiply-add chains into the accumulators (the
    // compiler does not reassociate sums on its own)
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
    const float ri = __builtin_amdgcn_rsqf(r2);
    const float ri2 = ri * ri;
    const float ri3 = ri * ri2;
    const float ri5 = ri3 * ri2;
    const float ri7 = ri5 * ri2;
    // Q = (xx yy zz xy xz yz)
    const float Px = __builtin_fmaf(Q[4], dz, __builtin_fmaf(Q[3], dy, Q[0] * dx));
    const float Py = __builtin_fmaf(Q[5], dz, __builtin_fmaf(Q[1], dy, Q[3] * dx));
    const float Pz = __builtin_fmaf(Q[2], dz, __builtin_fmaf(Q[5], dy, Q[4] * dx));
    const float q = __builtin_fmaf(dz, Pz, __builtin_fmaf(dy, Py, dx * Px));
    const float h = 2.5f * ri7;
    const float e = 5.f * ri7;
    const float hq = h * q;
    const float ca = __builtin_fmaf(M, ri3, hq);
    const float beta = ri2 * __builtin_fmaf(4.f, hq, 3.f * ca);
    const float nr5 = -ri5;
    if (!kTidal) {
        A.ax = __builtin_fmaf(nr5, Px, __builtin_fmaf(ca, dx, A.ax));
        A.ay = __builtin_fmaf(nr5, Py, __builtin_fmaf(ca, dy, A.ay));
        A.az = __builtin_fmaf(nr5, Pz, __builtin_fmaf(ca, dz, A.az));
    }
    const float ePx = e * Px, ePy = e * Py, ePz = e * Pz;
    const float wx = __builtin_fmaf(-beta, dx, ePx), wy = __builtin_fmaf(-beta, dy, ePy),
                wz = __builtin_fmaf(-beta, dz, ePz);
    sca += ca;
    A.sxx = __builtin_fmaf(nr5, Q[0], __builtin_fmaf(wx + ePx, dx, A.sxx));
    A.syy = __builtin_fmaf(nr5, Q[1], __builtin_fmaf(wy + ePy, dy, A.syy));
    A.szz = __builtin_fmaf(nr5, Q[2], __builtin_fmaf(wz + ePz, dz, A.szz));
    A.sxy = __builtin_fmaf(nr5, Q[3], __builtin_fmaf(ePy, dx, __builtin_fmaf(wx, dy, A.sxy)));
    A.sxz = __builtin_fmaf(nr5, Q[4], __builtin_fmaf(ePz, dx, __builtin_fmaf(wx, dz, A.sxz)));
    A.syz = __builtin_fmaf(nr5, Q[5], __builtin_fmaf(ePz, dy, __builtin_fmaf(wy, dz, A.syz)));
    if (kTidal) return;
    const float Vx = __builtin_fmaf(Qd[4], dz, __builtin_fmaf(Qd[3], dy, __builtin_fmaf(Qd[0], dx,
                     __builtin_fmaf(Q[4], nz, __builtin_fmaf(Q[3], ny, Q[0] * nx)))));
    const float Vy = __builtin_fmaf(Qd[5], dz, __builtin_fmaf(Qd[1], dy, __builtin_fmaf(Qd[3], dx,
                     __builtin_fmaf(Q[5], nz, __builtin_fmaf(Q[1], ny, Q[3] * nx)))));
    const float Vz = __builtin_fmaf(Qd[2], dz, __builtin_fmaf(Qd[5], dy, __builtin_fmaf(Qd[4], dx,
                     __builtin_fmaf(Q[2], nz, __builtin_fmaf(Q[5], ny, Q[4] * nx)))));
    const float dn = __builtin_fmaf(dz, nz, __builtin_fmaf(dy, ny, dx * nx));
    const float Pn = __builtin_fmaf(Pz, nz, __builtin_fmaf(Py, ny, Px * nx));
    const float qd = __builtin_fmaf(dz, Vz, __builtin_fmaf(dy, Vy, __builtin_fmaf(dx, Vx, -Pn)));
    const float cd = __builtin_fmaf(h, qd, __builtin_fmaf(-beta, dn, e * Pn));
    const float cp = e * dn;
    A.jx = __builtin_fmaf(nr5, Vx, __builtin_fmaf(cp, Px, __builtin_fmaf(cd, dx, __builtin_fmaf(ca, nx, A.jx))));
    A.jy = __builtin_fmaf(nr5, Vy, __builtin_fmaf(cp, Py, __builtin_fmaf(cd, dy, __builtin_fmaf(ca, ny, A.jy))));
    A.jz = __builtin_fmaf(nr5, Vz, __builtin_fmaf(cp, Pz, __builtin_fmaf(cd, dz, __builtin_fmaf(ca, nz, A.jz))));
}

// one staged tile of sources (layout set by the policy)
template <int NT>
struct TileLds {
    float4 tile[NT * kW];
    int tidx[kW];          // sorted index of each staged particle (self exclusion)
};
// lists of one traversal
struct ListLds {
    int plist[kPCap + kListSlack];
    int nlist[kNCap];
    int2 stack[kSCap];
};
// LDS of a wave that walks a group on its own
template <int NT>
struct WalkLds : ListLds, TileLds<NT> {};

struct Target {
    float tx, ty, tz;      // position relative to the group centre
    float vx, vy, vz;
    int p;                 // sorted position
    bool grp;              // Ewald correction summed once for the whole group
    float g0x, g0y, g0z;   // group centre relative to the image origin
    float h, hinv;         // the target's own softening length (per-particle softening)
};

// f and D of one softening length: the spline inside it, Newtonian beyond
__device__ __forceinline__ void soft_fd(float r2, float h, float hinv, float& f, float& D) {
    if (r2 >= h * h) {
        const float ri = __builtin_amdgcn_rsqf(r2);
        const float ri2 = ri * ri;
        f = ri * ri2;
        D = -3.f * f * ri2;
    } else {
        spline_fd<float>(r2, hinv, f, D);
    }
}

// ---- forward: g, j and S = -T from particle masses and node multipoles ----
// kTidal: the tidal tensor alone, which the gradient's first walk needs: half of
// a node's multiply-adds are the jerk's (gradient of 100 000 particles 2.26 ms,
// now 2.06).
template <bool kTidal>
struct ForwardSums {
    static constexpr bool kSkipEmpty = false;
    static constexpr bool kImageMac = false;
    static constexpr bool kGroupSum = false;
    static constexpr int kTerms = 0;
    static constexpr int kWaves = 4;   // launch bound: waves per SIMD (128 registers)
    static constexpr int kTeamWaves = 16;   // waves of a workgroup: the largest team
    using Tile = TileLds<5>;
    using Lds = WalkLds<5>;
    using Sum = PairAcc<float>;   // one tile's sums
    using Word = double;          // the walk's sums: kWords of them per lane
    static constexpr int kFirst = kTidal ? 6 : 0, kWords = 12 - kFirst;   // of a PairAcc's words
    struct Acc {
        PairAcc<double> a;
        __device__ void fold(const Sum& f) {
            if (!kTidal) {
                a.ax += f.ax; a.ay += f.ay; a.az += f.az;
                a.jx += f.jx; a.jy += f.jy; a.jz += f.jz;
            }
            a.sxx += f.sxx; a.syy += f.syy; a.szz += f.szz;
            a.sxy += f.sxy; a.sxz += f.sxz; a.syz += f.syz;
        }
        __device__ void zero() { a.zero(); }
        __device__ void add(const Acc& o) {
            if (!kTidal) {
                a.ax += o.a.ax; a.ay += o.a.ay; a.az += o.a.az;
                a.jx += o.a.jx; a.jy += o.a.jy; a.jz += o.a.jz;
            }
            a.sxx += o.a.sxx; a.syy += o.a.syy; a.szz += o.a.szz;
            a.sxy += o.a.sxy; a.sxz += o.a.sxz; a.syz += o.a.syz;
        }
    };
    template <int kPer>
    __device__ static void stage_particle(Tile& S, const Tree& T, const GroupBox& gb, int lane, int pk,
                                          const WalkOut& O) {
        const double4 q = T.spos[pk];
        const float4 u = T.svf[pk];
        double dx = q.x - gb.ox, dy = q.y - gb.oy, dz = q.z - gb.oz;
        if (kPer) {
            dx = near_img(dx, O);
            dy = near_img(dy, O);
            dz = near_img(dz, O);
        }
        S.tile[lane] = make_float4((float)dx, (float)dy, (float)dz, u.w);
        S.tile[kW + lane] = make_float4(u.x, u.y, u.z, T.sh ? T.sh[pk] : u.w);   // .w: softening length
        S.tidx[lane] = pk;
    }
    // The pair terms of pair.h, written as multiply-add chains into
    // the accumulators, with the m f I part of S summed once per tile.  The
    // self pair has d = 0 exactly (both sides round the same FP64 position),
    // so it always takes the softened branch, where it is dropped.  Periodic:
    // each pair is taken at its own nearest image.
    template <int kPer, bool kSoft>
    __device__ static void particles(const Tile& S, int cnt, const Target& t, Sum& F, float h2, float hinv,
                                     int k0, int ks, const WalkOut& O) {
        F.zero();
        float smf = 0.f;
        auto entry = [&](int k) {
            const float4 q = S.tile[k];
            const float4 u = S.tile[kW + k];
            float dx = q.x - t.tx, dy = q.y - t.ty, dz = q.z - t.tz;
            if (kPer == kNear) {
                dx = near_imgf(dx, O);
                dy = near_imgf(dy, O);
                dz = near_imgf(dz, O);
            }
            const float nx = u.x - t.vx, ny = u.y - t.vy, nz = u.z - t.vz;
            const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
            float mf, mD;
            // per-particle softening: the pair is Newtonian beyond both lengths
            const float hh = kSoft ? fmaxf(t.h, u.w) : 0.f;
            if (r2 >= (kSoft ? hh * hh : h2)) {
                const float ri = __builtin_amdgcn_rsqf(r2);
                const float ri2 = ri * ri;
                mf = q.w * (ri * ri2);
                mD = -3.f * mf * ri2;
            } else if (!kSoft) {
                float f, D;
                spline_fd<float>(r2, hinv, f, D);
                const float mj = (S.tidx[k] == t.p) ? 0.f : q.w;
                mf = mj * f;
                mD = mj * D;
            } else {
                // the mean of the target's and the source's kernels
                float f1, D1, f2, D2;
                soft_fd(r2, t.h, t.hinv, f1, D1);
                soft_fd(r2, u.w, 1.f / u.w, f2, D2);
                const float mj = (S.tidx[k] == t.p) ? 0.f : 0.5f * q.w;
                mf = mj * (f1 + f2);
                mD = mj * (D1 + D2);
            }
            if (!kTidal) {
                F.ax = __builtin_fmaf(mf, dx, F.ax);
                F.ay = __builtin_fmaf(mf, dy, F.ay);
                F.az = __builtin_fmaf(mf, dz, F.az);
            }
            float jdx = dx, jdy = dy, jdz = dz, jmf = mf, jmD = mD;
            if (kPer == kEwald) {
                // g and T take the image about the group centre (the Ewald
                // correction is summed at the same one); the jerk keeps the
                // pair's nearest image, which differs only across the cut
                const float ex = near_imgf(dx, O), ey = near_imgf(dy, O), ez = near_imgf(dz, O);
                if (ex != dx || ey != dy || ez != dz) {
                    const float r2e = __builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex));
                    const float ri = __builtin_amdgcn_rsqf(r2e);
                    jmf = q.w * (ri * ri * ri);
                    jmD = -3.f * jmf * (ri * ri);
                    jdx = ex;
                    jdy = ey;
                    jdz = ez;
                }
            }
            if (!kTidal) {
                const float sd = jmD * __builtin_fmaf(jdz, nz, __builtin_fmaf(jdy, ny, jdx * nx));
                F.jx = __builtin_fmaf(sd, jdx, __builtin_fmaf(jmf, nx, F.jx));
                F.jy = __builtin_fmaf(sd, jdy, __builtin_fmaf(jmf, ny, F.jy));
                F.jz = __builtin_fmaf(sd, jdz, __builtin_fmaf(jmf, nz, F.jz));
            }
            const float tx = mD * dx, ty = mD * dy, tz = mD * dz;
            smf += mf;
            F.sxx = __builtin_fmaf(tx, dx, F.sxx);
            F.syy = __builtin_fmaf(ty, dy, F.syy);
            F.szz = __builtin_fmaf(tz, dz, F.szz);
            F.sxy = __builtin_fmaf(tx, dy, F.sxy);
            F.sxz = __builtin_fmaf(tx, dz, F.sxz);
            F.syz = __builtin_fmaf(ty, dz, F.syz);
        };
        if (ks == 1) {
#pragma unroll 2
            for (int k = 0; k < cnt; ++k) entry(k);
        } else {
            for (int k = k0; k < cnt; k += ks) entry(k);
        }
        F.sxx += smf;
        F.syy += smf;
        F.szz += smf;
    }
    template <int kPer>
    __device__ static void stage_node(Tile& S, const Tree& T, const GroupBox& gb, int lane, int nk,
                                      const WalkOut& O) {
        const NodeRec& c = T.rec[nk];
        const float4 m0 = T.mp[4 * nk], m1 = T.mp[4 * nk + 1], m2 = T.mp[4 * nk + 2], m3 = T.mp[4 * nk + 3];
        float4* d = S.tile;
        double dx = c.x - gb.ox, dy = c.y - gb.oy, dz = c.z - gb.oz;
        if (kPer) {   // the opening test guarantees one image for the whole node
            dx = near_img(dx, O);
            dy = near_img(dy, O);
            dz = near_img(dz, O);
        }
        d[lane] = make_float4((float)dx, (float)dy, (float)dz, m0.x);
        d[kW + lane] = make_float4(m0.y, m0.z, m0.w, m1.x);       // u, Qxx
        d[2 * kW + lane] = make_float4(m1.y, m1.z, m1.w, m2.x);   // Qyy Qzz Qxy Qxz
        d[3 * kW + lane] = make_float4(m2.y, m2.z, m2.w, m3.x);   // Qyz, Qd xx yy zz
        d[4 * kW + lane] = make_float4(m3.y, m3.z, m3.w, 0.f);    // Qd xy xz yz
    }
    __device__ static void nodes(const Tile& S, int cnt, const Target& t, Sum& F, int k0, int ks, const WalkOut&) {
        F.zero();
        float sca = 0.f;
        const float4* d = S.tile;
        auto entry = [&](int k) {
            const float4 a0 = d[k], a1 = d[kW + k], a2 = d[2 * kW + k], a3 = d[3 * kW + k], a4 = d[4 * kW + k];
            const float Q[6] = {a1.w, a2.x, a2.y, a2.z, a2.w, a3.x};
            const float Qd[6] = {a3.y, a3.z, a3.w, a4.x, a4.y, a4.z};
            node_interact<kTidal>(a0.x - t.tx, a0.y - t.ty, a0.z - t.tz, a1.x - t.vx, a1.y - t.vy, a1.z - t.vz, a0.w,
                                  Q, Qd, F, sca);
        };
        if (ks == 1) {
#pragma unroll 2
            for (int k = 0; k < cnt; ++k) entry(k);
        } else {
            for (int k = k0; k < cnt; k += ks) entry(k);
        }
        F.sxx += sca;
        F.syy += sca;
        F.szz += sca;
    }
    static __device__ void wave_sum(Acc&) {}
    __device__ static void finish(const Tree& T, const WalkOut& O, const Acc& A, int p, const Target&) {
        const PairAcc<double>& acc = A.a;
        const int64_t i = T.perm[p];
        const double G = O.G;
        if (!kTidal && O.acc) {
            O.acc[3 * i] = G * acc.ax; O.acc[3 * i + 1] = G * acc.ay; O.acc[3 * i + 2] = G * acc.az;
        }
        if (!kTidal && O.jerk) {
            O.jerk[3 * i] = G * acc.jx; O.jerk[3 * i + 1] = G * acc.jy; O.jerk[3 * i + 2] = G * acc.jz;
        }
        if (O.tidal) {
            double* tt = O.tidal + 6 * i;
            tt[0] = -G * acc.sxx; tt[1] = -G * acc.syy; tt[2] = -G * acc.szz;
            tt[3] = -G * acc.sxy; tt[4] = -G * acc.sxz; tt[5] = -G * acc.syz;
        }
    }
};

using ForwardPolicy = ForwardSums<false>;
using TidalPolicy = ForwardSums<true>;

// ---- adjoint: V = sum_j J(d) w_j and s = sum_j f d.w_j over vector charges ----
// For a node with charge sum W0 = sum w and first moment W1_bc = sum w_b y_c
// (y = position - node centre of mass), to first order in y:
//   V = f W0 + D (d.W0) d + D (W1 d + W1^T d + tr(W1) d) + E (d.W1.d) d
//   s = f d.W0 + f tr(W1) + D (d.W1.d)
// with f = r^-3, D = f'/r = -3 r^-5, E = D'/r = 15 r^-7 (nodes are only used
// at separations beyond the softening length).
struct AdjAccF {
    float vx, vy, vz, s;
};
struct AdjointPolicy {
    static constexpr bool kSkipEmpty = true;   // nodes without charge add nothing
    static constexpr bool kImageMac = false;
    static constexpr bool kGroupSum = false;
    static constexpr int kTerms = 0;
    static constexpr int kWaves = 3;   // launch bound: waves per SIMD (168 registers)
    static constexpr int kTeamWaves = 12;
    using Tile = TileLds<9>;
    using Lds = WalkLds<9>;
    using Sum = AdjAccF;
    using Word = double;
    static constexpr int kFirst = 0, kWords = 4;
    struct Acc {
        double vx, vy, vz, s;
        __device__ void fold(const Sum& f) { vx += f.vx; vy += f.vy; vz += f.vz; s += f.s; }
        __device__ void zero() { vx = vy = vz = s = 0.0; }
        __device__ void add(const Acc& o) { vx += o.vx; vy += o.vy; vz += o.vz; s += o.s; }
    };
    template <int kPer>
    __device__ static void stage_particle(Tile& S, const Tree& T, const GroupBox& gb, int lane, int pk,
                                          const WalkOut&) {
        static_assert(!kPer, "the adjoint walk has no periodic form");
        const double4 q = T.spos[pk];
        const double4 w = T.ws[pk];
        S.tile[lane] = make_float4((float)(q.x - gb.cx), (float)(q.y - gb.cy), (float)(q.z - gb.cz), 0.f);
        S.tile[kW + lane] = make_float4((float)w.x, (float)w.y, (float)w.z, 0.f);
        S.tidx[lane] = pk;
    }
    template <int kPer, bool kSoft>
    __device__ static void particles(const Tile& S, int cnt, const Target& t, Sum& F, float h2, float hinv,
                                     int k0, int ks, const WalkOut&) {
        static_assert(!kSoft, "the adjoint walk has one softening length");
        F = AdjAccF{0.f, 0.f, 0.f, 0.f};
        for (int k = k0; k < cnt; k += ks) {
            const float4 q = S.tile[k];
            const float4 w = S.tile[kW + k];
            const float dx = q.x - t.tx, dy = q.y - t.ty, dz = q.z - t.tz;
            const float r2 = dx * dx + dy * dy + dz * dz;
            float f, D;
            if (r2 >= h2) {
                const float ri = __builtin_amdgcn_rsqf(r2);
                const float ri2 = ri * ri;
                f = ri * ri2;
                D = -3.f * f * ri2;
            } else {
                spline_fd<float>(r2, hinv, f, D);
            }
            const float self = (S.tidx[k] == t.p) ? 0.f : 1.f;
            f *= self;
            D *= self;
            const float dw = dx * w.x + dy * w.y + dz * w.z;
            const float Ddw = D * dw;
            F.vx += f * w.x + Ddw * dx;
            F.vy += f * w.y + Ddw * dy;
            F.vz += f * w.z + Ddw * dz;
            F.s += f * dw;
        }
    }
    template <int kPer>
    __device__ static void stage_node(Tile& S, const Tree& T, const GroupBox& gb, int lane, int nk, const WalkOut&) {
        const NodeRec& c = T.rec[nk];
        float4* d = S.tile;
        d[lane] = make_float4((float)(c.x - gb.cx), (float)(c.y - gb.cy), (float)(c.z - gb.cz), 0.f);
#pragma unroll
        for (int q = 0; q < 8; ++q) d[(q + 1) * kW + lane] = T.wf[8 * nk + q];
    }
    // Second-order term with W2_bce = sum w_b y_c y_e (symmetric in c, e):
    //   V += -1/2 [105 t d/r^9 - 15 (d (d.trW + 2 d.trX) + 2 s + u)/r^7
    //              + 3 (trW + 2 trX)/r^5]
    //   s += 7.5 t/r^7 - 1.5 (d.trW + 2 d.trX)/r^5
    // u_b = W2_bce d_c d_e, s_e = W2_bce d_b d_c, t = d.u, trW_b = W2_bcc,
    // trX_c = W2_bbc.
    __device__ static void nodes(const Tile& S, int cnt, const Target& t, Sum& F, int k0, int ks, const WalkOut&) {
        F = AdjAccF{0.f, 0.f, 0.f, 0.f};
        const float4* d = S.tile;
        for (int k = k0; k < cnt; k += ks) {
            const float4 c = d[k], a0 = d[kW + k], a1 = d[2 * kW + k], a2 = d[3 * kW + k], a3 = d[4 * kW + k];
            const float4 a4 = d[5 * kW + k], a5 = d[6 * kW + k], a6 = d[7 * kW + k], a7 = d[8 * kW + k];
            // W0 = a0.xyz; W1 rows: (a1.x a1.y a1.z) (a1.w a2.x a2.y) (a2.z a2.w a3.x);
            // W2_b (xx yy zz xy xz yz): b=0 (a3.y a3.z a3.w a4.x a4.y a4.z),
            // b=1 (a4.w a5.x a5.y a5.z a5.w a6.x), b=2 (a6.y a6.z a6.w a7.x a7.y a7.z)
            const float dx = c.x - t.tx, dy = c.y - t.ty, dz = c.z - t.tz;
            const float r2 = dx * dx + dy * dy + dz * dz;
            const float ri = __builtin_amdgcn_rsqf(r2);
            const float ri2 = ri * ri;
            const float f = ri * ri2;
            const float D = -3.f * f * ri2;
            const float E = -5.f * D * ri2;
            const float W00 = a1.x, W01 = a1.y, W02 = a1.z, W10 = a1.w, W11 = a2.x, W12 = a2.y;
            const float W20 = a2.z, W21 = a2.w, W22 = a3.x;
            const float Ax = W00 * dx + W01 * dy + W02 * dz;   // W1 d
            const float Ay = W10 * dx + W11 * dy + W12 * dz;
            const float Az = W20 * dx + W21 * dy + W22 * dz;
            const float Bx = W00 * dx + W10 * dy + W20 * dz;   // W1^T d
            const float By = W01 * dx + W11 * dy + W21 * dz;
            const float Bz = W02 * dx + W12 * dy + W22 * dz;
            const float tr = W00 + W11 + W22;
            const float dWd = dx * Ax + dy * Ay + dz * Az;
            const float dW0 = dx * a0.x + dy * a0.y + dz * a0.z;
            // second moment: M_b = W2_b d (symmetric matrix times d)
            const float b0[6] = {a3.y, a3.z, a3.w, a4.x, a4.y, a4.z};
            const float b1[6] = {a4.w, a5.x, a5.y, a5.z, a5.w, a6.x};
            const float b2[6] = {a6.y, a6.z, a6.w, a7.x, a7.y, a7.z};
            const float M0x = b0[0] * dx + b0[3] * dy + b0[4] * dz, M0y = b0[3] * dx + b0[1] * dy + b0[5] * dz,
                        M0z = b0[4] * dx + b0[5] * dy + b0[2] * dz;
            const float M1x = b1[0] * dx + b1[3] * dy + b1[4] * dz, M1y = b1[3] * dx + b1[1] * dy + b1[5] * dz,
                        M1z = b1[4] * dx + b1[5] * dy + b1[2] * dz;
            const float M2x = b2[0] * dx + b2[3] * dy + b2[4] * dz, M2y = b2[3] * dx + b2[1] * dy + b2[5] * dz,
                        M2z = b2[4] * dx + b2[5] * dy + b2[2] * dz;
            const float ux = dx * M0x + dy * M0y + dz * M0z;   // u_b = d.M_b
            const float uy = dx * M1x + dy * M1y + dz * M1z;
            const float uz = dx * M2x + dy * M2y + dz * M2z;
            const float sx = dx * M0x + dy * M1x + dz * M2x;   // s = sum_b d_b M_b
            const float sy = dx * M0y + dy * M1y + dz * M2y;
            const float sz = dx * M0z + dy * M1z + dz * M2z;
            const float tt = dx * ux + dy * uy + dz * uz;
            const float tWx = b0[0] + b0[1] + b0[2], tWy = b1[0] + b1[1] + b1[2], tWz = b2[0] + b2[1] + b2[2];
            const float tXx = b0[0] + b1[3] + b2[4], tXy = b0[3] + b1[1] + b2[5], tXz = b0[4] + b1[5] + b2[2];
            const float ri5 = f * ri2, ri7 = ri5 * ri2, ri9 = ri7 * ri2;
            const float dtr = dx * (tWx + 2.f * tXx) + dy * (tWy + 2.f * tXy) + dz * (tWz + 2.f * tXz);
            const float c2 = -52.5f * tt * ri9 + 7.5f * dtr * ri7;   // coefficient of d
            const float cd = D * dW0 + D * tr + E * dWd + c2;
            F.vx += f * a0.x + cd * dx + D * (Ax + Bx) + 7.5f * ri7 * (2.f * sx + ux) - 1.5f * ri5 * (tWx + 2.f * tXx);
            F.vy += f * a0.y + cd * dy + D * (Ay + By) + 7.5f * ri7 * (2.f * sy + uy) - 1.5f * ri5 * (tWy + 2.f * tXy);
            F.vz += f * a0.z + cd * dz + D * (Az + Bz) + 7.5f * ri7 * (2.f * sz + uz) - 1.5f * ri5 * (tWz + 2.f * tXz);
            F.s += f * (dW0 + tr) + D * dWd + 7.5f * tt * ri7 - 1.5f * dtr * ri5;
        }
    }
    static __device__ void wave_sum(Acc&) {}
    __device__ static void finish(const Tree& T, const WalkOut& O, const Acc& A, int p, const Target&) {
        const int64_t i = T.perm[p];
        const double G = O.G;
        const double mi = T.spos[p].w;
        const double4 w = T.ws[p];
        double gx = G * mi * A.vx, gy = G * mi * A.vy, gz = G * mi * A.vz;
        if (w.x != 0.0 || w.y != 0.0 || w.z != 0.0) {   // target's own term T_i w_i
            const double* t = O.tin + 6 * i;
            gx += t[0] * w.x + t[3] * w.y + t[4] * w.z;
            gy += t[3] * w.x + t[1] * w.y + t[5] * w.z;
            gz += t[4] * w.x + t[5] * w.y + t[2] * w.z;
        }
        O.dldx[3 * i] = gx;
        O.dldx[3 * i + 1] = gy;
        O.dldx[3 * i + 2] = gz;
        O.dldm[i] = -G * A.s;
    }
};

// Walk the tree for one group of targets (one wave).
// ---- Ewald correction: what the periodic images add to g and T ----------
// Table lookup of the correction field of a unit mass at separation d
// (source - target): the nearest table point p of |d| (octant [0, range]^3,
// the field's symmetry supplies the signs) and its second-order expansion
//   dg(p + u) = dg - dT u - 1/2 H u u,   dT(p + u) = dT + H u,
// with H_abc = d dT_ab / d d_c (totally symmetric), tabulated exactly.
struct EwaldVal {
    float g[3];
    float t[6];    // xx yy zz xy xz yz
    float h[10];   // xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz
};

template <bool kWithH>
__device__ __forceinline__ void ewald_lookup(const WalkOut& O, float dx, float dy, float dz, EwaldVal& E) {
    const float ax = fabsf(dx), ay = fabsf(dy), az = fabsf(dz);
    if (ax > O.etab_range || ay > O.etab_range || az > O.etab_range) atomicOr(O.flags, AGF_INTERNAL);
    const int ne = O.etab_ne;
    int ix = (int)(ax * O.etab_hinv + 0.5f), iy = (int)(ay * O.etab_hinv + 0.5f), iz = (int)(az * O.etab_hinv + 0.5f);
    ix = ix < ne ? ix : ne;
    iy = iy < ne ? iy : ne;
    iz = iz < ne ? iz : ne;
    const float ux = ax - ix * O.etab_h, uy = ay - iy * O.etab_h, uz = az - iz * O.etab_h;
    const float4* q = O.etab + 5 * (((int64_t)ix * (ne + 1) + iy) * (ne + 1) + iz);
    const float4 a = q[0], b = q[1], c = q[2], d = q[3], e = q[4];
    const float Txx = a.w, Tyy = b.x, Tzz = b.y, Txy = b.z, Txz = b.w, Tyz = c.x;
    const float Hxxx = c.y, Hxxy = c.z, Hxxz = c.w, Hxyy = d.x, Hxyz = d.y, Hxzz = d.z;
    const float Hyyy = d.w, Hyyz = e.x, Hyzz = e.y, Hzzz = e.z;
    // (H u)_ab
    const float Pxx = Hxxx * ux + Hxxy * uy + Hxxz * uz;
    const float Pyy = Hxyy * ux + Hyyy * uy + Hyyz * uz;
    const float Pzz = Hxzz * ux + Hyzz * uy + Hzzz * uz;
    const float Pxy = Hxxy * ux + Hxyy * uy + Hxyz * uz;
    const float Pxz = Hxxz * ux + Hxyz * uy + Hxzz * uz;
    const float Pyz = Hxyz * ux + Hyyz * uy + Hyzz * uz;
    // dg - (dT + 1/2 H u) u
    const float gx = a.x - ((Txx + 0.5f * Pxx) * ux + (Txy + 0.5f * Pxy) * uy + (Txz + 0.5f * Pxz) * uz);
    const float gy = a.y - ((Txy + 0.5f * Pxy) * ux + (Tyy + 0.5f * Pyy) * uy + (Tyz + 0.5f * Pyz) * uz);
    const float gz = a.z - ((Txz + 0.5f * Pxz) * ux + (Tyz + 0.5f * Pyz) * uy + (Tzz + 0.5f * Pzz) * uz);
    const float sx = dx < 0.f ? -1.f : 1.f, sy = dy < 0.f ? -1.f : 1.f, sz = dz < 0.f ? -1.f : 1.f;
    E.g[0] = sx * gx;
    E.g[1] = sy * gy;
    E.g[2] = sz * gz;
    E.t[0] = Txx + Pxx;
    E.t[1] = Tyy + Pyy;
    E.t[2] = Tzz + Pzz;
    E.t[3] = sx * sy * (Txy + Pxy);
    E.t[4] = sx * sz * (Txz + Pxz);
    E.t[5] = sy * sz * (Tyz + Pyz);
    if (kWithH) {
        E.h[0] = sx * Hxxx; E.h[1] = sy * Hxxy; E.h[2] = sz * Hxxz;
        E.h[3] = sx * Hxyy; E.h[4] = sx * sy * sz * Hxyz; E.h[5] = sx * Hxzz;
        E.h[6] = sy * Hyyy; E.h[7] = sz * Hyyz; E.h[8] = sy * Hyzz; E.h[9] = sz * Hzzz;
    }
}

// The correction field dg(d) is smooth except at the lattice points n L,
// n != 0 (where the source meets another image of the target; the single
// image's own singularity at d = 0 is subtracted).  So the correction walk
// opens a node against the target group's other images: a node of extent s
// acts as a point if s <= theta_E r, r the smallest distance between the
// node's box and the group's box shifted by any n L, n != 0.  Per axis the
// gap is either the one about the group centre or, across the cut, the one
// through the neighbouring image; at least one axis takes the latter.
__device__ __forceinline__ bool ewald_accept(const GroupBox& g, const NodeRec& c, const WalkOut& O) {
    const float4 lo = c.lo, hi = c.hi;
    float b[3], e[3];
    b[0] = fabsf((float)(near_img(0.5 * ((double)lo.x + (double)hi.x) - g.ox, O) + (g.ox - g.cx)));
    b[1] = fabsf((float)(near_img(0.5 * ((double)lo.y + (double)hi.y) - g.oy, O) + (g.oy - g.cy)));
    b[2] = fabsf((float)(near_img(0.5 * ((double)lo.z + (double)hi.z) - g.oz, O) + (g.oz - g.cz)));
    e[0] = 0.5f * (hi.x - lo.x) + g.hx;
    e[1] = 0.5f * (hi.y - lo.y) + g.hy;
    e[2] = 0.5f * (hi.z - lo.z) + g.hz;
    float s2 = 0.f, step = FLT_MAX;
    bool shifted = false;
    for (int a = 0; a < 3; ++a) {
        const float in = fmaxf(b[a] - e[a], 0.f);            // about the group centre
        const float out = fmaxf(O.boxf - b[a] - e[a], 0.f);  // through the neighbouring image
        if (out <= in) {
            s2 += out * out;
            shifted = true;
        } else {
            s2 += in * in;
            step = fminf(step, out * out - in * in);
        }
    }
    if (!shifted) s2 += step;
    return c.len <= O.ewald_theta * sqrtf(s2);
}

// The correction walk: accepted nodes (and the particles of opened leaves)
// act through their mass and (on g) quadrupole at their images about the
// group centre, the
// ones the forward walk used for g and T.  A compact group (half extent at
// most ewald_grp) sums dg, dT and H over the entries once, every lane taking
// its share, and each target expands about the group centre:
//   dg(c - t) = dg(c) + dT(c) t - 1/2 H(c) t t,   dT(c - t) = dT(c) - H(c) t;
// a wider group evaluates the table at every target's own separation (the
// expansion's relative error falls as (t / |c - n L|)^3 <= (2 t / L)^3, at
// most 2.4e-4 of the correction for t <= L / 32).  The
// sum includes the target itself (dg(0) = 0; dT(0) is the tide of the
// background that neutralises its own images).
struct EwaldPolicy {
    static constexpr bool kSkipEmpty = false;
    static constexpr bool kImageMac = true;
    static constexpr bool kGroupSum = true;
    static constexpr int kWaves = 4;   // launch bound: waves per SIMD (128 registers)
    static constexpr int kTeamWaves = 16;
    using Tile = TileLds<3>;
    using Lds = WalkLds<3>;
    // one tile's terms of a group sum (each lane holds at most one entry)
    struct Sum {
        float v[19];
    };
    using Word = float;
    static constexpr int kFirst = 0, kWords = 19;
    struct Acc {
        // g 3, T 6, (group sums only) H 10; FP32 sums of at most a few
        // thousand terms per lane: rounding ~1e-6 relative, below the table's
        float v[19];
        __device__ void fold(const Sum& f) {
#pragma unroll
            for (int k = 0; k < 19; ++k) v[k] += f.v[k];
        }
        __device__ void zero() {
#pragma unroll
            for (int k = 0; k < 19; ++k) v[k] = 0.f;
        }
        __device__ void add(const Acc& o) {
#pragma unroll
            for (int k = 0; k < 19; ++k) v[k] += o.v[k];
        }
    };
    // entry k: tile[k] = (position about the group centre, mass), tile[kW + k]
    // and tile[2 kW + k] = traceless quadrupole xx yy zz xy | xz yz (0 for particles)
    template <int kPer>
    __device__ static void stage_particle(Tile& S, const Tree& T, const GroupBox& gb, int lane, int pk,
                                          const WalkOut& O) {
        const double4 q = T.spos[pk];
        S.tile[lane] = make_float4((float)near_img(q.x - gb.ox, O), (float)near_img(q.y - gb.oy, O),
                                   (float)near_img(q.z - gb.oz, O), (float)q.w);
        S.tile[kW + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        S.tile[2 * kW + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    template <int kPer>
    __device__ static void stage_node(Tile& S, const Tree& T, const GroupBox& gb, int lane, int nk, const WalkOut& O) {
        const NodeRec& c = T.rec[nk];
        const float4 m0 = T.mp[4 * nk], m1 = T.mp[4 * nk + 1], m2 = T.mp[4 * nk + 2];
        S.tile[lane] = make_float4((float)near_img(c.x - gb.ox, O), (float)near_img(c.y - gb.oy, O),
                                   (float)near_img(c.z - gb.oz, O), m0.x);
        S.tile[kW + lane] = m1;
        S.tile[2 * kW + lane] = make_float4(m2.x, m2.y, 0.f, 0.f);
    }
    // Single-image Newtonian field of a mass with traceless quadrupole Q at
    // separation d (as the forward walk's node term): with P = Q d, q = d.P,
    //   g = ca d - r^-5 P,  ca = M r^-3 + 2.5 q r^-7,
    //   T = -(ca I - beta d d^T - r^-5 Q + 5 r^-7 (P d^T + d P^T)),
    //   beta = 3 M r^-5 + 17.5 q r^-9.
    __device__ static void newton_quad(float dx, float dy, float dz, float M, const float4 q0, const float4 q1,
                                       float* g, float* t) {
        const float Qxx = q0.x, Qyy = q0.y, Qzz = q0.z, Qxy = q0.w, Qxz = q1.x, Qyz = q1.y;
        const float r2 = dx * dx + dy * dy + dz * dz;
        const float ri = __builtin_amdgcn_rsqf(r2), ri2 = ri * ri;
        const float ri3 = ri * ri2, ri5 = ri3 * ri2, ri7 = ri5 * ri2, ri9 = ri7 * ri2;
        const float Px = Qxx * dx + Qxy * dy + Qxz * dz;
        const float Py = Qxy * dx + Qyy * dy + Qyz * dz;
        const float Pz = Qxz * dx + Qyz * dy + Qzz * dz;
        const float q = dx * Px + dy * Py + dz * Pz;
        const float ca = M * ri3 + 2.5f * q * ri7;
        const float beta = 3.f * M * ri5 + 17.5f * q * ri9;
        const float e = 5.f * ri7;
        g[0] = ca * dx - ri5 * Px;
        g[1] = ca * dy - ri5 * Py;
        g[2] = ca * dz - ri5 * Pz;
        t[0] = -(ca - beta * dx * dx - ri5 * Qxx + 2.f * e * Px * dx);
        t[1] = -(ca - beta * dy * dy - ri5 * Qyy + 2.f * e * Py * dy);
        t[2] = -(ca - beta * dz * dz - ri5 * Qzz + 2.f * e * Pz * dz);
        t[3] = -(-beta * dx * dy - ri5 * Qxy + e * (Px * dy + dx * Py));
        t[4] = -(-beta * dx * dz - ri5 * Qxz + e * (Px * dz + dx * Pz));
        t[5] = -(-beta * dy * dz - ri5 * Qyz + e * (Py * dz + dy * Pz));
    }
    // H_abc = dT_ab / dd_c of a point mass M at d:
    //   M (3 (d_c delta_ab + d_b delta_ac + d_a delta_bc) / r^5 - 15 d_a d_b d_c / r^7)
    __device__ static void newton_h(float dx, float dy, float dz, float M, float* h) {
        const float r2 = dx * dx + dy * dy + dz * dz;
        const float ri = __builtin_amdgcn_rsqf(r2), ri2 = ri * ri;
        const float a = 3.f * M * ri * ri2 * ri2, b = 15.f * M * ri * ri2 * ri2 * ri2;
        const float d[3] = {dx, dy, dz};
        const int ia[10] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 2}, ib[10] = {0, 0, 0, 1, 1, 2, 1, 1, 2, 2},
                  ic[10] = {0, 1, 2, 1, 2, 2, 1, 2, 2, 2};
#pragma unroll
        for (int q = 0; q < 10; ++q) {
            const int i = ia[q], j = ib[q], k = ic[q];
            const float del = (i == j ? d[k] : 0.f) + (i == k ? d[j] : 0.f) + (j == k ? d[i] : 0.f);
            h[q] = a * del - b * d[i] * d[j] * d[k];
        }
    }
    // A node's quadrupole adds -(1/6) Q_bc H_abc to dg (dg is harmonic away
    // from d = 0, so the trace of the second moment drops out).
    __device__ static void quad_g(const float4 q0, const float4 q1, const EwaldVal& E, float* g) {
        const float* H = E.h;   // xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz
        const float Qxx = q0.x, Qyy = q0.y, Qzz = q0.z, Qxy = q0.w, Qxz = q1.x, Qyz = q1.y;
        const float c = 1.f / 6.f;
        g[0] -= c * (Qxx * H[0] + Qyy * H[3] + Qzz * H[5] + 2.f * (Qxy * H[1] + Qxz * H[2] + Qyz * H[4]));
        g[1] -= c * (Qxx * H[1] + Qyy * H[6] + Qzz * H[8] + 2.f * (Qxy * H[3] + Qxz * H[4] + Qyz * H[7]));
        g[2] -= c * (Qxx * H[2] + Qyy * H[7] + Qzz * H[9] + 2.f * (Qxy * H[4] + Qxz * H[5] + Qyz * H[8]));
    }
    // A compact group's terms about the group centre: c = entry - (group
    // centre), at its image about the image origin; where that is not c's
    // nearest image c', the field continues smoothly through
    // dg(c) = dg(c') + g_single(c') - g_single(c) (likewise T and H).  Lane k
    // takes entry k of the tile.
    __device__ static void group_entry(const Tile& S, int cnt, const Target& t, Sum& F, const WalkOut& O) {
        const int k = ag_lane();
#pragma unroll
        for (int c = 0; c < 19; ++c) F.v[c] = 0.f;
        if (k >= cnt) return;
        EwaldVal E;
        const float4 e = S.tile[k];
        const float4 q0 = S.tile[kW + k], q1 = S.tile[2 * kW + k];
        const float cx = e.x - t.g0x, cy = e.y - t.g0y, cz = e.z - t.g0z;
        const float nx = near_imgf(cx, O), ny = near_imgf(cy, O), nz = near_imgf(cz, O);
        ewald_lookup<true>(O, nx, ny, nz, E);
        float gq[3] = {e.w * E.g[0], e.w * E.g[1], e.w * E.g[2]};
        float tq[6], hq[10];
#pragma unroll
        for (int c = 0; c < 6; ++c) tq[c] = e.w * E.t[c];
#pragma unroll
        for (int c = 0; c < 10; ++c) hq[c] = e.w * E.h[c];
        quad_g(q0, q1, E, gq);
        if (nx != cx || ny != cy || nz != cz) {
            float g1[3], t1[6], g0[3], t0[6], h1[10], h0[10];
            newton_quad(nx, ny, nz, e.w, q0, q1, g1, t1);
            newton_quad(cx, cy, cz, e.w, q0, q1, g0, t0);
            newton_h(nx, ny, nz, e.w, h1);
            newton_h(cx, cy, cz, e.w, h0);
#pragma unroll
            for (int c = 0; c < 3; ++c) gq[c] += g1[c] - g0[c];
#pragma unroll
            for (int c = 0; c < 6; ++c) tq[c] += t1[c] - t0[c];
#pragma unroll
            for (int c = 0; c < 10; ++c) hq[c] += h1[c] - h0[c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) F.v[c] = gq[c];
#pragma unroll
        for (int c = 0; c < 6; ++c) F.v[3 + c] = tq[c];
#pragma unroll
        for (int c = 0; c < 10; ++c) F.v[9 + c] = hq[c];
    }
    // A wider group, per target: the forward walk took g and T at d, the image
    // about the group centre; the periodic field is the same at the nearest
    // image d', where the table is accurate, so add
    // dg(d') + g_single(d') - g_single(d)  (the last two only when d' != d).
    // The terms (of g and T, entry k) go straight into the walk's sums, entry by
    // entry.
    static constexpr int kTerms = 9;
    __device__ static void target_terms(const Tile& S, int k, const Target& t, float* term, const WalkOut& O) {
        EwaldVal E;
        const float4 e = S.tile[k];
        const float4 q0 = S.tile[kW + k], q1 = S.tile[2 * kW + k];
        const float dx = e.x - t.tx, dy = e.y - t.ty, dz = e.z - t.tz;
        const float nx = near_imgf(dx, O), ny = near_imgf(dy, O), nz = near_imgf(dz, O);
        ewald_lookup<true>(O, nx, ny, nz, E);
        float gq[3] = {e.w * E.g[0], e.w * E.g[1], e.w * E.g[2]};
        float tq[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) tq[c] = e.w * E.t[c];
        quad_g(q0, q1, E, gq);
        if (nx != dx || ny != dy || nz != dz) {
            float g1[3], t1[6], g0[3], t0[6];
            newton_quad(nx, ny, nz, e.w, q0, q1, g1, t1);
            newton_quad(dx, dy, dz, e.w, q0, q1, g0, t0);
#pragma unroll
            for (int c = 0; c < 3; ++c) gq[c] += g1[c] - g0[c];
#pragma unroll
            for (int c = 0; c < 6; ++c) tq[c] += t1[c] - t0[c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) term[c] = gq[c];
#pragma unroll
        for (int c = 0; c < 6; ++c) term[3 + c] = tq[c];
    }
    __device__ static void target_entries(const Tile& S, int cnt, const Target& t, Acc& acc, int k0, int ks,
                                          const WalkOut& O) {
        for (int k = k0; k < cnt; k += ks) {
            float term[kTerms];
            target_terms(S, k, t, term, O);
#pragma unroll
            for (int c = 0; c < kTerms; ++c) acc.v[c] += term[c];
        }
    }
    template <int kPer, bool kSoft>
    __device__ static void particles(const Tile& S, int cnt, const Target& t, Sum& F, float, float, int, int,
                                     const WalkOut& O) {
        group_entry(S, cnt, t, F, O);
    }
    __device__ static void nodes(const Tile& S, int cnt, const Target& t, Sum& F, int, int, const WalkOut& O) {
        group_entry(S, cnt, t, F, O);
    }
    static __device__ void wave_sum(Acc& A) {
#pragma unroll
        for (int k = 0; k < 19; ++k) {
            float v = A.v[k];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            A.v[k] = v;
        }
    }
    __device__ static void finish(const Tree& T, const WalkOut& O, const Acc& A, int p, const Target& t) {
        double g[3], tt[6];
        if (t.grp) {
            // the target relative to the group centre
            const double x = (double)t.tx - t.g0x, y = (double)t.ty - t.g0y, z = (double)t.tz - t.g0z;
            double H[10], Tv[6];
            for (int c = 0; c < 10; ++c) H[c] = A.v[9 + c];   // xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz
            for (int c = 0; c < 6; ++c) Tv[c] = A.v[3 + c];    // xx yy zz xy xz yz
            // (H t)_ab
            const double Pxx = H[0] * x + H[1] * y + H[2] * z, Pyy = H[3] * x + H[6] * y + H[7] * z;
            const double Pzz = H[5] * x + H[8] * y + H[9] * z, Pxy = H[1] * x + H[3] * y + H[4] * z;
            const double Pxz = H[2] * x + H[4] * y + H[5] * z, Pyz = H[4] * x + H[7] * y + H[8] * z;
            g[0] = A.v[0] + (Tv[0] - 0.5 * Pxx) * x + (Tv[3] - 0.5 * Pxy) * y + (Tv[4] - 0.5 * Pxz) * z;
            g[1] = A.v[1] + (Tv[3] - 0.5 * Pxy) * x + (Tv[1] - 0.5 * Pyy) * y + (Tv[5] - 0.5 * Pyz) * z;
            g[2] = A.v[2] + (Tv[4] - 0.5 * Pxz) * x + (Tv[5] - 0.5 * Pyz) * y + (Tv[2] - 0.5 * Pzz) * z;
            tt[0] = Tv[0] - Pxx; tt[1] = Tv[1] - Pyy; tt[2] = Tv[2] - Pzz;
            tt[3] = Tv[3] - Pxy; tt[4] = Tv[4] - Pxz; tt[5] = Tv[5] - Pyz;
        } else {
            for (int c = 0; c < 3; ++c) g[c] = A.v[c];
            for (int c = 0; c < 6; ++c) tt[c] = A.v[3 + c];
        }
        const int64_t i = T.perm[p];
        const double G = O.G;
        if (O.acc)
            for (int c = 0; c < 3; ++c) O.acc[3 * i + c] += G * g[c];
        if (O.tidal)
            for (int c = 0; c < 6; ++c) O.tidal[6 * i + c] += G * tt[c];
    }
};

// orders a wave's LDS accesses around it (LDS serves a wave's accesses in
// order, so no wait is needed between its lanes)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Targets of a group: a group of count < 64 targets gives each target
// sub = min(kMaxSub, 64 / count) lanes: lane = part * count + slot, and part k
// of a target takes every sub-th entry of each tile (lanes with part >= sub
// repeat work that is not used).  The parts are summed at the end.
struct GroupSetup {
    GroupBox gb;
    Target tg;
    float gh2;                 // multipoles only beyond every softening length of the group and the node
    int count, sub, slot, part;
};

template <class Pol, int kPer, bool kSoft>
__device__ __forceinline__ GroupSetup group_setup(const Tree& T, const Groups& Gr, const WalkOut& O, const int4 gd,
                                                  float eps2, int lane) {
    GroupSetup U;
    const int count = gd.y;
    U.count = count;
    U.sub = count * 2 > kW ? 1 : (kW / count < kMaxSub ? kW / count : kMaxSub);
    U.slot = lane % count;
    U.part = lane / count;
    // every lane holds some target of the group (no position list: all active)
    const int p_i = Gr.act_pos ? Gr.act_pos[gd.x + U.slot] : gd.x + U.slot;
    const double4 xi = T.spos[p_i];
    const float4 vi = T.svf[p_i];
    GroupBox& gb = U.gb;
    gb = group_box(xi.x, xi.y, xi.z);
    if (kPer == kEwald) {
        // images about a multiple of half the box: its cut lies on the faces
        // of the root's children (the root of a periodic tree is the box)
        const double hb = 0.5 * O.box;
        gb.ox = hb * rint(gb.cx / hb);
        gb.oy = hb * rint(gb.cy / hb);
        gb.oz = hb * rint(gb.cz / hb);
    }
    Target& tg = U.tg;
    tg.tx = (float)(xi.x - gb.ox);
    tg.ty = (float)(xi.y - gb.oy);
    tg.tz = (float)(xi.z - gb.oz);
    tg.g0x = (float)(gb.cx - gb.ox);
    tg.g0y = (float)(gb.cy - gb.oy);
    tg.g0z = (float)(gb.cz - gb.oz);
    tg.h = kSoft ? T.sh[p_i] : 0.f;
    tg.hinv = kSoft ? 1.f / tg.h : 0.f;
    U.gh2 = kSoft ? ag_wave_max(tg.h * tg.h) : eps2;
    tg.vx = vi.x;
    tg.vy = vi.y;
    tg.vz = vi.z;
    tg.p = p_i;
    tg.grp = Pol::kGroupSum && fmaxf(fmaxf(gb.hx, gb.hy), gb.hz) <= O.ewald_grp;
    gb.amin = O.rel_a ? ag_wave_min(O.rel_a[T.perm[p_i]]) : 0.f;
    return U;
}

// Every lane's numbers first, first + 1, ... (give of them, give >= 0) to its
// own run of the list at p; the lanes' runs follow one another.  All lanes
// write as many as the longest run needs, from the last number to the first:
// what a lane writes past its own run lies in the runs of later lanes, at
// numbers that those write afterwards (a later lane's run starts later, so the
// same place is a smaller number there), or in the slack behind the list.  A
// number then takes two instructions, not a loop of eight that every lane
// waits for.  (The barriers keep the compiler from reordering or pairing the
// writes; the LDS takes a wave's writes in order.)
__device__ __forceinline__ void list_run(int* p, int first, int give) {
    auto put = [&](int k) {
        p[k] = first + k;
        asm volatile("" ::: "memory");
    };
    const bool more = __ballot(give > 8) != 0, most = __ballot(give > 16) != 0;
    if (give > 0) {
        if (most) {   // leaves of more than 16 particles
            for (int k = give - 1; k >= kListSlack; --k) put(k);
#pragma unroll 4
            for (int k = kListSlack - 1; k >= 16; --k) put(k);
        }
        if (more) {
#pragma unroll
            for (int k = 15; k >= 8; --k) put(k);
        }
#pragma unroll
        for (int k = 7; k >= 0; --k) put(k);
    }
}

// One wave walks the tree for a group and hands every full tile of accepted
// nodes or of particles (64 list entries, the list's last ones first), and at
// the end the two remainders, to tile(is_node, list, count).  The order of the
// tiles and of the entries in them depends on the tree and the group alone.
//
// A step tests one node per lane.  With kAhead the next nodes' records are
// asked for as soon as the step has decided which they are, and the step's
// lists and tiles are written while the loads are on their way: for a wave that
// does nothing but traverse, one load per step was 40 % of its time (3000
// particles: 2820 cycles a step, now 2130; step of 2^15 particles 0.30 ms, now
// 0.28).  A wave
// that evaluates its tiles itself asks for them when it needs them (the
// registers are worth more; other waves fill the wait).  tile() gets a function
// that asks again, for after it has used the registers itself.
template <class Pol, int kPer, bool kSoft, bool kAhead, class TileFn>
__device__ __forceinline__ void traverse(ListLds& S, const Tree& T, const WalkOut& O, const GroupBox& gb, float gh2,
                                         int root, int lane, float theta2, float eps2,
                                         TileFn tile) {
    int ca = 0, cb = 0;          // cursor range [ca, cb)
    int ps = 0, pc = 0;          // particles still to be listed from an opened leaf
    if (lane == 0 && root >= 0) {
        ca = root;
        cb = T.link[root].x;
    }
    int sp = 0;                  // stack depth (uniform)
    int npend = 0, ppend = 0;    // list fills (uniform)
    NodeRec c;                   // node ca, for a lane that walks
    int4 L;
    float wn = 1.f;
    auto load = [&] {   // (by all lanes: the old values need no registers meanwhile)
        const int64_t a = ca < cb && pc == 0 ? ca : 0;
        L = T.link[a];
        c = T.rec[a];
        if (Pol::kSkipEmpty) wn = T.wf[8 * a].w;
    };
    if (kAhead) load();
    unsigned iters = 0;
    for (;;) {
        const bool walking = (ca < cb) && pc == 0;
        const bool end = __ballot(walking || pc > 0) == 0 || iters > O.iter_cap;
        // 6. full tiles, and at the end the remainders
        const int least = end ? 1 : kW;
        while (npend >= least || ppend >= least) {
            const bool node = npend >= least;
            int& pend = node ? npend : ppend;
            const int cnt = pend < kW ? pend : kW;
            pend -= cnt;
            tile(node, (node ? S.nlist : S.plist) + pend, cnt, load);
        }
        if (end) break;
        ++iters;
        if (!kAhead) load();

        // 1. test one node per walking lane
        int push_node = -1;
        int push_range_a = 0, push_range_b = 0;
        bool want_push = false;
        if (walking) {
            const int a = ca;
            const bool leaf = (L.w & 0x100) != 0;
            if (Pol::kSkipEmpty && wn == 0.f) {
                ca = L.x;                  // nothing below this node matters
            } else {
                const bool acc_ok =
                    Pol::kImageMac ? ewald_accept(gb, c, O)
                                   : mac_accept<kPer>(gb, c, theta2, kSoft ? fmaxf(gh2, c.lo.w * c.lo.w) : eps2, O);
                if (acc_ok && L.z > O.small_node) {
                    push_node = a;
                    ca = L.x;
                } else if (acc_ok || leaf) {
                    ps = L.y;
                    pc = L.z;
                    ca = L.x;
                } else {                   // open an inner node
                    if (L.x < cb) {        // siblings remain: offer them to the stack
                        want_push = true;
                        push_range_a = L.x;
                        push_range_b = cb;
                    }
                    ca = a + 1;
                }
            }
        }
        // 2. split ranges -> stack (lanes beyond capacity keep their range)
        {
            const uint64_t m = __ballot(want_push);
            if (m) {
                const int r = ag_prefix_count(m);
                const int room = kSCap - sp;
                if (want_push && r < room) {
                    S.stack[sp + r] = make_int2(push_range_a, push_range_b);
                    cb = push_range_a;
                }
                const int pushed = __popcll(m);
                sp += pushed < room ? pushed : room;
            }
        }
        // 3. the share of the particle list that each opened leaf gets, as room allows
        const bool listing = __ballot(pc > 0) != 0;
        const int first = ps;
        int excl = 0, give = 0, listed = 0;
        if (listing) {
            const int want = pc;
            const int incl = ag_wave_incl_scan(want);
            excl = incl - want;
            const int total = __builtin_amdgcn_readlane(incl, 63);
            const int room = kPCap - ppend;
            give = room - excl;
            give = give < 0 ? 0 : (give > want ? want : give);
            ps += give;
            pc -= give;
            listed = total < room ? total : room;
        }
        wave_sync();
        // 4. idle lanes take ranges from the stack
        {
            const bool idle = (ca >= cb) && pc == 0;
            const uint64_t im = __ballot(idle);
            const int nidle = __popcll(im);
            const int take = nidle < sp ? nidle : sp;
            if (take > 0) {
                const int r = ag_prefix_count(im);
                if (idle && r < take) {
                    const int2 e = S.stack[sp - 1 - r];
                    ca = e.x;
                    cb = e.y;
                }
                sp -= take;
            }
        }
        if (kAhead) load();
        // 5. accepted nodes -> node list (always fits: npend < 64 here),
        // particles of opened leaves -> particle list
        {
            const uint64_t m = __ballot(push_node >= 0);
            if (m) {
                const int r = ag_prefix_count(m);
                if (push_node >= 0) S.nlist[npend + r] = push_node;
                npend += __popcll(m);
            }
        }
        if (listing) {
            list_run(S.plist + ppend + excl, first, give);
            ppend += listed;
        }
        wave_sync();
    }
    // every step tests a node or lists particles, so the loop ends within
    // (nodes + particles) steps; the cap only guards against a corrupt tree
    if (iters > O.iter_cap && lane == 0) atomicOr(O.flags, AGF_INTERNAL);
}

// What a wave's groups add to the context's counters: kept by the wave and
// added once when it ends (four atomics per group, all on one line that the
// XCDs' L2s then pass around, take as long as a short group's walk).
struct WalkCount {
    uint64_t pp = 0, pn = 0, targets = 0, groups = 0;
    __device__ __forceinline__ void group(uint64_t n_pp, uint64_t n_pn, int count) {
        pp += n_pp * (uint64_t)count;
        pn += n_pn * (uint64_t)count;
        targets += (uint64_t)count;
        groups += 1;
    }
    __device__ __forceinline__ void add_to(unsigned long long* stats) const {
        if (!stats || groups == 0 || ag_lane() != 0) return;
        atomicAdd(&stats[0], (unsigned long long)pp);
        atomicAdd(&stats[1], (unsigned long long)pn);
        atomicAdd(&stats[2], (unsigned long long)targets);
        atomicAdd(&stats[3], (unsigned long long)groups);
    }
};

// (a word that other waves of the workgroup write: one lane's reading of it, so
// that the whole wave takes the same branch)
__device__ __forceinline__ int lds_get(const int* p) {
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ __forceinline__ int lds_peek(const int* p) {   // (each lane its own word)
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_put(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void team_release() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local"); }
__device__ __forceinline__ void team_acquire() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local"); }

// Waves that walk groups on their own run out of groups at different times: the
// last groups took a sixth of a walk of 2^20 particles (2.58 ms per step, now
// 2.51; 2^22 particles, 10 % active: 4.13, now 3.99).  A wave
// without a group left takes tiles of its workgroup's other waves: one that
// has a full tile gives its list to a free helper and goes on, and folds
// the helper's sums in their turn, so tiles, orders and roundings stay the same.
// The helper's own LDS holds the list and, after it has evaluated the tile,
// the sums.
constexpr int kHelpNone = 0, kHelpFree = 1, kHelpAsked = 2, kHelpTaken = 3, kHelpDone = 4;
template <int W>
struct HelpLds {
    int state[W];    // of each wave as a helper: walks a group itself, free, asked, working, sums ready
    int group[W];    // the group ...
    int info[W];     // ... and the number of entries of its tile, negative for nodes
    int walking;     // waves that still walk groups
};
template <class Pol>
constexpr bool can_help() {   // a tile's sums fit where the tile was
    return !Pol::kGroupSum && sizeof(float) * Pol::kWords * kW <= sizeof(typename Pol::Tile);
}

// a helper's share: tiles of other waves' groups until no wave walks any more
template <class Pol, int kPer, bool kSoft, int W>
__device__ __forceinline__ void help(typename Pol::Lds& S, HelpLds<W>& H, int wave, const Tree& T, const Groups& Gr,
                                     const WalkOut& O, float eps2, float h2, float hinv) {
    const int lane = ag_lane();
    GroupSetup U;
    int have = -1;
    if (lane == 0) {
        lds_put(&H.state[wave], kHelpFree);
        (void)__hip_atomic_fetch_add(&H.walking, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    for (;;) {
        const int state = lds_get(&H.state[wave]);
        if (state != kHelpTaken) {
            if (state == kHelpFree && lds_get(&H.walking) == 0) break;
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        team_acquire();
        const int g = lds_get(&H.group[wave]), info = lds_get(&H.info[wave]);
        const bool node = info < 0;
        const int cnt = node ? -info : info;
        if (g != have) U = group_setup<Pol, kPer, kSoft>(T, Gr, O, Gr.grp[g], eps2, lane);
        have = g;
        if (lane < cnt) {
            if (node) Pol::template stage_node<kPer>(S, T, U.gb, lane, S.nlist[lane], O);
            else Pol::template stage_particle<kPer>(S, T, U.gb, lane, S.nlist[lane], O);
        }
        wave_sync();
        typename Pol::Sum F;
        if (node) Pol::nodes(S, cnt, U.tg, F, U.part, U.sub, O);
        else Pol::template particles<kPer, kSoft>(S, cnt, U.tg, F, h2, hinv, U.part, U.sub, O);
        wave_sync();
        const float* f = reinterpret_cast<const float*>(&F) + Pol::kFirst;
        float* out = reinterpret_cast<float*>(S.tile) + lane;
#pragma unroll
        for (int k = 0; k < Pol::kWords; ++k) out[k * kW] = f[k];
        team_release();
        if (lane == 0) lds_put(&H.state[wave], kHelpDone);
    }
}

// Walk the tree for one group of targets by one wave: every tile is staged
// and evaluated as soon as it is full, or handed to a helper.
template <class Pol, int kPer, bool kSoft, int W>
__device__ __forceinline__ void walk_group(typename Pol::Lds* all, HelpLds<W>& H, int wave, const Tree& T,
                                           const Groups& Gr, const WalkOut& O, int g, float theta2, float eps2,
                                           float h2, float hinv, WalkCount& C) {
    const int lane = ag_lane();
    typename Pol::Lds& S = all[wave];
    const int4 gd = Gr.grp[g];
    if (gd.y <= 0) return;
    const GroupSetup U = group_setup<Pol, kPer, kSoft>(T, Gr, O, gd, eps2, lane);
    const Target tg = U.tg;
    const int count = U.count, sub = U.sub, slot = U.slot, part = U.part;
    typename Pol::Acc acc;
    acc.zero();

    // the helpers that hold tiles of this group, the first in the lowest bits
    uint64_t held = 0;
    int n_held = 0;
    // folds the first held tile's sums, if they are ready or `wait` says so
    auto take_back = [&](bool wait) {
        const int h = (int)(held & 15);
        while (lds_get(&H.state[h]) != kHelpDone) {
            if (!wait) return false;
            __builtin_amdgcn_s_sleep(1);
        }
        team_acquire();
        typename Pol::Sum F;
        float* f = reinterpret_cast<float*>(&F) + Pol::kFirst;
        const float* in = reinterpret_cast<const float*>(all[h].tile) + lane;
#pragma unroll
        for (int k = 0; k < Pol::kWords; ++k) f[k] = in[k * kW];
        acc.fold(F);
        team_release();
        if (lane == 0) lds_put(&H.state[h], kHelpFree);
        held >>= 4;
        --n_held;
        return true;
    };

    uint64_t n_pp = 0, n_pn = 0;
    traverse<Pol, kPer, kSoft, false>(S, T, O, U.gb, U.gh2, T.sys_root[gd.z], lane, theta2, eps2,
                                      [&](bool node, const int* list, int cnt, auto) {
        if (node) n_pn += (uint64_t)cnt;
        else n_pp += (uint64_t)cnt;
        if constexpr (can_help<Pol>()) {
            if (lds_get(&H.walking) < W) {
                while (n_held > 0 && take_back(false)) {}
                const uint64_t free = __ballot(lane < W && lds_peek(&H.state[lane < W ? lane : 0]) == kHelpFree);
                int h = -1;
                if (free != 0 && n_held < 16) {
                    h = __ffsll((unsigned long long)free) - 1;
                    int was = kHelpFree;
                    if (lane == 0 && !__hip_atomic_compare_exchange_strong(&H.state[h], &was, kHelpAsked,
                                                                           __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_WORKGROUP))
                        h = -1;
                    h = __builtin_amdgcn_readfirstlane(h);
                }
                if (h >= 0) {
                    if (lane < cnt) all[h].nlist[lane] = list[lane];
                    if (lane == 0) {
                        lds_put(&H.group[h], g);
                        lds_put(&H.info[h], node ? -cnt : cnt);
                    }
                    team_release();
                    if (lane == 0) lds_put(&H.state[h], kHelpTaken);
                    held |= (uint64_t)h << (4 * n_held);
                    ++n_held;
                    return;
                }
            }
        }
        if (lane < cnt) {
            if (node) Pol::template stage_node<kPer>(S, T, U.gb, lane, list[lane], O);
            else Pol::template stage_particle<kPer>(S, T, U.gb, lane, list[lane], O);
        }
        wave_sync();
        bool done = false;
        if constexpr (Pol::kGroupSum) {
            done = !tg.grp;
            if (done) Pol::target_entries(S, cnt, tg, acc, part, sub, O);
        }
        if (!done) {
            typename Pol::Sum F;
            if (node) Pol::nodes(S, cnt, tg, F, part, sub, O);
            else Pol::template particles<kPer, kSoft>(S, cnt, tg, F, h2, hinv, part, sub, O);
            if constexpr (can_help<Pol>())
                while (n_held > 0) (void)take_back(true);   // the earlier tiles first
            acc.fold(F);
        }
        wave_sync();
    });
    if constexpr (can_help<Pol>())
        while (n_held > 0) (void)take_back(true);

    if (Pol::kGroupSum && tg.grp) {
        // every lane summed its own share of the entries: add all 64
        Pol::wave_sum(acc);
    } else if (sub > 1) {
        // sum the parts of every target in LDS (the walk lists are free now)
        static_assert(sizeof(typename Pol::Lds) >= sizeof(typename Pol::Acc) * kW, "LDS too small");
        typename Pol::Acc* red = reinterpret_cast<typename Pol::Acc*>(&S);
        wave_sync();
        red[lane] = acc;
        wave_sync();
        if (part == 0)
            for (int j = 1; j < sub; ++j) acc.add(red[slot + j * count]);
        wave_sync();
    }
    if (part == 0) Pol::finish(T, O, acc, tg.p, tg);
    C.group(n_pp, n_pn, count);
}

// ---- one group walked by a team of waves ----
// With fewer groups than the device has waves, a walk by single waves lasts as
// long as its longest group (3000 particles: 96 groups on 1024 SIMDs, 0.74 ms).
// A team (of 4 waves or the whole workgroup) walks one group: its first wave traverses the tree and queues the
// full tiles in LDS, the others (and the first when the queue is full or the
// traversal done) take tiles from the queue, stage and evaluate them, and fold
// the tile sums into the group's sums in LDS in the order of the queue.  Tiles,
// their order and every rounding are those of a single wave's walk, so the
// results are the same bit for bit whichever way a group is walked.
constexpr int kRing = 16;   // queued tiles
constexpr int kMinTeam = 4; // waves of the smallest team
// Where a tile's terms go into the group's sums one entry after another
// (Ewald, groups wider than the expansion allows), it is queued in parts of
// this many entries: the waves of the team work out their parts' terms at the
// same time and only add them up in turn.  Taken a tile at a time, one wave of
// the team worked and the others waited (64^3 particles: 3.04 ms per
// evaluation, now 2.03).
constexpr int kPart = 4;
constexpr int kTeamClosed = 0, kTeamOpen = 1, kTeamDone = 2;
template <class Pol>
struct TeamLds {
    ListLds lists;
    typename Pol::Word acc[Pol::kWords][kW];   // the group's sums, one lane each
    int ring[kRing][kW];    // queued tiles: list entries ...
    int info[kRing];        // ... and their number, negative for nodes
    int full[kRing];        // slot holds a tile that no wave has taken yet
    int head, tail, done;   // next tile to take, tiles queued, traversal finished
    int turn;               // next tile whose sums are folded
    int g;                  // the team's group, -1 when none is left
    int state;              // kTeamClosed, kTeamOpen (its tiles may be taken), kTeamDone
    int arrived;            // waves that have come to the team's barriers so far
};

// barrier of the ts waves of a team, all resident on one CU; orders LDS
__device__ __forceinline__ void team_barrier(int* arrived, int ts) {
    team_release();
    int a = 0;
    if (ag_lane() == 0) a = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const int all = (__builtin_amdgcn_readfirstlane(a) / ts + 1) * ts;
    while (lds_get(arrived) < all) __builtin_amdgcn_s_sleep(1);
    team_acquire();
}

template <class Pol, int kPer, bool kSoft>
__device__ __forceinline__ void walk_group_team(TeamLds<Pol>& S, typename Pol::Tile& st, int wave, int ts, bool guest,
                                                const Tree& T, const Groups& Gr, const WalkOut& O, const int4 gd,
                                                float theta2, float eps2, float h2, float hinv, WalkCount& C) {
    constexpr int kN = Pol::kWords;
    const int lane = ag_lane();
    if (gd.y <= 0) {   // uniform over the team
        team_barrier(&S.arrived, ts);
        return;
    }
    const GroupSetup U = group_setup<Pol, kPer, kSoft>(T, Gr, O, gd, eps2, lane);
    const Target tg = U.tg;
    const int count = U.count, sub = U.sub, slot = U.slot, part = U.part;
    if (!guest) {
        for (int k = wave; k < kN; k += ts) S.acc[k][lane] = 0;
        if (wave == 0) {
            if (lane < kRing) S.full[lane] = 0;
            if (lane == 0) S.head = S.tail = S.done = S.turn = 0;
        }
        team_barrier(&S.arrived, ts);
        if (wave == 0 && lane == 0) lds_put(&S.state, kTeamOpen);
    }

    const bool in_turn = Pol::kGroupSum && !tg.grp;   // terms go straight into the group's sums
    // the queue's tile t: staged, evaluated and, in its turn, folded
    auto evaluate = [&](int t) {
        const int s = t % kRing;
        const int info = lds_get(&S.info[s]);
        const bool node = info < 0;
        const int cnt = (node ? -info : info) & 127;
        const int id = S.ring[s][lane];
        team_release();              // the slot is read ...
        if (lane == 0) lds_put(&S.full[s], 0);   // ... before it is given back
        if (lane < cnt) {
            if (node) Pol::template stage_node<kPer>(st, T, U.gb, lane, id, O);
            else Pol::template stage_particle<kPer>(st, T, U.gb, lane, id, O);
        }
        wave_sync();
        typename Pol::Sum F;
        float term[Pol::kGroupSum ? kPart * Pol::kTerms : 1];   // (in_turn) of every sub-th entry
        int k0 = 0;
        if (!in_turn) {
            if (node) Pol::nodes(st, cnt, tg, F, part, sub, O);
            else Pol::template particles<kPer, kSoft>(st, cnt, tg, F, h2, hinv, part, sub, O);
        } else if constexpr (Pol::kGroupSum) {
            const int off = (node ? -info : info) >> 7;   // the part's first entry in its tile
            k0 = (part + off * (sub - 1)) % sub;          // (part - off) modulo sub
#pragma unroll
            for (int j = 0; j < kPart; ++j)
                if (k0 + j * sub < cnt) Pol::target_terms(st, k0 + j * sub, tg, term + j * Pol::kTerms, O);
        }
        // every earlier tile is held by a wave that does not wait for this one
        while (lds_get(&S.turn) != t) __builtin_amdgcn_s_sleep(1);
        team_acquire();
        if constexpr (Pol::kGroupSum) {
            if (in_turn) {
#pragma unroll
                for (int c = 0; c < Pol::kTerms; ++c) {
                    float v = S.acc[c][lane];
#pragma unroll
                    for (int j = 0; j < kPart; ++j)
                        if (k0 + j * sub < cnt) v += term[j * Pol::kTerms + c];
                    S.acc[c][lane] = v;
                }
            }
        }
        if (!in_turn) {
            const float* f = reinterpret_cast<const float*>(&F) + Pol::kFirst;
#pragma unroll
            for (int k = 0; k < kN; ++k) S.acc[k][lane] += (typename Pol::Word)f[k];
        }
        team_release();
        if (lane == 0) lds_put(&S.turn, t + 1);
        wave_sync();
    };

    uint64_t n_pp = 0, n_pn = 0;
    int tail = 0;
    if (wave == 0 && !guest) {
        __builtin_amdgcn_s_setprio(2);   // the team waits for this wave's tiles
        traverse<Pol, kPer, kSoft, true>(S.lists, T, O, U.gb, U.gh2, T.sys_root[gd.z], lane,
                                         theta2, eps2, [&](bool node, const int* list, int cnt, auto reload) {
            const int step = in_turn ? kPart : kW;
            for (int off = 0; off < cnt; off += step) {
                const int n = cnt - off < step ? cnt - off : step;
                const int s = tail % kRing;
                int full = lds_get(&S.full[s]);
                const int id = lane < n ? list[off + lane] : 0;
                // a full queue: take its oldest tile that no wave has asked for,
                // or wait for the wave that has asked for the slot's
                while (full != 0) {
                    int t = -1;
                    if (lane == 0) {
                        int h = lds_get(&S.head);
                        if (h < tail && __hip_atomic_compare_exchange_strong(&S.head, &h, h + 1, __ATOMIC_RELAXED,
                                                                             __ATOMIC_RELAXED,
                                                                             __HIP_MEMORY_SCOPE_WORKGROUP))
                            t = h;
                    }
                    t = __builtin_amdgcn_readfirstlane(t);
                    if (t >= 0) {
                        team_acquire();
                        evaluate(t);
                        reload();
                    } else {
                        __builtin_amdgcn_s_sleep(1);
                    }
                    full = lds_get(&S.full[s]);
                }
                if (lane < n) S.ring[s][lane] = id;
                if (lane == 0) {
                    lds_put(&S.info[s], node ? -(n + 128 * off) : n + 128 * off);
                    lds_put(&S.full[s], 1);
                }
                // (the LDS takes a wave's writes in order: no wait for the tile's
                // before the one that announces it)
                asm volatile("" ::: "memory");
                ++tail;
                if (lane == 0) lds_put(&S.tail, tail);
            }
            if (node) n_pn += (uint64_t)cnt;
            else n_pp += (uint64_t)cnt;
            wave_sync();
        });
        __builtin_amdgcn_s_setprio(0);
        team_release();
        if (lane == 0) lds_put(&S.done, 1);
    }
    // take tiles until the traversal is done and none is left
    for (;;) {
        int t = 0;
        if (lane == 0) t = __hip_atomic_fetch_add(&S.head, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        t = __builtin_amdgcn_readfirstlane(t);
        bool any = true;
        while (lds_get(&S.tail) <= t) {   // the traversal goes on without this wave
            if (lds_get(&S.done) != 0) {
                team_acquire();
                any = lds_get(&S.tail) > t;   // (the last tiles are queued before done is set)
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (!any) break;
        team_acquire();
        evaluate(t);
    }
    if (guest) return;
    team_barrier(&S.arrived, ts);
    if (wave == 0) {
        while (lds_get(&S.turn) != tail) __builtin_amdgcn_s_sleep(1);   // guests may hold the last tiles
        team_acquire();
        typename Pol::Acc acc;
        typename Pol::Word* a = reinterpret_cast<typename Pol::Word*>(&acc) + Pol::kFirst;
#pragma unroll
        for (int k = 0; k < kN; ++k) a[k] = S.acc[k][lane];
        if (Pol::kGroupSum && tg.grp) {
            Pol::wave_sum(acc);
        } else if (part == 0) {
            for (int j = 1; j < sub; ++j)
#pragma unroll
                for (int k = 0; k < kN; ++k) a[k] += S.acc[k][slot + j * count];
        }
        if (part == 0) Pol::finish(T, O, acc, tg.p, tg);
        C.group(n_pp, n_pn, count);
    }
}

// Next group of a persistent walk: eight work queues, one per contiguous
// eighth of the (Morton-ordered) group list.  A workgroup starts on queue
// blockIdx % 8 -- the XCD the hardware dispatches it to, so spatially
// neighbouring groups share that XCD's L2 -- and steals from the other queues
// when its own runs dry (q counts the queues it has left).  Each queue's counter
// has a cache line of its own, which stays in its XCD's L2.
__device__ __forceinline__ int pop_group(const int32_t* __restrict__ ord, int* __restrict__ qctr, int n_groups,
                                         int& q) {
    const int home = blockIdx.x & 7;
    while (q < 8) {
        const int qq = (home + q) & 7;
        const int lo = (int)((int64_t)n_groups * qq / 8);
        const int hi = (int)((int64_t)n_groups * (qq + 1) / 8);
        const int k = atomicAdd(&qctr[qq * kQueueStride], 1);
        if (lo + k < hi) return ord ? ord[lo + k] : lo + k;
        ++q;
    }
    return -1;
}

// Persistent walk by workgroups of W waves, which walk groups each on its own
// or in teams, by the number of groups the device finds.  The register budget
// is held to 128 VGPRs (four waves per SIMD); the few values this spills live
// outside the interaction loops.
struct TeamRule {
    int solo_above, teams_above;   // more groups than this: single waves; teams of kMinTeam waves; else of W waves
};
template <class Pol, int kPer, bool kSoft, int W>
__global__ void __launch_bounds__(W * kW, Pol::kWaves) k_walk_team(Tree T, Groups Gr, WalkOut O,
                                             int* __restrict__ qctr, TeamRule R,
                                             float theta2, float eps2, float h2, float hinv) {
    using Solo = typename Pol::Lds;
    using Tile = typename Pol::Tile;
    using Team = TeamLds<Pol>;
    static_assert(W % kMinTeam == 0, "teams of kMinTeam waves fill a workgroup");
    constexpr size_t kTeamBytes = W * sizeof(Tile) + W / kMinTeam * sizeof(Team);
    constexpr size_t kBytes = W * sizeof(Solo) > kTeamBytes ? W * sizeof(Solo) : kTeamBytes;
    __shared__ __align__(16) char s_mem[kBytes];   // one or the other, never both
    __shared__ HelpLds<W> s_help;
    const int2 hdr = *reinterpret_cast<const int2*>(Gr.hdr);   // (one load: the next would wait as long again)
    const int n_groups = hdr.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int q = 0;
    WalkCount C;
    if (n_groups > R.solo_above) {
        if (threadIdx.x < W) s_help.state[threadIdx.x] = kHelpNone;
        if (threadIdx.x == 0) s_help.walking = W;
        __syncthreads();
        Solo* all = reinterpret_cast<Solo*>(s_mem);
        for (;;) {
            int g = -1;
            if (ag_lane() == 0) g = pop_group(nullptr, qctr, n_groups, q);
            g = __builtin_amdgcn_readfirstlane(g);
            if (g < 0) break;
            walk_group<Pol, kPer, kSoft, W>(all, s_help, wave, T, Gr, O, g, theta2, eps2, h2, hinv, C);
            wave_sync();
        }
        if constexpr (can_help<Pol>()) help<Pol, kPer, kSoft, W>(all[wave], s_help, wave, T, Gr, O, eps2, h2, hinv);
    } else {
        const int ts = hdr.y > R.teams_above ? kMinTeam : W;
        Team* teams = reinterpret_cast<Team*>(s_mem + W * sizeof(Tile));
        const int n_teams = W / ts, own = wave / ts;
        Tile& st = reinterpret_cast<Tile*>(s_mem)[wave];
        const int me = wave % ts;
        if (me == 0 && ag_lane() == 0) {
            teams[own].arrived = 0;
            teams[own].state = kTeamClosed;
        }
        __syncthreads();
        bool guest = false;
        for (;;) {
            int team = own;
            if (!guest) {
                if (me == 0 && ag_lane() == 0) {
                    lds_put(&teams[own].state, kTeamClosed);
                    // (closed before the queue is asked: a wave that finds the queues
                    // empty after this must not find the team still open on the group
                    // before the one it gets here)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    const int g = pop_group(kPer == kOpen && ts < W ? Gr.ord : nullptr, qctr, n_groups, q);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    lds_put(&teams[own].g, g);
                    if (g < 0) lds_put(&teams[own].state, kTeamDone);
                }
                team_barrier(&teams[own].arrived, ts);
                guest = lds_get(&teams[own].g) < 0;
            }
            if (guest) {
                // No group is left for any team (the queues only run up): a
                // team that is open walks its last one, and this wave takes
                // tiles of it.  The waves of a team start at different hosts.
                bool left = false;
                team = -1;
                for (int k = 0; k < n_teams - 1; ++k) {
                    const int o = (own + 1 + (me + k) % (n_teams - 1)) % n_teams;
                    const int state = lds_get(&teams[o].state);
                    left |= state != kTeamDone;
                    if (team < 0 && state == kTeamOpen &&
                        (lds_get(&teams[o].done) == 0 || lds_get(&teams[o].head) < lds_get(&teams[o].tail)))
                        team = o;
                }
                if (!left) break;
                if (team < 0) {
                    __builtin_amdgcn_s_sleep(8);
                    continue;
                }
                team_acquire();
            }
            const int g = lds_get(&teams[team].g);
            if (g < 0) continue;   // the host has just ended
            walk_group_team<Pol, kPer, kSoft>(teams[team], st, me, ts, guest, T, Gr, O, Gr.grp[g], theta2, eps2, h2,
                                              hinv, C);
        }
    }
    C.add_to(O.stats);
}

// ---------------------------------------------------------------------------
// Ewald correction table
// ---------------------------------------------------------------------------
// The periodic field of a unit mass (G = 1) and its images with a uniform
// neutralising background, split with alpha = 2 / L:
//   g = sum_n B(r_n) y_n + (4 pi / L^3) sum_k k / k^2 exp(-k^2 / 4 alpha^2) sin(k.d),
//   B(r) = erfc(alpha r) / r^3 + (2 alpha / sqrt(pi)) exp(-alpha^2 r^2) / r^2,
// y_n = d + n L; with C = B'/r and D = C'/r per image,
//   T_ab = -(B delta_ab + C y_a y_b),
//   H_abc = dT_ab / dd_c = -(C (y_c delta_ab + y_b delta_ac + y_a delta_bc) + D y_a y_b y_c),
// and the reciprocal terms -w k_a k_b cos(k.d), +w k_a k_b k_c sin(k.d).  The
// n = 0 image enters without its Newtonian part (B -> B - 1/r^3), by the
// series of that difference where alpha r < 1/2, so the table holds the
// correction dg = g - d / |d|^3 (and its derivatives), smooth up to d = 0.
// Images |n_a| <= 3, wave vectors |h_a| <= 4 (dropped terms below 1e-19).
__device__ void ewald_radial(double r, double alpha, bool newton_removed, double& B, double& C, double& D) {
    const double sp = 1.1283791670955126;   // 2 / sqrt(pi)
    const double z = alpha * r;
    if (newton_removed && z < 0.5) {
        // c_k = (-1)^k 2k / ((2k + 1) k!) alpha^(2k+1):  B = sp sum_{k>=1} c_k r^(2k-2),
        // C = sp sum_{k>=2} c_k (2k-2) r^(2k-4),  D = sp sum_{k>=3} c_k (2k-2)(2k-4) r^(2k-6)
        double sb = 0.0, sc = 0.0, sd = 0.0;
        double ak = alpha * alpha * alpha, fact = 1.0;
        double r2 = r * r, pb = 1.0, pc = 1.0, pd = 1.0;
        for (int k = 1; k <= 24; ++k) {
            if (k > 1) {
                ak *= alpha * alpha;
                fact *= k;
                pb *= r2;
            }
            if (k > 2) pc *= r2;
            if (k > 3) pd *= r2;
            const double c = ((k & 1) ? -1.0 : 1.0) * (2.0 * k) / ((2.0 * k + 1.0) * fact) * ak;
            sb += c * pb;
            if (k >= 2) sc += c * (2.0 * k - 2.0) * pc;
            if (k >= 3) sd += c * (2.0 * k - 2.0) * (2.0 * k - 4.0) * pd;
        }
        B = sp * sb;
        C = sp * sc;
        D = sp * sd;
        return;
    }
    const double e = exp(-z * z), ec = erfc(z);
    const double r2 = r * r, r3 = r2 * r, r4 = r2 * r2, r5 = r4 * r;
    double b = ec / r3 + sp * alpha * e / r2;
    double b1 = -3.0 * ec / r4 - sp * alpha * e * (3.0 / r3 + 2.0 * alpha * alpha / r);
    double b2 = 12.0 * ec / r5 + sp * alpha * e * (12.0 / r4 + 8.0 * alpha * alpha / r2 + 4.0 * alpha * alpha * alpha * alpha);
    if (newton_removed) {
        b -= 1.0 / r3;
        b1 += 3.0 / r4;
        b2 -= 12.0 / r5;
    }
    B = b;
    C = b1 / r;
    D = b2 / r2 - b1 / r3;
}

__global__ void k_ewald_table(double L, int ne, double h, float4* __restrict__ tab) {
    const int np = (ne + 1) * (ne + 1) * (ne + 1);
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= np) return;
    const int iz = id % (ne + 1), iy = (id / (ne + 1)) % (ne + 1), ix = id / ((ne + 1) * (ne + 1));
    const double d[3] = {ix * h, iy * h, iz * h};
    const double alpha = 2.0 / L;
    double g[3] = {0, 0, 0}, T[6] = {0, 0, 0, 0, 0, 0}, H[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    // index pairs of T and triples of H
    const int ta[6] = {0, 1, 2, 0, 0, 1}, tb[6] = {0, 1, 2, 1, 2, 2};
    const int ha[10] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 2}, hb[10] = {0, 0, 0, 1, 1, 2, 1, 1, 2, 2},
              hc[10] = {0, 1, 2, 1, 2, 2, 1, 2, 2, 2};
    for (int a = -3; a <= 3; ++a)
        for (int b = -3; b <= 3; ++b)
            for (int c = -3; c <= 3; ++c) {
                const double y[3] = {d[0] + a * L, d[1] + b * L, d[2] + c * L};
                const double r = sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]);
                double B, C, D;
                ewald_radial(r, alpha, a == 0 && b == 0 && c == 0, B, C, D);
                for (int q = 0; q < 3; ++q) g[q] += B * y[q];
                for (int q = 0; q < 6; ++q) T[q] -= (ta[q] == tb[q] ? B : 0.0) + C * y[ta[q]] * y[tb[q]];
                for (int q = 0; q < 10; ++q) {
                    const int i = ha[q], j = hb[q], k = hc[q];
                    const double del = (i == j ? y[k] : 0.0) + (i == k ? y[j] : 0.0) + (j == k ? y[i] : 0.0);
                    H[q] -= C * del + D * y[i] * y[j] * y[k];
                }
            }
    const double pre = 4.0 * 3.14159265358979323846 / (L * L * L);
    const double kf = 2.0 * 3.14159265358979323846 / L;
    for (int a = -4; a <= 4; ++a)
        for (int b = -4; b <= 4; ++b)
            for (int c = -4; c <= 4; ++c) {
                if (a == 0 && b == 0 && c == 0) continue;
                const double k[3] = {kf * a, kf * b, kf * c};
                const double k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2];
                const double w = pre * exp(-k2 / (4.0 * alpha * alpha)) / k2;
                double sn, cs;
                sincos(k[0] * d[0] + k[1] * d[1] + k[2] * d[2], &sn, &cs);
                for (int q = 0; q < 3; ++q) g[q] += w * k[q] * sn;
                for (int q = 0; q < 6; ++q) T[q] -= w * k[ta[q]] * k[tb[q]] * cs;
                for (int q = 0; q < 10; ++q) H[q] += w * k[ha[q]] * k[hb[q]] * k[hc[q]] * sn;
            }
    float4* o = tab + 5 * (int64_t)id;
    o[0] = make_float4((float)g[0], (float)g[1], (float)g[2], (float)T[0]);
    o[1] = make_float4((float)T[1], (float)T[2], (float)T[3], (float)T[4]);
    o[2] = make_float4((float)T[5], (float)H[0], (float)H[1], (float)H[2]);
    o[3] = make_float4((float)H[3], (float)H[4], (float)H[5], (float)H[6]);
    o[4] = make_float4((float)H[7], (float)H[8], (float)H[9], 0.f);
}

// ---------------------------------------------------------------------------
// active rows -> groups
// ---------------------------------------------------------------------------
// A group is a run of consecutive sibling cells, each with at most 64 active
// targets, whose parent holds more than 64 (so a group never reaches beyond
// its parent cell), packed up to 64 targets; a leaf holding more than 64
// active targets (coincident points at the deepest level) is cut in chunks
// of 64.  Cells of the system-prefix levels are never packed together, so a
// group never mixes systems.
// Active rows -> sorted positions, without atomics: every listed entry k stamps
// k + 1 at its row's position; a position is active if the entry its stamp
// names still names its row (stamps of earlier lists fail that unless a
// current entry names the row, and then the stamp is that entry's).  A list
// whose entries are in range and unique marks as many positions as it has
// entries; otherwise the flag is raised.  The list's length is n_act, or, with
// n_dev set, the count stored at *n_dev (at most n_act = n; a count outside
// [0, n] raises the flag and lists none).
__device__ __forceinline__ int64_t list_len(int64_t n_act, const int64_t* __restrict__ n_dev) {
    if (!n_dev) return n_act;
    const int64_t v = *n_dev;
    return (v < 0 || v > n_act) ? 0 : v;
}

__global__ void k_mark_stamp(int64_t n_act, const int64_t* __restrict__ n_dev, const int32_t* __restrict__ idx,
                             int64_t n, const int32_t* __restrict__ rank, int32_t* __restrict__ stamp,
                             int32_t* __restrict__ flags, int64_t* __restrict__ n_total) {
    if (n_dev && blockIdx.x == 0 && threadIdx.x == 0) {
        const int64_t v = *n_dev;
        if (v < 0 || v > n_act) atomicOr(flags, AGF_BADINDEX);
        else if (n_total) *n_total += v;   // running total of evaluations
    }
    n_act = list_len(n_act, n_dev);
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_act;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx[k];
        if (i >= 0 && i < n) stamp[rank[i]] = (int32_t)(k + 1);
    }
}

constexpr int kMarkTile = 2048;   // positions a workgroup takes
__global__ void __launch_bounds__(256) k_mark_flag(int64_t n_act, const int64_t* __restrict__ n_dev,
                                                   const int32_t* __restrict__ idx, int64_t n,
                                                   const int32_t* __restrict__ perm,
                                                   const int32_t* __restrict__ stamp, int32_t* __restrict__ flag,
                                                   int32_t* __restrict__ tile_sum) {
    __shared__ int s_sum[4];
    n_act = list_len(n_act, n_dev);
    int sum = 0;
#pragma unroll
    for (int r = 0; r < kMarkTile / 256; ++r) {
        const int64_t p = (int64_t)blockIdx.x * kMarkTile + r * 256 + threadIdx.x;
        if (p >= n) continue;
        const int64_t k = (int64_t)stamp[p] - 1;
        const int f = k >= 0 && k < n_act && idx[k] == perm[p];
        flag[p] = f;
        sum += f;
    }
    sum = ag_wave_sum(sum);
    if (ag_lane() == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

// offsets of the active positions (n + 1 of them) and their list
__global__ void __launch_bounds__(256) k_mark_list(int64_t n_act, const int64_t* __restrict__ n_dev, int64_t n,
                                                   const int32_t* __restrict__ flag,
                                                   const int32_t* __restrict__ tile_sum, bool scanned,
                                                   int32_t* __restrict__ off, int32_t* __restrict__ out,
                                                   int32_t* __restrict__ flags) {
    __shared__ int s_tmp[4];
    int run = ag_tiles_before256(tile_sum, (int)blockIdx.x, scanned, s_tmp);
    for (int r = 0; r < kMarkTile / 256; ++r) {
        const int64_t p = (int64_t)blockIdx.x * kMarkTile + r * 256 + threadIdx.x;
        const int f = p < n ? flag[p] : 0;
        int tot;
        const int e = run + ag_block_scan256(f, s_tmp, &tot);
        if (p < n) off[p] = e;
        if (f) out[e] = (int32_t)p;
        run += tot;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        off[n] = run;
        if (run != list_len(n_act, n_dev)) atomicOr(flags, AGF_BADINDEX);
    }
}

struct GroupCtx {
    const int4* __restrict__ link;
    const int32_t* __restrict__ slot;   // row of an inner node's children ...
    const int4* __restrict__ child;     // ... by octant (-1: none), two int4 a row
    const int32_t* __restrict__ aoff;   // exclusive scan of the active flags over sorted positions (null: all)
    const int64_t* __restrict__ sys_off;
    int n_sys;
    int sys_levels;
    int span;   // cap on the particles of a group's cells (0 = none)
    int cap;    // targets per group (at most one wave)
    int split;  // groups of 33 .. split targets are emitted as two halves (0 = none)
    int pack;   // 1: runs of small children are cut every `cap` targets, not at child boundaries
};

__device__ __forceinline__ int sys_of_pos(const GroupCtx& C, int64_t p) {
    int lo = 0, hi = C.n_sys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (C.sys_off[mid] <= p) lo = mid; else hi = mid;
    }
    return lo;
}

// Count (out == nullptr) or write the groups node `id` is responsible for.
__device__ int node_groups(const GroupCtx& C, int id, int4* __restrict__ out) {
    const int4 L = C.link[id];
    const int lvl = L.w & 0xff;
    const bool leaf = (L.w & 0x100) != 0;
    const int a0 = C.aoff ? C.aoff[L.y] : L.y;
    const int a = (C.aoff ? C.aoff[L.y + L.z] : L.y + L.z) - a0;
    const bool forced = lvl < C.sys_levels;
    // too many targets for one wave, or (span) a cell too large to be one
    // compact group even if few of its particles are active
    const bool big = forced || a > C.cap || (C.span > 0 && !leaf && L.z > C.span);
    int ng = 0;
    auto emit1 = [&](int start, int cnt, int64_t pos) {
        if (out) out[ng] = make_int4(start, cnt, C.n_sys > 1 ? sys_of_pos(C, pos) : 0, 0);
        ++ng;
    };
    // a wave gives each of k targets 64 / k lanes (whole lanes): 33 .. 42
    // targets leave a third or more of the lanes idle, two halves of 17 .. 21
    // use three lanes each
    auto emit = [&](int start, int cnt, int64_t pos) {
        if (C.split > 0 && cnt > 32 && cnt <= C.split) {
            emit1(start, cnt / 2, pos);
            emit1(start + cnt / 2, cnt - cnt / 2, pos);
        } else {
            emit1(start, cnt, pos);
        }
    };
    if (!big) {
        if (id == 0 && a > 0) emit(a0, a, L.y);   // a small whole tree is one group
        return ng;
    }
    if (leaf) {
        for (int k = 0; k < a; k += C.cap) emit(a0 + k, a - k < C.cap ? a - k : C.cap, L.y);
        return ng;
    }
    int run_start = 0, run_cnt = 0, run_span = 0;
    int64_t run_pos = 0;
    // (pack: a run, contiguous in the target order, is cut into groups of
    // `cap` targets and a remainder, which may split a child between two
    // groups; the groups stay inside this node's cell)
    auto emit_run = [&](int start, int cnt, int64_t pos) {
        if (!C.pack) {
            emit(start, cnt, pos);
            return;
        }
        for (int k = 0; k < cnt; k += C.cap) emit(start + k, cnt - k < C.cap ? cnt - k : C.cap, pos);
    };
    // the children (in order) all at once from the node's row: following their
    // skip links would take a chain of up to eight loads
    const int64_t row = C.slot[id];
    const int4 ra = C.child[2 * row], rb = C.child[2 * row + 1];
    const int ch8[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
    int4 link8[8];
    int act0[8], act1[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) link8[k] = ch8[k] >= 0 ? C.link[ch8[k]] : make_int4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        act0[k] = C.aoff && ch8[k] >= 0 ? C.aoff[link8[k].y] : link8[k].y;
        act1[k] = C.aoff && ch8[k] >= 0 ? C.aoff[link8[k].y + link8[k].z] : link8[k].y + link8[k].z;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (ch8[k] < 0) continue;
        const int4 Lc = link8[k];
        const int c0 = act0[k], ac = act1[k] - c0;
        const bool leafc = (Lc.w & 0x100) != 0;
        const bool bigc = (Lc.w & 0xff) < C.sys_levels || ac > C.cap || (C.span > 0 && !leafc && Lc.z > C.span);
        if (bigc || ac == 0 || forced) {
            if (run_cnt > 0) emit_run(run_start, run_cnt, run_pos);
            run_cnt = 0;
            run_span = 0;
            if (forced && !bigc && ac > 0) emit(c0, ac, Lc.y);
            continue;
        }
        if ((!C.pack && run_cnt + ac > C.cap) || (C.span > 0 && run_span + Lc.z > C.span)) {
            if (run_cnt > 0) emit_run(run_start, run_cnt, run_pos);
            run_cnt = 0;
            run_span = 0;
        }
        if (run_cnt == 0) {
            run_start = c0;
            run_pos = Lc.y;
        }
        run_cnt += ac;
        run_span += Lc.z;
    }
    if (run_cnt > 0) emit_run(run_start, run_cnt, run_pos);
    return ng;
}

// Groups each node owns, and the total of every tile of nodes.
// One node a thread: the work is a chain of dependent loads, so more nodes a
// thread only lengthen it (four: 25 + 16 us for the two kernels at 2^15
// particles, now 7 + 7; 22 + 25 at 2^20, now 8 + 10).
constexpr int kGroupTile = 256;   // nodes a workgroup takes at a time
__global__ void __launch_bounds__(256) k_group_count(GroupCtx C, const int64_t* __restrict__ hdr,
                                                     int32_t* __restrict__ gcnt, int32_t* __restrict__ tile_sum) {
    __shared__ int s_sum[4];
    const int64_t nn = hdr[0];
    for (int64_t t = blockIdx.x; t * kGroupTile < nn; t += gridDim.x) {
        const int64_t id = t * kGroupTile + threadIdx.x;
        const int g = id < nn ? node_groups(C, (int)id, nullptr) : 0;
        if (id < nn) gcnt[id] = g;
        const int sum = ag_wave_sum(g);
        __syncthreads();
        if (ag_lane() == 0) s_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) tile_sum[t] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    }
}

// The groups in node order, their number, and the walks' work queues reset.
// Where they hold fewer than kFew targets on average the team rule is given four
// times their number (launch_walk).
constexpr int kFew = 8;
__global__ void __launch_bounds__(256) k_group_emit(GroupCtx C, const int64_t* __restrict__ hdr,
                                                    const int32_t* __restrict__ gcnt,
                                                    const int32_t* __restrict__ tile_sum, bool scan,
                                                    int4* __restrict__ grp, int32_t* __restrict__ ord, int32_t* __restrict__ ghdr,
                                                    int* __restrict__ qctr) {
    __shared__ int s_tmp[4];
    const int64_t nn = hdr[0];
    const int n = C.link[0].z, targets = C.aoff ? C.aoff[n] : n;   // (the root holds every position)
    const bool scanned = scan && (nn + kGroupTile - 1) / kGroupTile > kTilesRead;
    if (blockIdx.x == 0 && threadIdx.x < 2 * 8) qctr[threadIdx.x * kQueueStride] = 0;   // two walks' queues
    for (int64_t t = blockIdx.x; t * kGroupTile < nn; t += gridDim.x) {
        const int64_t id = t * kGroupTile + threadIdx.x;
        const int before = ag_tiles_before256(tile_sum, (int)t, scanned, s_tmp);
        const int g = id < nn ? gcnt[id] : 0;
        int tot;
        const int e = before + ag_block_scan256(g, s_tmp, &tot);
        if (g > 0) {
            node_groups(C, (int)id, grp + e);
            for (int k = 0; k < g; ++k) ord[e + k] = e + k;   // (k_group_order may change it)
        }
        if ((t + 1) * kGroupTile >= nn && threadIdx.x == 0) {
            const int ng = before + tot;
            ghdr[0] = ng;
            ghdr[1] = targets < (int64_t)kFew * ng ? (int)std::min<int64_t>(4 * (int64_t)ng, INT_MAX) : ng;
        }
    }
}

// The order in which teams take the groups: in each work queue's share of them
// those first that take longest, so that the last ones to start are short.  By
// a group's targets (above 32, each has one lane and every tile takes 64
// steps), or with the relative opening test by its smallest |a_old|, to a
// factor of sqrt(2): it sets how far the nodes are opened.  By one workgroup,
// for as many groups as are walked in such teams.
__global__ void __launch_bounds__(256) k_group_amin(Groups Gr, OrderRange R, const int32_t* __restrict__ perm,
                                                    const float* __restrict__ rel_a, float* __restrict__ amin) {
    const int n = Gr.hdr[0], lane = ag_lane();
    if (!R.holds(n)) return;
    for (int g = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; g < n; g += (gridDim.x * blockDim.x) >> 6) {
        const int4 gd = Gr.grp[g];
        float a = FLT_MAX;
        if (lane < gd.y) a = rel_a[perm[Gr.act_pos ? Gr.act_pos[gd.x + lane] : gd.x + lane]];
        a = ag_wave_min(a);
        if (lane == 0) amin[g] = a;
    }
}

__global__ void __launch_bounds__(1024) k_group_order(const int32_t* __restrict__ ghdr, OrderRange R,
                                                      const int4* __restrict__ grp, const float* __restrict__ amin,
                                                      int32_t* __restrict__ ord) {
    constexpr int K = 512;   // classes: exponent and one bit of the fraction
    __shared__ int s_at[8 * K], s_w[16];
    const int n = ghdr[0], t = threadIdx.x;
    if (!R.holds(n)) return;
    auto key = [&](int g) {
        int q = (int)((int64_t)g * 8 / n);   // the work queue that holds g (pop_group)
        while (g >= (int)((int64_t)n * (q + 1) / 8)) ++q;
        const int k = amin ? (__float_as_int(amin[g]) >> 22) & (K - 1) : (grp[g].y > 32 ? 0 : 1);
        return q * K + k;
    };
    for (int i = t; i < 8 * K; i += 1024) s_at[i] = 0;
    __syncthreads();
    for (int g = t; g < n; g += 1024) atomicAdd(&s_at[key(g)], 1);
    __syncthreads();
    int c[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = sum;
        sum += s_at[4 * t + k];
    }
    const int incl = ag_wave_incl_scan(sum);
    if ((t & 63) == 63) s_w[t >> 6] = incl;
    __syncthreads();
    int base = incl - sum;
    for (int w = 0; w < (t >> 6); ++w) base += s_w[w];
#pragma unroll
    for (int k = 0; k < 4; ++k) s_at[4 * t + k] = base + c[k];
    __syncthreads();
    for (int g = t; g < n; g += 1024) ord[atomicAdd(&s_at[key(g)], 1)] = g;
}

int grid_for(int64_t n, int threads = 256) {
    int64_t b = (n + threads - 1) / threads;
    if (b > 8192) b = 8192;
    return (int)(b < 1 ? 1 : b);
}

}  // namespace

int ag_prepare_groups(ag_ctx* c, const int32_t* idx, int64_t n_act, int64_t* max_groups, const int64_t* n_dev,
                      int64_t* n_total) {
    const int64_t n = c->n;
    const int64_t mg = n_act + c->n_sys + 1;   // every group holds at least one target
    const int64_t mtiles = (n + kMarkTile - 1) / kMarkTile, gtiles = (c->max_nodes + kGroupTile - 1) / kGroupTile;
    AG_TRY(ag_ensure(c, c->act_flag, n * 4));
    AG_TRY(ag_ensure(c, c->act_off, (n + 1) * 4));
    AG_TRY(ag_ensure(c, c->act_pos, n * 4));
    AG_TRY(ag_ensure(c, c->grp, mg * 16));
    AG_TRY(ag_ensure(c, c->grp_hdr, (1 + 2 * 8) * kQueueStride * sizeof(int32_t)));
    AG_TRY(ag_ensure(c, c->grp_cnt, c->max_nodes * 4));
    AG_TRY(ag_ensure(c, c->grp_tile, gtiles * 4));
    PhaseScope phase(c, AG_PHASE_GROUPS);
    hipStream_t st = c->stream;
    int32_t* off = c->act_off.as<int32_t>();
    c->all_active = idx == nullptr;
    if (idx) {
        int32_t* flag = c->act_flag.as<int32_t>();
        int32_t* stamp = c->in_cnt.as<int32_t>();
        int32_t* msum = c->vals[0].as<int32_t>();   // (as many as tiles at least)
        int32_t* flags = c->dflags.as<int32_t>();
        hipLaunchKernelGGL(k_mark_stamp, dim3(grid_for(n_act)), dim3(256), 0, st, n_act, n_dev, idx, n,
                           c->rank.as<int32_t>(), stamp, flags, n_total);
        hipLaunchKernelGGL(k_mark_flag, dim3((unsigned)mtiles), dim3(256), 0, st, n_act, n_dev, idx, n,
                           c->perm.as<int32_t>(), stamp, flag, msum);
        const bool scan = mtiles > kTilesRead;
        if (scan) ag_tile_scan(c, msum, 1, mtiles);
        hipLaunchKernelGGL(k_mark_list, dim3((unsigned)mtiles), dim3(256), 0, st, n_act, n_dev, n, flag, msum, scan,
                           off, c->act_pos.as<int32_t>(), flags);
    }
    // with every particle active the flags, their scan and the position list
    // are the identity: the grouping and the walk use sorted positions directly
    GroupCtx C{c->nd_link.as<int4>(), c->nd_slot.as<int32_t>(), c->child.as<int4>(), idx ? off : (const int32_t*)nullptr, c->sys_off.as<int64_t>(), c->n_sys,
               c->sys_levels, c->group_span, c->group_cap, c->group_split, c->group_pack};
    const int64_t* hdr = c->tree_hdr.as<int64_t>();
    int32_t* gcnt = c->grp_cnt.as<int32_t>();
    int32_t* gsum = c->grp_tile.as<int32_t>();
    int32_t* ghdr = c->grp_hdr.as<int32_t>();
    const unsigned gblocks = (unsigned)std::min<int64_t>(gtiles, 4096);
    hipLaunchKernelGGL(k_group_count, dim3(gblocks), dim3(256), 0, st, C, hdr, gcnt, gsum);
    // (a tree has far fewer nodes than there is room for: of 2^22 particles a
    // million, 4000 tiles, with room for nine)
    const bool scan = gtiles > 4 * kTilesRead;
    if (scan) ag_tile_scan(c, gsum, 1, gtiles, hdr, kGroupTile);
    hipLaunchKernelGGL(k_group_emit, dim3(gblocks), dim3(256), 0, st, C, hdr, gcnt, gsum, scan,
                       c->grp.as<int4>(), c->in_off.as<int32_t>(), ghdr, ghdr + kQueueStride);
    *max_groups = mg;
    return AG_OK;
}

namespace {

// ---------------------------------------------------------------------------
// vector-charge moments of the adjoint weights
// ---------------------------------------------------------------------------
// per node (FP64, 31 doubles): W0 (3), W1 row-major (9: W1_bc = sum w_b y_c),
// W2 (18: for b = x, y, z the symmetric sum w_b y y^T as xx yy zz xy xz yz),
// number of charged particles; FP32 copy as 8 float4 (W0 + count, W1, W2).
constexpr int kW64 = 31;

__device__ void store_w(int64_t id, const double* r, double* __restrict__ w64, float4* __restrict__ wf) {
    double* o = w64 + id * kW64;
#pragma unroll
    for (int k = 0; k < kW64; ++k) o[k] = r[k];
    float4* f = wf + 8 * id;
    f[0] = make_float4((float)r[0], (float)r[1], (float)r[2], (float)r[30]);
#pragma unroll
    for (int q = 1; q < 8; ++q)
        f[q] = make_float4((float)r[4 * q - 1], (float)r[4 * q], (float)r[4 * q + 1],
                           q < 7 ? (float)r[4 * q + 2] : 0.f);
}

// the same by G lanes that all hold r: lane s writes every G-th word
template <int G>
__device__ __forceinline__ void store_w_part(int64_t id, int s, const double* r, double* __restrict__ w64,
                                             float4* __restrict__ wf) {
    double* o = w64 + id * kW64;
#pragma unroll
    for (int k = 0; k < kW64; ++k)
        if (k % G == s) o[k] = r[k];
    float4* f = wf + 8 * id;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (q % G == s)
            f[q] = q == 0 ? make_float4((float)r[0], (float)r[1], (float)r[2], (float)r[30])
                          : make_float4((float)r[q > 0 ? 4 * q - 1 : 0], (float)r[4 * q], (float)r[4 * q + 1],
                                        q < 7 ? (float)r[4 * q + 2] : 0.f);
}

// sum_w w_b y_c y_e over the 6 symmetric (c, e) pairs into W2 (18 entries)
__device__ __forceinline__ void add_w2(double* W2, const double* wv, const double* y) {
    const int a[6] = {0, 1, 2, 0, 0, 1}, b[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int bb = 0; bb < 3; ++bb)
#pragma unroll
        for (int k = 0; k < 6; ++k) W2[6 * bb + k] += wv[bb] * y[a[k]] * y[b[k]];
}

// sorted weights: w of active rows, zero elsewhere
// weights in key order; a row carries its charge if it is listed: by the
// flags, or every row (all = 1), or none (all = 0 with no flags)
__global__ void k_gather_w(int64_t n, const int32_t* __restrict__ perm, const int32_t* __restrict__ flag, int all,
                           const double* __restrict__ w, double4* __restrict__ ws) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = perm[p];
        const bool charged = flag ? flag[p] != 0 : all != 0;
        ws[p] = charged ? make_double4(w[3 * i], w[3 * i + 1], w[3 * i + 2], 1.0) : make_double4(0, 0, 0, 0);
    }
}

__global__ void k_leaf_wmoments(const int64_t* __restrict__ hdr, const int32_t* __restrict__ leaves,
                                const int4* __restrict__ link, const double* __restrict__ m64,
                                const double4* __restrict__ spos, const double4* __restrict__ ws,
                                double* __restrict__ w64, float4* __restrict__ wf) {
    const int64_t nl = hdr[0] - hdr[2];
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nl;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t id = leaves[t];
        const int4 L = link[id];
        const double* c = m64 + id * 25 + 1;   // node centre of mass
        double r[kW64];
#pragma unroll
        for (int q = 0; q < kW64; ++q) r[q] = 0.0;
        for (int j = L.y; j < L.y + L.z; ++j) {
            const double4 w = ws[j];
            if (w.w == 0.0) continue;
            const double4 x = spos[j];
            const double y[3] = {x.x - c[0], x.y - c[1], x.z - c[2]};
            const double wv[3] = {w.x, w.y, w.z};
            for (int b = 0; b < 3; ++b) {
                r[b] += wv[b];
                for (int cc = 0; cc < 3; ++cc) r[3 + 3 * b + cc] += wv[b] * y[cc];
            }
            add_w2(r + 12, wv, y);
            r[30] += 1.0;
        }
        store_w(id, r, w64, wf);
    }
}

// Shifted to the parent centre (y = y_child + dl):
//   W1_bc  = sum (W1_bc + W0_b dl_c)
//   W2_bce = sum (W2_bce + W1_bc dl_e + W1_be dl_c + W0_b dl_c dl_e)
// from an inner node's children, a lane per child.
template <int G>
__device__ __forceinline__ void form_inner_w(int t, int id, int s, const int4* __restrict__ child,
                                             const double* __restrict__ m64, double* __restrict__ w64,
                                             float4* __restrict__ wf) {
    static_assert(G == 8, "a lane per octant");
    const int4 c0 = child[2 * (int64_t)t], c1 = child[2 * (int64_t)t + 1];
    const int ch8[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    int ch = 0;   // picked by masks (no indexing by the lane number)
#pragma unroll
    for (int k = 0; k < 8; ++k) ch |= ch8[k] & -(int)(k == s);
    const double* c = m64 + (int64_t)id * 25 + 1;
    double r[kW64];
#pragma unroll
    for (int q = 0; q < kW64; ++q) r[q] = 0.0;
    if (ch >= 0) {
        const double* cw = w64 + (int64_t)ch * kW64;
        const double* cc = m64 + (int64_t)ch * 25 + 1;
#pragma unroll
        for (int q = 0; q < kW64; ++q) r[q] = cw[q];
        const double dl[3] = {cc[0] - c[0], cc[1] - c[1], cc[2] - c[2]};
        constexpr int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int b = 0; b < 3; ++b) {
#pragma unroll
            for (int k = 0; k < 6; ++k)
                r[12 + 6 * b + k] += r[3 + 3 * b + ia[k]] * dl[ib[k]] + r[3 + 3 * b + ib[k]] * dl[ia[k]] +
                                     r[b] * dl[ia[k]] * dl[ib[k]];
#pragma unroll
            for (int q = 0; q < 3; ++q) r[3 + 3 * b + q] += r[b] * dl[q];
        }
    }
#pragma unroll
    for (int q = 0; q < kW64; ++q) r[q] = grp_sum<G>(r[q]);
    store_w_part<G>(id, s, r, w64, wf);
}

// Levels l_hi down to l_lo: one level per launch (l_hi = l_lo, any grid),
// or several in a single-workgroup launch, the workgroup barrier between
// levels ordering each level after its children's.
// (One thread per node, its children one after another, took 20 us a level, a
// lane per child 7: gradient of 100 000 particles 2065 us, now 1920.)
__global__ void __launch_bounds__(256) k_inner_wlevel(int l_hi, int l_lo, const int32_t* __restrict__ lvl,
                               const int32_t* __restrict__ lvl_list, const int4* __restrict__ child,
                               const double* __restrict__ m64, double* __restrict__ w64, float4* __restrict__ wf) {
    constexpr int G = 8;
    const int s = threadIdx.x & (G - 1);
    for (int level = l_hi; level >= l_lo; --level) {
        if (level < l_hi) __syncthreads();   // single-workgroup launches only
        const int t_lo = lvl[kLvlOff + level], t_hi = lvl[kLvlOff + level + 1];
        for (int64_t t = t_lo + (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G; t < t_hi;
             t += (int64_t)gridDim.x * blockDim.x / G)   // uniform over the group
            form_inner_w<G>((int)t, lvl_list[t], s, child, m64, w64, wf);
    }
}

}  // namespace

static Tree make_tree(ag_ctx* c) {
    Tree T;
    T.rec = c->nd_rec.as<NodeRec>();
    T.sh = c->tree_soft ? c->soft_s.as<float>() : nullptr;
    T.link = c->nd_link.as<int4>();
    T.mp = c->nd_mp.as<float4>();
    T.spos = c->spos.as<double4>();
    T.svf = c->svf.as<float4>();
    T.perm = c->perm.as<int32_t>();
    T.sys_root = c->sys_root.as<int32_t>();
    T.ws = c->wsorted.as<double4>();
    T.wf = c->nd_wf.as<float4>();
    return T;
}

static int device_cus(ag_ctx* c) {
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
    return cus;
}

// A walk by workgroups of Pol::kTeamWaves waves, one workgroup resident per CU:
// AG_OPT_WALK_WAVES_PER_CU waves per CU in whole workgroups, where that is less
// than one by workgroups on some of the CUs (as many for each XCD).  How the groups
// are walked goes by how many there are for the P waves launched, read on the device:
//   above 4 P   single waves: they keep every lane at interactions, and the
//               last groups' tail is short (2^20 particles, 23 000 groups:
//               2.64 ms per step, 2.79 in teams of 4)
//   above P/4   teams of 4, whose traversing wave keeps three evaluating and
//               whose waves help the others at the end (64 systems of 4000
//               particles, 5900 groups: 1.25 ms per step, 2.2 by single waves,
//               1.8 by whole workgroups; 180 000 with the relative opening
//               test, whose longest groups set the time: 1.33, 4.2 and 1.6);
//               of fewer than 8 targets a group on average above P/16: such a
//               group has few tiles, and what it takes is its traversal (300 000
//               particles, 1000 active in 887 groups: 114 us, 233 by whole
//               workgroups, four rounds of them; 6 targets a group in 317 groups
//               72 and 93, but 17 in 353 197 and 145)
//   else        the whole workgroup (3000 particles, 96 groups: 0.20 ms per
//               step, 0.23 in teams of 8, 0.25 of 4, 0.63 by single waves;
//               32^3 periodic ones, 704 groups: 0.90 ms, 0.93, 1.12 and 3.5)
static int64_t walk_blocks(ag_ctx* c, int W) {
    const int64_t cus = device_cus(c);
    return c->walk_waves_per_cu >= W ? cus * (c->walk_waves_per_cu / W)
                                     : (cus * c->walk_waves_per_cu / W + 7) / 8 * 8;
}

template <class Pol, int kPer, bool kSoft = false>
static void launch_walk(ag_ctx* c, int64_t max_groups, const Groups& Gr, const WalkOut& O, int32_t* qctr,
                        float theta2, float eps2, float h2, float hinv) {
    constexpr int W = Pol::kTeamWaves;
    int64_t blocks = walk_blocks(c, W);
    const int waves = (int)(blocks * W);
    if (blocks > max_groups) blocks = (max_groups + 7) / 8 * 8;
    const TeamRule R{4 * waves, waves / 4};
    hipLaunchKernelGGL((k_walk_team<Pol, kPer, kSoft, W>), dim3((unsigned)blocks), dim3(W * kW), 0, c->stream,
                       make_tree(c), Gr, O, qctr, R, theta2, eps2, h2, hinv);
}

// Ewald table: spacing box / 64 over the octant [0, box / 2]^3 of the cell
constexpr int kEwaldPerBox = 64;
constexpr int kEwaldNE = 32;
constexpr int kEwaldGroupDiv = 32;    // groups of half extent <= box / 32 sum once

static int ewald_table(ag_ctx* c) {
    if (c->ewald_tab_box == c->box && c->ewald_tab.bytes) return AG_OK;
    const int np = (kEwaldNE + 1) * (kEwaldNE + 1) * (kEwaldNE + 1);
    AG_TRY(ag_ensure(c, c->ewald_tab, (size_t)np * 5 * sizeof(float4)));
    hipLaunchKernelGGL(k_ewald_table, dim3((np + 127) / 128), dim3(128), 0, c->stream, c->box, kEwaldNE,
                       c->box / kEwaldPerBox, c->ewald_tab.as<float4>());
    c->ewald_tab_box = c->box;
    return AG_OK;
}

static WalkOut make_out(ag_ctx* c, double G) {
    WalkOut O{};
    O.stats = c->stats.as<unsigned long long>();
    O.G = G;
    O.flags = c->dflags.as<int32_t>();
    O.iter_cap = (unsigned)std::min<int64_t>(c->max_nodes + c->n + 1024, UINT_MAX - 1);
    O.small_node = c->small_node;
    O.mac_offset = c->mac_offset != 0;
    O.box = c->box;
    O.box_inv = c->box > 0.0 ? 1.0 / c->box : 0.0;
    O.boxf = (float)O.box;
    O.boxf_inv = (float)O.box_inv;
    // a margin of a few float ulps keeps every accepted node clear of the cut
    O.box_half = (float)(0.5 * c->box * (1.0 - 1e-5));
    O.ewald_theta = 1.0f / (float)c->ewald_open;
    O.ewald_grp = (float)(c->box / kEwaldGroupDiv);
    O.etab = c->ewald_tab.as<float4>();
    O.etab_ne = kEwaldNE;
    O.etab_h = (float)(c->box / kEwaldPerBox);
    O.etab_hinv = (float)(kEwaldPerBox / c->box);
    O.etab_range = (float)(c->box * kEwaldNE / kEwaldPerBox * (1.0 + 1e-4));   // a few ulps of slack
    return O;
}

// The groups' order for a walk of n_act targets.  Groups hold 10 to 64 of them,
// 40 on average where all are active, so with fewer targets than 40 000 whole
// workgroups walk them and with far more single waves do: the launch (2 us)
// is spared there.  Measured with and without: 180 000 particles with the
// relative opening test 1.17 and 1.29 ms, gradient of 100 000 1.80 and 1.92,
// 2^17 with neighbour lengths 1.01 and 1.03, 64 systems of 4000 1.19 and 1.21;
// Ewald sums, where a group's cost goes by its width, no better.
static int order_groups(ag_ctx* c, int64_t n_act, bool rel, const Groups& Gr) {
    if (n_act < 40000 || n_act / 48 > kOrderMax) return AG_OK;
    // for either walk: the adjoint's workgroups hold fewer teams, the others more waves
    constexpr int Wa = AdjointPolicy::kTeamWaves, Wf = ForwardPolicy::kTeamWaves;
    const OrderRange R{(int)(walk_blocks(c, Wa) * (Wa / kMinTeam)),
                       (int)std::min<int64_t>(4 * walk_blocks(c, Wf) * Wf, kOrderMax)};
    PhaseScope phase(c, AG_PHASE_GROUPS);
    if (rel) {
        AG_TRY(ag_ensure(c, c->grp_amin, kOrderMax * sizeof(float)));
        hipLaunchKernelGGL(k_group_amin, dim3(1024), dim3(256), 0, c->stream, Gr, R, c->perm.as<int32_t>(),
                           c->rel_a.as<float>(), c->grp_amin.as<float>());
    }
    hipLaunchKernelGGL(k_group_order, dim3(1), dim3(1024), 0, c->stream, Gr.hdr, R, Gr.grp,
                       rel ? c->grp_amin.as<float>() : (const float*)nullptr, c->in_off.as<int32_t>());
    return AG_OK;
}

int ag_launch_eval(ag_ctx* c, const int32_t* idx, int64_t n_act, double theta, double eps, double G, double* acc,
                   double* jerk, double* tidal, const int64_t* n_dev, int64_t* n_total) {
    int64_t mg = 0;
    AG_TRY(ag_prepare_groups(c, idx, n_act, &mg, n_dev, n_total));
    Groups Gr{c->all_active ? (const int32_t*)nullptr : c->act_pos.as<int32_t>(), c->grp.as<int4>(),
              c->grp_hdr.as<int32_t>(), c->in_off.as<int32_t>()};
    const bool ewald = c->box > 0.0 && c->ewald;
    if (c->box <= 0.0) AG_TRY(order_groups(c, idx ? n_act : c->n, c->rel_n > 0, Gr));
    if (ewald) AG_TRY(ewald_table(c));
    WalkOut O = make_out(c, G);   // after the table, for its address
    O.acc = acc;
    O.jerk = jerk;
    O.tidal = tidal;
    if (c->rel_n > 0) {
        O.rel_a = c->rel_a.as<float>();
        O.rel_alpha = (float)c->rel_alpha;
        O.rel_g = (float)fabs(G);
    }
    const float th = (float)theta;
    const float e2 = (float)(eps * eps);
    int32_t* qctr = c->grp_hdr.as<int32_t>() + kQueueStride;
    {
        PhaseScope phase(c, AG_PHASE_WALK);
        const float hi = (float)(1.0 / eps);
        if (c->tree_soft) {   // per-particle softening lengths
            if (ewald) launch_walk<ForwardPolicy, kEwald, true>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
            else if (c->box > 0.0) launch_walk<ForwardPolicy, kNear, true>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
            else launch_walk<ForwardPolicy, kOpen, true>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
        } else if (ewald) {
            launch_walk<ForwardPolicy, kEwald>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
        } else if (c->box > 0.0) {
            launch_walk<ForwardPolicy, kNear>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
        } else if (!acc && !jerk) {
            launch_walk<TidalPolicy, kOpen>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
        } else {
            launch_walk<ForwardPolicy, kOpen>(c, mg, Gr, O, qctr, th * th, e2, e2, hi);
        }
    }
    if (ewald && (acc || tidal)) {
        // what the periodic images add to g and T, at the same images
        PhaseScope phase(c, AG_PHASE_EWALD);
        WalkOut E = O;
        E.stats = nullptr;
        E.rel_a = nullptr;
        launch_walk<EwaldPolicy, kEwald>(c, mg, Gr, E, qctr + 8 * kQueueStride, 0.f, 0.f, e2, (float)(1.0 / eps));
    }
    return AG_OK;
}

// Adjoint of L = sum_k w_k . g_k:
//   1. forward walk for T at the listed rows (the T_k w_k term);
//   2. sorted weights (zero on unlisted rows) and their node moments W0, W1, W2;
//   3. adjoint walk over all n targets with the same opening test, both walks
//      at theta * AG_OPT_ADJOINT_OPEN / 100.
int ag_launch_backward(ag_ctx* c, const int32_t* idx, int64_t n_act, const double* w, double theta, double eps,
                       double G, double* dLdx, double* dLdm) {
    const int64_t n = c->n;
    AG_TRY(ag_ensure(c, c->tmp_tidal, n * 6 * sizeof(double)));
    AG_TRY(ag_ensure(c, c->wsorted, n * sizeof(double4)));
    AG_TRY(ag_ensure(c, c->nd_w, c->max_nodes * kW64 * sizeof(double)));
    AG_TRY(ag_ensure(c, c->nd_wf, c->max_nodes * 8 * sizeof(float4)));
    double* tin = c->tmp_tidal.as<double>();
    // both walks open nodes at a fraction of theta: their kernels (the tidal
    // tensor and J, 1/r^3) are one derivative deeper than the force's
    theta *= c->adj_open / 100.0;
    if (n_act > 0) AG_TRY(ag_launch_eval(c, idx, n_act, theta, eps, G, nullptr, nullptr, tin));
    // charges: the listed rows (flags of that evaluation), all rows, or none
    const int32_t* cflag = (n_act > 0 && !c->all_active) ? c->act_flag.as<int32_t>() : nullptr;
    const int call = n_act > 0 && c->all_active ? 1 : 0;

    PhaseScope phase(c, AG_PHASE_ADJOINT);
    hipStream_t st = c->stream;
    hipLaunchKernelGGL(k_gather_w, dim3(grid_for(n)), dim3(256), 0, st, n, c->perm.as<int32_t>(), cflag, call, w,
                       c->wsorted.as<double4>());
    hipLaunchKernelGGL(k_leaf_wmoments, dim3(grid_for(n / 4 + 1)), dim3(256), 0, st, c->tree_hdr.as<int64_t>(),
                       c->leaf_list.as<int32_t>(), c->nd_link.as<int4>(), c->nd_64.as<double>(),
                       c->spos.as<double4>(), c->wsorted.as<double4>(), c->nd_w.as<double>(), c->nd_wf.as<float4>());
    const int64_t inner_bound = c->max_nodes - n;
    int g = grid_for(8 * (inner_bound > 0 ? inner_bound : 1));   // eight lanes a node
    if (g > 1024) g = 1024;
    {
        // levels below the deepest the host has seen in one single-workgroup
        // launch (usually empty), then one launch per level down to 3, and
        // levels 2-0 (at most 73 nodes) in one single-workgroup launch
        const int32_t* lvl = reinterpret_cast<const int32_t*>(c->tree_hdr.as<int64_t>() + 8);
        const int32_t* ll = c->lvl_list.as<int32_t>();
        const int4* ch = c->child.as<int4>();
        const double* m64 = c->nd_64.as<double>();
        double* w64 = c->nd_w.as<double>();
        float4* wf = c->nd_wf.as<float4>();
        constexpr int kTop = 2;
        int lc = c->seen_max_level - 1;
        if (c->seen_max_level < 0 || lc > AG_MAX_LEVEL - 1) lc = AG_MAX_LEVEL - 1;
        if (lc < kTop + 1) lc = kTop;
        if (lc < AG_MAX_LEVEL - 1)
            hipLaunchKernelGGL(k_inner_wlevel, dim3(1), dim3(256), 0, st, AG_MAX_LEVEL - 1, lc + 1, lvl, ll, ch, m64,
                               w64, wf);
        for (int l = lc; l > kTop; --l)
            hipLaunchKernelGGL(k_inner_wlevel, dim3(g), dim3(256), 0, st, l, l, lvl, ll, ch, m64, w64, wf);
        hipLaunchKernelGGL(k_inner_wlevel, dim3(1), dim3(256), 0, st, kTop, 0, lvl, ll, ch, m64, w64, wf);
    }
    // every particle is a target: the first walk's groups, in its order, where it
    // had all rows (and the second set of work queues), else groups of their own
    int64_t mg = n + c->n_sys + 1;
    const bool grouped = call != 0;
    if (!grouped) AG_TRY(ag_prepare_groups(c, nullptr, n, &mg, nullptr, nullptr));
    Groups Gr{c->all_active ? (const int32_t*)nullptr : c->act_pos.as<int32_t>(), c->grp.as<int4>(),
              c->grp_hdr.as<int32_t>(), c->in_off.as<int32_t>()};
    if (!grouped) AG_TRY(order_groups(c, n, false, Gr));
    WalkOut O = make_out(c, G);
    O.dldx = dLdx;
    O.dldm = dLdm;
    O.tin = tin;
    const float th = (float)theta;
    const float e2 = (float)(eps * eps);
    int32_t* qctr = c->grp_hdr.as<int32_t>() + (grouped ? 9 : 1) * kQueueStride;
    launch_walk<AdjointPolicy, kOpen>(c, mg, Gr, O, qctr, th * th, e2, e2,
                                      (float)(1.0 / eps));
    return AG_OK;
}
