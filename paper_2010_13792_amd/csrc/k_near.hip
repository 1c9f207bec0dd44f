// k_near.hip -- sums over near neighbours, found by the tree: the distance to
// the k-th nearest particle, the Price & Monaghan lengths with Omega, their
// factors Z and their correction's acceleration.
//
// Work decomposition: a group of the gravity walk (at most 64 targets of
// neighbouring cells) is cut into runs of a few targets (8 to 16), and one
// wave takes one run.  It traverses the tree for the leaves near the run's box
// and takes their particles 64 at a time, lane = particle, position in
// registers.  For each target of the run in turn every lane forms its
// particle's FP64 distance; the ballot of the near ones compacts them into the
// target's list in LDS, in particle order.  What a near particle costs beyond
// its distance is paid on the compact lists, again with lane = entry.  (With
// lane = target and a loop over the particles, as the gravity walk does it,
// each lane meets about 900 particles for the 50 it wants, and whatever one
// lane does for a near one the whole wave sits through: 2^17 particles, k =
// 32, took 1.13 ms, by k smallest distances in registers as well as by
// binning the distances in LDS.)
#include <float.h>

#include "ag_internal.h"

namespace {

constexpr int kW = 64;
constexpr int kSCap = 384;              // stacked nodes
constexpr int kDeep = 7 * AG_MAX_LEVEL; // most nodes that taking one node at a time adds to the stack
constexpr int kLeaves = 64;             // leaves whose particles are taken together
constexpr int kWords = 1024;            // 8-byte words of the targets' lists (14 waves per CU in 160 KB)
constexpr int kMaxRun = 16;             // targets of a run at most
constexpr int kDenList = 128;           // list of one target in the density solve: 64 kept, 64 new
constexpr int kSumList = 128;           // ... in the sums
constexpr int kWalkRun = 8;             // targets of a run that take their Newton steps together

struct NearArgs {
    const int4* __restrict__ link;
    const int32_t* __restrict__ slot;    // row of an inner node's children ...
    const int4* __restrict__ child;      // ... by octant, -1 where there is none (two int4 a row)
    const NodeRec* __restrict__ rec;
    const double4* __restrict__ spos;
    const int32_t* __restrict__ perm;
    const int32_t* __restrict__ sys_root;
    const int32_t* __restrict__ act_pos;   // null: every particle is a target
    const int4* __restrict__ grp;
    const int32_t* __restrict__ hdr;
    int32_t* __restrict__ flags;
    int64_t iter_cap;
    int n;                       // particles
    double box;                  // periodic cube side (kPer instances)
    int k;                       // which neighbour
    double scale;
    double* out;                 // lengths (input order)
    double ngb;                  // density condition: sum w(r / h) = 3 ngb / 32, self included
    double hiscale;              // at this times the root's diagonal every particle's sum passes the condition
    double* omega;
    double G;
    const double* h;             // sums: lengths, Omega, Z (input order)
    const double* om;
    const double* z;
    double* zout;
    double* acc;
    bool add;                    // correction: added to acc (else written)
};

enum { kLengths, kDensity, kDensityWalk, kFactors, kCorrect };

struct NearLds {
    int stack[kSCap];
    int2 leaf[2 * kLeaves];   // first position, particles
    int before[kLeaves];      // particles of the leaves before each
    int near[2 * kW];         // particles near the run not yet passed on
    union {
        unsigned long long key[kWords];   // lengths: bits of squared distances
        double r[kWords];                 // density solve: distances
        int id[2 * kWords];               // sums: sorted positions
    };
};

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ double lane_f64(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int l) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

// ---- the cubic spline with support 1 for the Price & Monaghan terms ----
// w(u) and w'(u) with W(r, h) = 8/(pi h^3) w(r/h); and -h^2 dphi/dh =
// psi(u) + u^2 F(u), where phi(r, h) = psi(r/h)/h is the potential of the
// spread unit mass and F = h^3 f its force kernel (the 1/u terms cancel):
//   16 u^2 - 48 u^4 + 192/5 u^5 - 14/5               (u < 1/2)
//   32 u^2 - 64 u^3 + 48 u^4 - 64/5 u^5 - 16/5        (1/2 <= u < 1), 0 beyond.
__device__ __forceinline__ double m4_w(double u) {
    return u < 0.5 ? 1.0 + u * u * (-6.0 + 6.0 * u) : (u < 1.0 ? 2.0 * (1.0 - u) * (1.0 - u) * (1.0 - u) : 0.0);
}
__device__ __forceinline__ double m4_wp(double u) {
    return u < 0.5 ? u * (-12.0 + 18.0 * u) : (u < 1.0 ? -6.0 * (1.0 - u) * (1.0 - u) : 0.0);
}
__device__ __forceinline__ double m4_dphi(double u) {
    const double u2 = u * u;
    return u < 0.5 ? u2 * (16.0 + u2 * (-48.0 + u * (192.0 / 5.0))) - 14.0 / 5.0
                   : (u < 1.0 ? u2 * (32.0 + u * (-64.0 + u * (48.0 - u * (64.0 / 5.0)))) - 16.0 / 5.0 : 0.0);
}

// One step of safeguarded Newton for S(h) = target with S increasing in h:
// s = S(h), sd = sum u w'(u) (so dS/dh = -sd / h).  The bracket [lo, hi]
// shrinks to the side of h the sign of S - target gives; the Newton point is
// taken when it falls strictly inside the bracket (growing h at most
// twofold), else twice h while h is below the root and the sum has no slope
// there, else the bracket's midpoint.
// Returns false once the length is settled, leaving hn = h: the step or the
// bracket below 2e-14 h (above the rounding noise of a sum of many terms,
// which keeps a tighter test from ever closing; Newton's last step had
// already brought h to that noise).
__device__ __forceinline__ bool pm_newton(double s, double sd, double target, double h, double& lo, double& hi,
                                          double& hn) {
    if (s < target) lo = h; else hi = h;
    hn = h;
    if (hi - lo <= 2e-14 * hi) return false;
    double t = sd < 0.0 ? h + (s - target) * h / sd : -1.0;
    // a settled Newton step is tested first: below an ulp it returns h
    // itself, which the bracket test would take for a failed step
    if (sd < 0.0 && fabs(t - h) <= 2e-14 * h) return false;
    if (s < target && t > 2.0 * h) t = 2.0 * h;
    if (!(t > lo && t < hi)) t = s < target && sd == 0.0 && 2.0 * h < hi ? 2.0 * h : 0.5 * (lo + hi);
    hn = t;
    return true;
}

// a run's box, rounded outward to FP32
struct NearBox {
    float lox, loy, loz, hix, hiy, hiz;
};
__device__ __forceinline__ float f_dn(double d) {
    const float f = (float)d;
    return (double)f > d ? nextafterf(f, -FLT_MAX) : f;
}
__device__ __forceinline__ float f_upr(double d) {
    const float f = (float)d;
    return (double)f < d ? nextafterf(f, FLT_MAX) : f;
}
__device__ __forceinline__ NearBox near_box(double x, double y, double z) {
    NearBox b;
    b.lox = f_dn(ag_wave_min_f64(x)); b.loy = f_dn(ag_wave_min_f64(y)); b.loz = f_dn(ag_wave_min_f64(z));
    b.hix = f_upr(ag_wave_max_f64(x)); b.hiy = f_upr(ag_wave_max_f64(y)); b.hiz = f_upr(ag_wave_max_f64(z));
    return b;
}

// Squared gap of a node's box and the run's.  Both boxes are rounded
// outward, their gaps are exact in FP64, and the caller's relative margin
// covers the rounding of the squares: a node farther than R holds no particle
// at a computed d^2 <= R^2.  Periodic: per axis the gap between two arcs of a
// circle of length L, the centres' distance taken the short way round less
// both half widths (every node lies inside the box, so no arc crosses the cut).
template <bool kPer>
__device__ __forceinline__ double axis_gap(float lo, float hi, float glo, float ghi, double box) {
    if (!kPer) return fmax(fmax((double)lo - ghi, (double)glo - hi), 0.0);
    double c = fabs(0.5 * ((double)lo + hi) - 0.5 * ((double)glo + ghi));
    c = fmin(c, box - c);
    return fmax(c - 0.5 * (((double)hi - lo) + ((double)ghi - glo)), 0.0);
}
template <bool kPer>
__device__ __forceinline__ double box_gap2(const NearBox& g, const float4 lo, const float4 hi, double box) {
    const double gx = axis_gap<kPer>(lo.x, hi.x, g.lox, g.hix, box);
    const double gy = axis_gap<kPer>(lo.y, hi.y, g.loy, g.hiy, box);
    const double gz = axis_gap<kPer>(lo.z, hi.z, g.loz, g.hiz, box);
    return gx * gx + gy * gy + gz * gz;
}

// Squared gap of a particle and the run's box (periodic: at the box's own
// outward rounding a point is an arc of no width).
template <bool kPer>
__device__ __forceinline__ double point_gap2(const NearBox& g, const double4& p, double box) {
    double d[3];
    const double x[3] = {p.x, p.y, p.z};
    const float lo[3] = {g.lox, g.loy, g.loz}, hi[3] = {g.hix, g.hiy, g.hiz};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (!kPer) {
            d[c] = fmax(fmax(x[c] - hi[c], lo[c] - x[c]), 0.0);
        } else {
            const double q = fabs(x[c] - 0.5 * ((double)lo[c] + hi[c]));
            d[c] = fmax(fmin(q, box - q) - 0.5 * ((double)hi[c] - lo[c]), 0.0);
        }
    }
    return d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
}

// d^2 = (dx^2 + dy^2) + dz^2, d = p - x, each operation rounded once (hipcc
// contracts a * b + c into one fma by default: not here).  Periodic: every
// difference goes to its nearest image first, d - L rint(d / L) (the division
// correctly rounded).
template <bool kPer>
__device__ __forceinline__ double dist2(const double4& p, double x, double y, double z, double L) {
#pragma clang fp contract(off)
    double dx = p.x - x, dy = p.y - y, dz = p.z - z;
    if (kPer) {
        dx = dx - L * rint(dx / L);
        dy = dy - L * rint(dy / L);
        dz = dz - L * rint(dz / L);
    }
    return (dx * dx + dy * dy) + dz * dz;
}

// One wave's run of targets: lane l holds target l % n (its own up to n).
struct Run {
    int n, lane, p;
    double x, y, z, m;
    int64_t row;
};

// f(pk, p, valid): the particles of every leaf within R of the run's box (or,
// with kNodeH, within the node's largest length), 64 at a time, one per lane.
// A stack of nodes in LDS: each step tests as many as there are lanes and
// pushes all children of those it opens, read from the node's child row (the
// pre-order skip links alone would make a step per sibling: 32 steps instead
// of 16 at 2^16 particles).  Leaves are gathered 64 at a time; a lane finds its
// particle among them by bisecting their running count, and those outside R of
// the run's box, four in ten, are left out.  The order depends on the tree and
// the run alone.
template <bool kPer, bool kNodeH, class F>
__device__ __forceinline__ void each_near(NearLds& S, const NearArgs& A, const NearBox& gb, double R2, int root,
                                          int lane, F f) {
    int sp = 1, nl = 0, nn = 0;  // nodes stacked, leaves gathered, particles near the run (uniform)
    if (lane == 0) S.stack[0] = root;
    wave_sync();
    auto pass_on = [&](int base, int n) {
        const bool valid = lane < n;
        const int pk = valid ? S.near[base + lane] : -1;
        const double4 p = valid ? A.spos[pk] : make_double4(0.0, 0.0, 0.0, 0.0);
        f(pk, p, valid);
        wave_sync();
    };
    auto take_leaves = [&](int base, int n) {
        const int2 l = lane < n ? S.leaf[base + lane] : make_int2(0, 0);
        const int incl = ag_wave_incl_scan(l.y);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        S.before[lane] = incl - l.y;
        wave_sync();
        for (int c = 0; c < total; c += kW) {
            int j = 0;           // the last leaf that starts at or before the lane's particle
#pragma unroll
            for (int b = kLeaves / 2; b > 0; b >>= 1) j += S.before[j + b] <= c + lane ? b : 0;
            bool in = c + lane < total;
            const int pk = S.leaf[base + j].x + c + lane - S.before[j];
            if (in) {
                const double4 p = A.spos[pk];
                double r2 = R2;
                if (kNodeH) {
                    const double hk = A.h[A.perm[pk]];
                    r2 = fmax(r2, hk * hk);
                }
                in = point_gap2<kPer>(gb, p, A.box) <= r2 * (1.0 + 1e-12);
            }
            const uint64_t m = __ballot(in);
            if (in) S.near[nn + ag_prefix_count(m)] = pk;
            nn += __popcll(m);
            wave_sync();
            if (nn >= kW) {
                nn -= kW;
                pass_on(nn, kW);
            }
        }
        wave_sync();
    };
    int64_t iters = 0;
    while (sp > 0) {
        // (every step tests a node; the cap only guards against a corrupt tree)
        if (++iters > A.iter_cap) {
            if (lane == 0) atomicOr(A.flags, AGF_INTERNAL);
            break;
        }
        // as many nodes as lanes, as long as all their children fit and taking
        // them one by one from there on does
        int m = (kSCap - kDeep - sp) / 7;
        m = m < 1 ? 1 : (m > kW ? kW : m);
        m = m < sp ? m : sp;
        sp -= m;
        bool leaf = false, open = false;
        int4 L = make_int4(0, 0, 0, 0);
        int4 c0 = make_int4(-1, -1, -1, -1), c1 = c0;
        if (lane < m) {
            const int a = S.stack[sp + lane];
            L = A.link[a];
            const float4 lo = A.rec[a].lo, hi = A.rec[a].hi;
            const int row = A.slot[a];
            double r2 = R2;
            if (kNodeH) {
                const double hn = (double)lo.w * (1.0 + 1e-6);   // covers the float rounding of each length
                r2 = fmax(r2, hn * hn);
            }
            if (box_gap2<kPer>(gb, lo, hi, A.box) <= r2 * (1.0 + 1e-12)) {
                leaf = (L.w & 0x100) != 0;
                open = !leaf;
                if (open) {
                    c0 = A.child[2 * (int64_t)row];
                    c1 = A.child[2 * (int64_t)row + 1];
                }
            }
        }
        wave_sync();
        const uint64_t lm = __ballot(leaf);
        if (lm) {
            if (leaf) S.leaf[nl + ag_prefix_count(lm)] = make_int2(L.y, L.z);
            nl += __popcll(lm);
        }
        if (__ballot(open)) {
            const int ch[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            int nch = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) nch += ch[k] >= 0;
            const int incl = ag_wave_incl_scan(nch);
            int at = sp + incl - nch;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (ch[k] >= 0) S.stack[at++] = ch[k];
            sp += __builtin_amdgcn_readlane(incl, 63);
        }
        wave_sync();
        if (nl >= kLeaves) {
            nl -= kLeaves;
            take_leaves(nl, kLeaves);
        }
    }
    if (nl > 0) take_leaves(0, nl);
    if (nn > 0) pass_on(0, nn);
}

// the next one, when the target with the fewest found c of k neighbours
__device__ __forceinline__ double next_radius(double R, double c, double k) {
    return R * fmin(fmax(1.15 * cbrt(k / fmax(c, 0.5)), 1.15), 4.0);
}

__device__ __forceinline__ unsigned long long key_of(double d2) { return (unsigned long long)__double_as_longlong(d2); }

// The k-th smallest of the n keys e0 (lane < 64), e1 (lane + 64; ~0 where
// there is none), all below `top`, by halving a range of values and counting
// ballots until one key is left in it (or the range is one value).
__device__ __forceinline__ unsigned long long kth_key(unsigned long long e0, unsigned long long e1, int k, int n,
                                                      unsigned long long top) {
    typedef unsigned long long u64;
    auto below = [&](u64 v) { return __popcll(__ballot(e0 < v)) + __popcll(__ballot(e1 < v)); };
    u64 lo = 0, hi = top;
    int clo = 0, chi = n;
    if (top > (1ull << 54)) {            // four octaves below the top, where it nearly always lies
        const u64 v = top - (1ull << 54);
        const int c = below(v);
        if (c < k) {
            lo = v;
            clo = c;
        } else {
            hi = v;
            chi = c;
        }
    }
    while (chi - clo > 1 && hi - lo > 1) {
        const u64 v = lo + ((hi - lo) >> 1);
        const int c = below(v);
        if (c < k) {
            lo = v;
            clo = c;
        } else {
            hi = v;
            chi = c;
        }
    }
    if (hi - lo <= 1) return lo;
    const u64 b0 = __ballot(e0 >= lo && e0 < hi);
    if (b0) return lane_u64(e0, __builtin_ctzll(b0));
    return lane_u64(e1, __builtin_ctzll(__ballot(e1 >= lo && e1 < hi)));
}

// A first radius for `k` neighbours of a run: 1.25 times the radius that holds
// them at a uniform density whose particles are as far apart as the median
// pair of neighbours in key order, from 8 positions before the run to 8 after
// it (near the largest wanted distance of a run on spheres and clumps alike; a
// box about the targets takes in the jumps of the key order, and one run with
// a far too large radius took as long as the whole launch).  A wrong guess
// costs another traversal, never the result.
template <bool kPer>
__device__ __forceinline__ double first_radius(const NearArgs& A, int p0, int n, int lane, double k, double diag) {
    const int w0 = p0 > 8 ? p0 - 8 : 0, w1 = p0 + n + 8 < A.n ? p0 + n + 8 : A.n;
    const bool pair = w0 + lane + 1 < w1;
    unsigned long long key = ~0ull;
    if (pair) {
        const double4 a = A.spos[w0 + lane], b = A.spos[w0 + lane + 1];
        key = key_of(dist2<kPer>(b, a.x, a.y, a.z, A.box));
    }
    const int m = __popcll(__ballot(pair));
    const double least = diag * 0x1p-20;
    if (m == 0) return least;
    const double d2 = __longlong_as_double((long long)kth_key(key, ~0ull, (m + 1) / 2, m, ~0ull - 1));
    return fmax(1.25 * cbrt(3.0 * k / (4.0 * 3.14159265358979)) * sqrt(d2), least);
}

// ---- the k-th smallest distance of every target ----
// A target's list holds k + 64 keys; when it would overflow it is cut to the
// k smallest, and only nearer particles are taken from there on.
template <bool kPer>
__device__ __forceinline__ void find_lengths(NearLds& S, const NearArgs& A, const Run& t, const NearBox& gb,
                                             int root, double diag, double R) {
    typedef unsigned long long u64;
    const int lane = t.lane, k = A.k, cap = k + kW;
    u64 bound = 0;
    int cnt = 0;                 // lane l < n: target l's list
    for (;;) {
        const bool all = !(R < diag);
        if (all) R = diag;
        const double R2 = R * R;
        bound = key_of(R2) + 1;  // keys below it are wanted
        cnt = 0;
        each_near<kPer, false>(S, A, gb, R2, root, lane, [&](int pk, const double4& p, bool valid) {
            for (int j = 0; j < t.n; ++j) {
                const double tx = lane_f64(t.x, j), ty = lane_f64(t.y, j), tz = lane_f64(t.z, j);
                const int tp = __builtin_amdgcn_readlane(t.p, j);
                const u64 bj = lane_u64(bound, j);
                int n = __builtin_amdgcn_readlane(cnt, j);
                const u64 key = key_of(dist2<kPer>(p, tx, ty, tz, A.box));
                bool hit = valid && pk != tp && key < bj;
                u64 m = __ballot(hit);
                if (m == 0) continue;
                u64* L = S.key + j * cap;
                if (n + __popcll(m) > cap) {
                    // cut to the k smallest: those below the k-th, and its equals
                    const u64 e0 = lane < n ? L[lane] : ~0ull, e1 = lane + kW < n ? L[lane + kW] : ~0ull;
                    const u64 kk = kth_key(e0, e1, k, n, bj + 1);   // (an earlier cut kept the bound itself)
                    const u64 m0 = __ballot(e0 < kk), m1 = __ballot(e1 < kk);
                    const int c0 = __popcll(m0), c1 = __popcll(m1);
                    wave_sync();
                    if (e0 < kk) L[ag_prefix_count(m0)] = e0;
                    if (e1 < kk) L[c0 + ag_prefix_count(m1)] = e1;
                    if (lane < k - c0 - c1) L[c0 + c1 + lane] = kk;
                    wave_sync();
                    n = k;
                    if (lane == j) bound = kk;
                    hit = hit && key < kk;
                    m = __ballot(hit);
                }
                if (hit) L[n + ag_prefix_count(m)] = key;
                if (lane == j) cnt = n + __popcll(m);
            }
        });
        const bool few = lane < t.n && cnt < k;
        if (__ballot(few) == 0) break;
        if (all) {               // (k < n: cannot be)
            if (lane == 0) atomicOr(A.flags, AGF_INTERNAL);
            break;
        }
        R = next_radius(R, ag_wave_min_f64(few ? (double)cnt : (double)k), k);
    }
    wave_sync();
    double d2 = 0.0;
    for (int j = 0; j < t.n; ++j) {
        const int n = __builtin_amdgcn_readlane(cnt, j);
        const u64* L = S.key + j * cap;
        const u64 e0 = lane < n ? L[lane] : ~0ull, e1 = lane + kW < n ? L[lane + kW] : ~0ull;
        const u64 kk = kth_key(e0, e1, k, n, lane_u64(bound, j) + 1);
        if (lane == j) d2 = __longlong_as_double((long long)kk);
    }
    if (lane < t.n) A.out[t.row] = A.scale * sqrt(d2);
}

// ---- lengths on the density condition, with Omega ----
// h with S(h) = 1 + sum_j w(r_j / h) = 3 N / 32 (self counted as 1), by
// pm_newton; Omega = -(32 / (9 N)) sum_j u_j w'(u_j) at h.

// Solves for the n distances at L in the bracket [0, hi].  kShort: S(hi) falls
// short.  kOpenRoot: no step settled, as where so many particles coincide that S
// passes the target at every h; h is then the smallest length known to pass.
// sd: the sum of u w'(u) at the solution.
enum { kShort, kSolved, kOpenRoot };
__device__ __forceinline__ int solve_list(const double* L, int n, int lane, double target, double hi, double& h,
                                           double& sd) {
    auto sums = [&](double hh) {
        const double hinv = 1.0 / hh;
        double a = 0.0, b = 0.0;
        for (int e = lane; e < n; e += kW) {
            const double u = L[e] * hinv;
            if (u < 1.0) {
                a += m4_w(u);
                b += u * m4_wp(u);
            }
        }
        sd = ag_wave_sum_f64(b);
        return 1.0 + ag_wave_sum_f64(a);
    };
    const double shi = sums(hi);
    h = hi;
    if (!(shi >= target)) return kShort;
    double lo = 0.0;
    // start where S would meet the target if the neighbours filled the ball
    // uniformly (S - 1 growing as h^3)
    if (shi > target) h = fmin(hi, hi * cbrt((target - 1.0) / (shi - 1.0)));
    for (int it = 0; it < 200; ++it) {
        const double s = sums(h);
        double hn;
        if (!pm_newton(s, sd, target, h, lo, hi, hn)) return kSolved;
        h = hn;
    }
    h = hi;
    return kOpenRoot;
}

// The targets' distances below R (or, all: any distance) into lists of `cap`,
// and their solutions.  When a list would overflow, its own solution bounds
// the target's (more particles only raise S) and what lies beyond is dropped;
// a target that keeps more than cap - 64 after that is left out (longer, with
// its bound in rmax).  A target whose sum falls short at R is not done.
struct Density {
    double h, sd, rmax;          // lane l < n: target l's
    int cnt;
    bool done, longer;
};
__device__ __forceinline__ void density_pass(NearLds& S, const NearArgs& A, const Run& t, const NearBox& gb, int root,
                                             double diag, double R, bool all, int cap, Density& D) {
    const int lane = t.lane;
    const double target = 3.0 * A.ngb / 32.0;
    D.rmax = all ? DBL_MAX : R;
    D.cnt = 0;
    D.longer = false;
    each_near<false, false>(S, A, gb, R * R, root, lane, [&](int pk, const double4& p, bool valid) {
        for (int j = 0; j < t.n; ++j) {
            if (__builtin_amdgcn_readlane((int)(D.done || D.longer), j)) continue;
            const double tx = lane_f64(t.x, j), ty = lane_f64(t.y, j), tz = lane_f64(t.z, j);
            const int tp = __builtin_amdgcn_readlane(t.p, j);
            const double rj = lane_f64(D.rmax, j);
            int n = __builtin_amdgcn_readlane(D.cnt, j);
            const double r2 = dist2<false>(p, tx, ty, tz, 0.0);
            bool hit = valid && pk != tp && r2 < rj * rj;
            uint64_t m = __ballot(hit);
            if (m == 0) continue;
            double* L = S.r + j * cap;
            if (n + __popcll(m) > cap) {
                double hs, ds;
                const double hi = all && !(rj < DBL_MAX) ? A.hiscale * diag : rj;
                if (solve_list(L, n, lane, target, hi, hs, ds) == kShort) hs = hi;
                hs = fmin(rj, hs * (1.0 + 1e-12));
                int kept = 0;
                for (int e = 0; e < n; e += kW) {
                    const double r = e + lane < n ? L[e + lane] : DBL_MAX;
                    const bool keep = r < hs;
                    const uint64_t km = __ballot(keep);
                    wave_sync();
                    if (keep) L[kept + ag_prefix_count(km)] = r;
                    kept += __popcll(km);
                    wave_sync();
                }
                n = kept;
                if (lane == j) D.rmax = hs;
                if (n > cap - kW) {
                    if (lane == j) D.longer = true;
                    continue;
                }
                hit = hit && r2 < hs * hs;
                m = __ballot(hit);
            }
            if (hit) L[n + ag_prefix_count(m)] = sqrt(r2);
            if (lane == j) D.cnt = n + __popcll(m);
        }
    });
    wave_sync();
    for (int j = 0; j < t.n; ++j) {
        if (__builtin_amdgcn_readlane((int)(D.done || D.longer), j)) continue;
        // (every particle a candidate: any length may be taken)
        const double rj = lane_f64(D.rmax, j), hi = all && !(rj < DBL_MAX) ? A.hiscale * diag : rj;
        double hj, ds;
        const int how = solve_list(S.r + j * cap, __builtin_amdgcn_readlane(D.cnt, j), lane, target, hi, hj, ds);
        if (lane == j) {
            D.h = hj;
            D.sd = ds;
            D.done = how != kShort || all;
            // (with every particle listed the sum does not fall short)
            if (how == kOpenRoot || (how == kShort && all)) atomicOr(A.flags, AGF_PMOPEN);
        }
    }
}

// Newton steps of the run's targets (M at most) together, from the lanes' h on, a
// traversal each: every lane adds its particles' terms for each target that still
// moves.
template <int M>
__device__ __forceinline__ void walk_density(NearLds& S, const NearArgs& A, const Run& t, const NearBox& gb, int root,
                                             double diag, double& h, double& sd) {
    const int lane = t.lane;
    const double target = 3.0 * A.ngb / 32.0;
    double lo = 0.0, hi = A.hiscale * diag, hn = h;
    bool moving = lane < t.n;
    for (int it = 0; __ballot(moving) != 0; ++it) {
        h = hn;
        const double h2 = moving ? h * h : 0.0, hinv = 1.0 / h;
        double a[M], b[M];
#pragma unroll
        for (int j = 0; j < M; ++j) a[j] = b[j] = 0.0;
        each_near<false, false>(S, A, gb, ag_wave_max_f64(h2), root, lane, [&](int pk, const double4& p, bool valid) {
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const double hj2 = lane_f64(h2, j);
                if (!(hj2 > 0.0)) continue;   // settled, or no target
                const int tp = __builtin_amdgcn_readlane(t.p, j);
                const double r2 = dist2<false>(p, lane_f64(t.x, j), lane_f64(t.y, j), lane_f64(t.z, j), 0.0);
                if (valid && pk != tp && r2 < hj2) {
                    const double u = sqrt(r2) * lane_f64(hinv, j);
                    a[j] += m4_w(u);
                    b[j] += u * m4_wp(u);
                }
            }
        });
        double s = 0.0, sn = 0.0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const double sa = ag_wave_sum_f64(a[j]), sb = ag_wave_sum_f64(b[j]);
            s = lane == j ? 1.0 + sa : s;
            sn = lane == j ? sb : sn;
        }
        if (moving) {
            sd = sn;
            moving = pm_newton(s, sd, target, h, lo, hi, hn);
            if (moving && it == 400) {
                atomicOr(A.flags, AGF_PMOPEN);
                moving = false;
            }
        }
    }
}

// Every target of the run in lists of 128; those that need more, one by one in
// a list of all the words; those that need more than that take Newton steps
// with a traversal each.
__device__ __forceinline__ void solve_density(NearLds& S, const NearArgs& A, const Run& t, const NearBox& gb,
                                              int root, double diag, double R, double& h_out, double& sd_out) {
    const int lane = t.lane;
    Density D;
    D.h = D.sd = 0.0;
    D.done = lane >= t.n;
    for (;;) {
        const bool all = !(R < diag);
        if (all) R = diag;
        density_pass(S, A, t, gb, root, diag, R, all, kDenList, D);
        if (__ballot(!D.done && !D.longer) == 0 || all) break;
        R = next_radius(R, ag_wave_min_f64(D.done || D.longer ? A.ngb : (double)D.cnt), A.ngb);
    }
    for (uint64_t left = __ballot(D.longer && lane < t.n); left; left &= left - 1) {
        const int j = __builtin_ctzll(left);
        Run o = t;
        o.n = 1;
        o.x = lane_f64(t.x, j); o.y = lane_f64(t.y, j); o.z = lane_f64(t.z, j);
        o.p = __builtin_amdgcn_readlane(t.p, j);
        const NearBox ob = near_box(o.x, o.y, o.z);
        Density E;
        E.h = E.sd = 0.0;
        E.done = lane > 0;
        double Rj = lane_f64(D.rmax, j);   // its bound, or the radius searched so far
        for (;;) {
            const bool all = !(Rj < diag);
            if (all) Rj = diag;
            density_pass(S, A, o, ob, root, diag, Rj, all, kWords, E);
            if (__ballot(!E.done && !E.longer) == 0 || all) break;
            Rj = next_radius(Rj, lane_f64((double)E.cnt, 0), A.ngb);
        }
        double h = lane_f64(E.h, 0), sd = lane_f64(E.sd, 0);
        if (__builtin_amdgcn_readlane((int)E.longer, 0)) {
            double hw = lane_f64(E.rmax, 0), sw = 0.0;
            walk_density<1>(S, A, o, ob, root, diag, hw, sw);
            h = lane_f64(hw, 0);
            sd = lane_f64(sw, 0);
        }
        if (lane == j) {
            D.h = h;
            D.sd = sd;
        }
    }
    h_out = D.h;
    sd_out = D.sd;
}

// ---- Price & Monaghan sums over the pairs inside a kernel support ----
// Factors:    Z_i = -(G m_i h_i^2 / (6 C Omega_i)) sum_{j != i, r < h_i} m_j
//             (psi + u^2 F)(r / h_i), C = 3 N / (4 pi) (number density n h^3);
// correction: a_i = -(1 / m_i) sum_{j != i} [Z_i W'(r, h_i) + Z_j W'(r, h_j)] d / r
//             over r < max(h_i, h_j), W'(r, h) = 8 / (pi h^4) w'(r / h), d = x_j - x_i.
// The lengths are the per-particle softening lengths the tree was built with
// (FP64, input order); each node's largest one (lo.w, a float) bounds the
// sources' supports in the correction.  Coincident pairs add nothing to it
// (w'(0) = 0).  A full list is summed and emptied.
template <int kMode>
__device__ __forceinline__ void sum_pairs(NearLds& S, const NearArgs& A, const Run& t, const NearBox& gb, int root) {
    const int lane = t.lane;
    const double h = A.h[t.row], zi = kMode == kCorrect ? A.z[t.row] : 0.0;
    const double R2 = ag_wave_max_f64(h * h);
    constexpr double k8pi = 8.0 / 3.14159265358979323846;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;   // lane l < n: target l's sums
    int cnt = 0;
    auto sum_list = [&](int j, int n) {
        const double tx = lane_f64(t.x, j), ty = lane_f64(t.y, j), tz = lane_f64(t.z, j);
        const double hj = lane_f64(h, j), zj = lane_f64(zi, j);
        const int* L = S.id + j * kSumList;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        for (int e = lane; e < n; e += kW) {
            const int pk = L[e];
            const double4 p = A.spos[pk];
            const double dx = p.x - tx, dy = p.y - ty, dz = p.z - tz;
            const double r = sqrt(dx * dx + dy * dy + dz * dz);
            if (kMode == kFactors) {
                a0 += p.w * m4_dphi(r / hj);
            } else {
                const int64_t row = A.perm[pk];
                const double hs = A.h[row], zs = A.z[row];
                const double ht4 = (hj * hj) * (hj * hj), hs4 = (hs * hs) * (hs * hs);
                const double c = k8pi * (zj * m4_wp(r / hj) / ht4 + zs * m4_wp(r / hs) / hs4) / r;
                a0 += c * dx;
                a1 += c * dy;
                a2 += c * dz;
            }
        }
        a0 = ag_wave_sum_f64(a0);
        if (kMode == kCorrect) {
            a1 = ag_wave_sum_f64(a1);
            a2 = ag_wave_sum_f64(a2);
        }
        if (lane == j) {
            s0 += a0;
            s1 += a1;
            s2 += a2;
            cnt = 0;
        }
    };
    each_near<false, kMode == kCorrect>(S, A, gb, R2, root, lane, [&](int pk, const double4& p, bool valid) {
        const double hk = kMode == kCorrect && valid ? A.h[A.perm[pk]] : 0.0;
        for (int j = 0; j < t.n; ++j) {
            const double tx = lane_f64(t.x, j), ty = lane_f64(t.y, j), tz = lane_f64(t.z, j), hj = lane_f64(h, j);
            const int tp = __builtin_amdgcn_readlane(t.p, j);
            int n = __builtin_amdgcn_readlane(cnt, j);
            const double dx = p.x - tx, dy = p.y - ty, dz = p.z - tz;
            const double r2 = dx * dx + dy * dy + dz * dz;
            bool hit = r2 < hj * hj;
            if (kMode == kCorrect) hit = r2 > 0.0 && (hit || r2 < hk * hk);
            hit = hit && valid && pk != tp;
            const uint64_t m = __ballot(hit);
            if (m == 0) continue;
            if (n + __popcll(m) > kSumList) {
                sum_list(j, n);
                n = 0;
                wave_sync();
            }
            if (hit) S.id[j * kSumList + n + ag_prefix_count(m)] = pk;
            if (lane == j) cnt = n + __popcll(m);
        }
    });
    wave_sync();
    for (int j = 0; j < t.n; ++j) sum_list(j, __builtin_amdgcn_readlane(cnt, j));
    if (lane >= t.n) return;
    const int64_t row = t.row;
    if (kMode == kFactors) {
        const double C = 3.0 * A.ngb / (4.0 * 3.14159265358979323846);
        A.zout[row] = -(A.G * t.m * h * h / (6.0 * C * A.om[row])) * s0;
    } else {
        const double a[3] = {s0, s1, s2};
        for (int c = 0; c < 3; ++c) {
            const double v = -a[c] / t.m;
            A.acc[3 * row + c] = A.add ? A.acc[3 * row + c] + v : v;
        }
    }
}

// Persistent waves.  Every group has `cuts` places; it is cut into as few runs
// of at most `run` targets as hold them, of equal length, and its other places
// are empty.  An eighth of the places (neighbouring groups) belongs to the
// waves of one XCD, which take them in turn, each wave another place of its group
// every time (where their number is a multiple of `cuts` it would be the same one,
// and the waves of the last places idle: 10^6 particles with k = 32 in runs of 10,
// five of seven places used, 3.01 ms, now 2.30): with a queue, the pops of one
// counter, 0.2 us each, took longer than the runs (2^20 particles: 4.0 ms).
template <int kMode, bool kPer>
__global__ void __launch_bounds__(kW, 4) k_near(NearArgs A, int run, int cuts) {
    __shared__ NearLds S;
    const int n_groups = A.hdr[0];
    const int lane = ag_lane();
    const int xcd = (int)(blockIdx.x & 7);
    const int g0 = (int)((int64_t)n_groups * xcd / 8), g1 = (int)((int64_t)n_groups * (xcd + 1) / 8);
    const int waves = (int)(gridDim.x >> 3), w = (int)(blockIdx.x >> 3);
    // (the steps of all waves alike: a group's places stay one to a wave)
    const int add_g = waves / cuts, add_c = waves % cuts != 0 ? waves % cuts : 1, carry = waves % cuts != 0;
    int g = g0 + w / cuts - add_g, c = w % cuts - add_c;
    for (;;) {
        g += add_g;
        c += add_c;
        if (c >= cuts) {
            c -= cuts;
            g += carry;
        }
        if (g >= g1) break;
        const int4 gd = A.grp[g];
        const int count = gd.y, nc = (count + run - 1) / run;
        const int root = A.sys_root[gd.z];
        if (c >= nc || root < 0) continue;
        const int t0 = count * c / nc, t1 = count * (c + 1) / nc;
        Run t;
        t.lane = lane;
        t.n = t1 - t0;
        const int first = gd.x + t0, slot = first + lane % t.n;
        t.p = A.act_pos ? A.act_pos[slot] : slot;
        t.row = A.perm[t.p];
        const double4 xi = A.spos[t.p];
        t.x = xi.x; t.y = xi.y; t.z = xi.z; t.m = xi.w;
        const NearBox gb = near_box(xi.x, xi.y, xi.z);
        if constexpr (kMode == kFactors || kMode == kCorrect) {
            sum_pairs<kMode>(S, A, t, gb, root);
        } else {
            // no two particles are farther apart (a margin for the rounding; not 0)
            const float4 lo = A.rec[root].lo, hi = A.rec[root].hi;
            const double ex = (double)hi.x - lo.x, ey = (double)hi.y - lo.y, ez = (double)hi.z - lo.z;
            const double diag = fmax(1.001 * sqrt(ex * ex + ey * ey + ez * ez), DBL_MIN);
            // (every particle is a target: positions are slots)
            // (few neighbours vary more: 14 % of the targets have none in the radius
            // that holds two on average, and nearly every run of 15 took a second
            // traversal for its one neighbour; 10^6 uniform ones, k = 1, 1.53 ms, now
            // 1.23, k = 4 1.58 and 1.40; from k = 13 on twice k is more)
            const double few = (A.k + 3.5 * sqrt((double)A.k)) / (1.25 * 1.25 * 1.25);
            const double R = first_radius<kPer>(A, first, t.n, lane, kMode == kLengths ? fmax(A.k, few) : A.ngb, diag);
            if constexpr (kMode == kLengths) {
                find_lengths<kPer>(S, A, t, gb, root, diag, R);
            } else {
                double h = R / 1.25, sd = 0.0;
                if constexpr (kMode == kDensity) solve_density(S, A, t, gb, root, diag, R, h, sd);
                else walk_density<kWalkRun>(S, A, t, gb, root, diag, h, sd);
                if (lane < t.n) {
                    A.out[t.row] = h;
                    A.omega[t.row] = -(32.0 / (9.0 * A.ngb)) * sd;
                }
            }
        }
        wave_sync();
    }
}

NearArgs near_args(ag_ctx* c) {
    NearArgs A{};
    A.link = c->nd_link.as<int4>();
    A.slot = c->nd_slot.as<int32_t>();
    A.child = c->child.as<int4>();
    A.rec = c->nd_rec.as<NodeRec>();
    A.spos = c->spos.as<double4>();
    A.perm = c->perm.as<int32_t>();
    A.sys_root = c->sys_root.as<int32_t>();
    A.act_pos = c->all_active ? nullptr : c->act_pos.as<int32_t>();
    A.grp = c->grp.as<int4>();
    A.hdr = c->grp_hdr.as<int32_t>();
    A.flags = c->dflags.as<int32_t>();
    A.iter_cap = c->max_nodes + c->n + 1024;
    A.n = (int)c->n;
    A.box = c->tree_box;
    A.scale = 1.0;
    return A;
}

// As many waves per CU as their LDS lets reside; runs of at most `run` targets
// (their lists fill a wave's share of LDS), shorter where that leaves waves
// idle: two runs a wave, but two targets a run at least, whose traversals are
// nearly one target's each (5000 particles in a halo: one run of 8 that needed
// long lists held the launch for 1.2 ms).
template <int kMode, bool kPer>
void launch_near(ag_ctx* c, const NearArgs& A, int64_t max_groups, int64_t targets, int run) {
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
    int64_t blocks = (int64_t)cus * (160 * 1024 / (int)sizeof(NearLds));
    const int64_t fair = targets / (2 * blocks) + 1;
    if (run > kMaxRun) run = kMaxRun;
    if (run > fair) run = fair > 2 ? (int)fair : 2;
    const int cuts = (AG_GROUP + run - 1) / run;
    if (blocks > max_groups * cuts) blocks = max_groups * cuts;
    blocks = (blocks + 7) / 8 * 8;   // as many for each XCD
    PhaseScope phase(c, AG_PHASE_NEIGHBOUR);
    hipLaunchKernelGGL((k_near<kMode, kPer>), dim3((unsigned)blocks), dim3(kW), 0, c->stream, A, run, cuts);
}

}  // namespace

// Measured (us; before: lists of k distances in registers, sums on one lane per
// target): k = 32 on a uniform sphere of 2^17, 1130 -> 364, of 10^6, 3510 ->
// 2300 (k = 8 to 16 of 10^6 2 to 5% slower); lengths and Omega at n_ngb = 32,
// 2^16: 2510 -> 418, 10^6: 15 700 -> 4400; Z, 2^16: 542 -> 142, 10^6: 1490 ->
// 1390; correction, 2^16: 697 -> 175, 10^6: 2270 -> 1950.  With long supports
// and many particles the sums are slower than one lane per target was (10^6,
// n_ngb = 400: Z 4100 -> 5300, correction 8300 -> 12 100), the lengths faster by
// more (lengths, Z and correction 53 500 -> 47 900).  Bound by instruction
// issue: of a run's time about a third each goes to the traversal (16 steps),
// the distances and the lists.

// distance of every particle to its k-th nearest other particle
int ag_launch_knn(ag_ctx* c, int32_t k, double scale, double* h_out) {
    int64_t mg = 0;
    AG_TRY(ag_prepare_groups(c, nullptr, c->n, &mg, nullptr, nullptr));
    NearArgs A = near_args(c);
    A.k = k;
    A.scale = scale;
    A.out = h_out;
    const int run = kWords / (k + kW);   // their lists of k + 64 keys fill the wave's share of LDS
    if (c->tree_box > 0.0) launch_near<kLengths, true>(c, A, mg, c->n, run);
    else launch_near<kLengths, false>(c, A, mg, c->n, run);
    return AG_OK;
}

// Price & Monaghan lengths and Omega of every particle
int ag_launch_pm_lengths(ag_ctx* c, double n_ngb, double* h, double* omega) {
    int64_t mg = 0;
    AG_TRY(ag_prepare_groups(c, nullptr, c->n, &mg, nullptr, nullptr));
    NearArgs A = near_args(c);
    A.ngb = n_ngb;
    A.out = h;
    A.omega = omega;
    // every particle lies within the root's diagonal D of every other, so
    // at h = D / u* the sum is at least n (1 - 6 u*^2) >= 3 N / 32 (w(u) >=
    // 1 - 6 u^2 for u < 1/2)
    const double f = 3.0 * n_ngb / 32.0 / (double)c->n;
    A.hiscale = 1.01 / fmin(0.5, sqrt((1.0 - f) / 6.0));
    // Supports that the lists of 128 do not hold go one target at a time through a
    // list of 1024, which is cut again and again where its first radius took in
    // too much; Newton steps of eight targets together read them as often as there
    // are steps but keep nothing (ms, lists and steps; n = 100 000, uniform and
    // Plummer: n_ngb 100 1.76, 1.73 and 45, 14.6; 400 6.6, 3.8 and 143, 56; 2000 47,
    // 11.8 and 299, 86).  A small set waits for its longest run, which is longer of
    // eight targets than of one (5000 in clumps: 200 0.42, 0.56; 400 0.86, 0.77).
    const double lists = c->n > 16384 ? 128.0 : 256.0;
    if (n_ngb > lists) launch_near<kDensityWalk, false>(c, A, mg, c->n, kWalkRun);
    else launch_near<kDensity, false>(c, A, mg, c->n, kWords / kDenList);
    return AG_OK;
}

// Price & Monaghan sums: Z (mode 0, z_out) or the correction (mode 1, acc)
int ag_launch_pm_sum(ag_ctx* c, int mode, double n_ngb, double G, const double* omega, const double* z,
                     double* z_out, double* acc, const int32_t* idx, const int64_t* n_dev, bool add) {
    int64_t mg = 0;
    AG_TRY(ag_prepare_groups(c, idx, c->n, &mg, idx ? n_dev : nullptr, nullptr));
    NearArgs A = near_args(c);
    A.ngb = n_ngb;
    A.G = G;
    A.h = c->soft_h.as<double>();
    A.om = omega;
    A.z = z;
    A.zout = z_out;
    A.acc = acc;
    A.add = add || idx != nullptr;
    if (mode == 0) launch_near<kFactors, false>(c, A, mg, c->n, 2 * kWords / kSumList);
    else launch_near<kCorrect, false>(c, A, mg, c->n, 2 * kWords / kSumList);
    return AG_OK;
}
