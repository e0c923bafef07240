// Device-side records and per-lane shape algorithms of libgeonav (gfx950, FP64).
//
// One lane evaluates one track. Every algorithm is branch-free over lanes:
// all candidate surfaces of a shape are evaluated and the valid smallest one
// is kept with selects, so a wavefront never diverges inside a shape. The
// only branches are on the shape kind and the hole and convexity flags,
// which are uniform across a wavefront where the daughters are walked in
// lockstep (shape queries, sequential navigator loops); in a batch of the
// compacted navigators the lanes hold different daughters, and lanes of
// each kind take that kind's code in turn.
//
// Each distance query is a minimum over per-surface candidates (faces,
// z-planes, the outer and inner cylinder/cone nappes): for DistFromOutside
// a candidate is a point where the line enters the solid through that
// surface; for DistFromInside it is the first crossing of that surface's
// constraint. Quadric roots use the cancellation-free pair of formulas
// (numerator and denominator chosen by the sign of B), one division each.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gn {

constexpr double kBig = 1e30;
constexpr int kMaxDaughters = 1024;  // daughters per volume (GEO_MAX_DAUGHTERS)
constexpr int kCensusSlots = 16, kCensusCull = 14, kCensusTracks = 15;
// kPcon is an uncut polycone, kPcons one cut to an azimuth range.
enum : int32_t { kBox = 0, kTube = 1, kCone = 2, kTubs = 3, kCons = 4, kPcon = 5, kPcons = 6 };

// Shape with host-derived constants.
//   BOX  c0..2 = dx, dy, dz
//   TUBE c0 = rmin, c1 = rmax, c2 = dz, c3 = rmin^2, c4 = rmax^2
//   CONE c0 = dz, radius r(z) = a + b z: c1 = a_out, c2 = b_out, c3 = a_in, c4 = b_in,
//        c5..8 = rmin1, rmax1, rmin2, rmax2, c9..12 = their squares,
//        c13 = 1/sqrt(1 + b_out^2), c14 = 1/sqrt(1 + b_in^2),
//        c15 = 1/|outer edge|^2, c16 = 1/|inner edge|^2 (profile edges in (r, z))
//   TUBS, CONS (segments: the tube or cone cut to the azimuths [phi1, phi2],
//        phi2 = phi1 + dphi < phi1 + 2 pi, axis included): the base kind's
//        constants, and c17, c18 = cos phi1, sin phi1; c19, c20 = cos phi2, sin phi2.
//   PCON, PCONS (polycone, uncut or cut): its sections live in a PconRec
//        (see below); PCONS keeps the azimuth range in c17..c20.
// Slack of the range tests at candidate hit points (see "Edges" below):
//   c21 = eps = 1e-12 x the shape's bounding radius, and the limits widened
//   by it: BOX c3..5 = dx, dy, dz + eps; TUBE/TUBS c5 = dz + eps,
//   c6, c7 = (rmin - eps)^2 (0 if rmin <= eps), (rmax + eps)^2; CONE/CONS
//   c22 = dz + eps, c23..26 = the same two squares at -dz and at +dz.
struct alignas(16) ShapeRec {
    int32_t kind;
    int32_t hole;    // tube/cone: an inner surface exists (not both inner radii 0)
    int32_t convex;  // segment: dphi <= pi (the azimuth range is convex)
    int32_t pad;
    double c[28];
};
static_assert(sizeof(ShapeRec) == 240, "ShapeRec layout");

// Polycone: nz planes z_0 < ... < z_{nz-1} (nz <= kPconMax) with radii
// rin/rout at each; between two planes the radii are linear in z, section
// j's nappes being r = ao[j] + bo[j] z (outer) and ai[j] + bi[j] z (inner,
// present when bit j of hole_mask is set: not both inner radii 0).
constexpr int kPconMax = 8;
struct alignas(16) PconRec {
    int32_t nz;
    int32_t hole_mask;
    int32_t pad[2];
    double z[kPconMax], rin[kPconMax], rout[kPconMax];
    double rin2_0, rout2_0, rin2_l, rout2_l;  // squared end radii, widened by eps (hit tests)
    double ao[kPconMax - 1], bo[kPconMax - 1], ai[kPconMax - 1], bi[kPconMax - 1];
    double inv_eo[kPconMax - 1], inv_ei[kPconMax - 1];   // 1 / |profile edge|^2, outer and inner
    double eps;  // slack of the range tests at hit points: 1e-12 x (max |z| + max rmax)
    double far2; // square of a radius about the origin that holds the polycone, 1e-6 enlarged
};
static_assert(sizeof(PconRec) == 592, "PconRec layout");

// A placed daughter: mother-frame point = R * local + T.
struct alignas(16) DaughterRec {
    double rot[9];   // R, row-major
    double tr[3];    // T
    double bound_r;  // radius of a sphere about the local origin holding the shape
    double cull_r;   // the culling radius: bound_r enlarged by 1e-6 relative + 1e-6
    double pad;
    const PconRec *pcon;  // the polycone's sections (device), or NULL
    ShapeRec shape;
};
static_assert(sizeof(DaughterRec) == 368, "DaughterRec layout");

// Tasks of few tracks on a volume that is walked in lockstep (VolumeRec.dense) are
// culled all the same: each daughter in lockstep would be a step of a serial
// chain for the few lanes. Lines up to kFewLines tracks by the tests on the matrix
// cores, up to kFewExact by those in FP64 (whose pairs come daughter by
// daughter); points up to kFewPoints by those in FP64. (The paper's toy detector,
// 8 daughters, us per call. Navigator of 16, 20, 24, 32, 48 tracks: matrix cores 4.7
// 6.4 6.6 7.5 9; FP64 4.9 6.0 6.4 6.6 7.7; lockstep 7.0 throughout. Safety of 16, 24,
// 32, 48: 3.8 4.4 5.2 6; 3.5 4.2 4.6 5.0; lockstep 5.2.)
constexpr int kFewLines = 16, kFewExact = 40, kFewPoints = 48;

// Culling block: the daughters' operands of the culling tests, for up to
// kCullBlock daughters of a volume. The tests run on the matrix cores (see
// "Culling" below): 8 half-precision entries of each wavefront lane, in the layout
// of the A operand of a 32 x 32 x 16 product, in the units of the lines and of the
// localization (a) and in those of the safety (near); or in FP64 (see exact_row).
constexpr int kCullBlock = 32;
// the radius of the sphere that bounds the starts in the tests' units, the largest
// coordinate of a daughter's centre they take, and constants beyond every product:
// of a daughter past the last (or, negative, one that always passes), and of a
// track that meets none
constexpr float kCullR = 256.0f, kCullMax = 512.0f, kCullFar = 3.8e6f, kCullMiss = 2.0e6f;
struct alignas(16) CullBlock {
    unsigned int a[64][4], near[64][4];
    double exact[kCullBlock][4];
};
static_assert(sizeof(CullBlock) == 3072, "CullBlock layout");

// How a kernel culls: not at all; by the tests on the matrix cores in the mother's
// units; or as the volume asks (VolumeRec.exact, moved): those kernels hold every
// form, and what they add would cost the others registers (the branch on moved
// alone 6 % of the navigator of every kind at 2^22 tracks, 70.3 to 74.4 us).
enum : int { kNoTests = 0, kMatrixTests = 1, kAnyTests = 2 };

struct alignas(16) VolumeRec {
    ShapeRec mother;
    int32_t nd;     // number of daughters
    int32_t first;  // index of daughter 0 in the daughter table
    const PconRec *pcon;  // the mother's polycone sections (device), or NULL
    // The culling tests' coordinates. The unit comes from the mother's bounding
    // radius: lengths times near_s = kCullR / bound_r (0 when that is not a
    // normal number). Where the daughters are too small for it (moved), the lines
    // and the localization take theirs from the sphere about (cx, cy, cz) that
    // holds the daughters: lengths times cull_s, kCullR the square root of out2
    // there; else cull_s = near_s and the centre is the origin. near_back and
    // cull_back are the lengths, in those units, by which a start is moved back
    // for its test. (The navigator's are together in front: a wavefront waits
    // for each line of 64 bytes that it takes of this record.)
    double cull_s;
    float cull_back;
    int32_t first_block;  // index of the volume's first culling block
    int32_t exact;        // the tasks that take the tests in FP64
    int32_t dense;        // the tasks that walk all daughters in lockstep
    int32_t moved;
    int32_t crowded;      // the safety queues its pairs daughter by daughter
    int32_t rounds;       // large localizations take several rounds per wavefront
    float near_back;
    double near_s, cx, cy, cz, out2;
    double bound_r;  // radius of a sphere about the origin holding the mother
    // the safety's bound from the nearest culling sphere (see the compacted
    // safety), in the tests' units: of the daughters whose Safety at distance
    // |w| > r is at most sqrt(|w|^2 + c), the largest r^2 + c; of the others,
    // at most |w| + q, the largest r^2 and q (q < 0: none)
    float safe_d, safe_r2, safe_q;
    // the largest radius of both, and its square (inside a sphere: the Safety
    // of its daughter is at most |w| + r)
    float near_r, near_r2;
};
static_assert(sizeof(VolumeRec) == 368, "VolumeRec layout");
enum : int32_t { kLineTasks = 1, kLocateTask = 2, kSafetyTask = 4 };  // of VolumeRec.exact and dense

struct TracksDev {
    const double *x, *y, *z, *ux, *uy, *uz;
    int64_t n;
};

// Work unit of the batched kernel: `count` tracks of volume `volume` at
// pool index `offset`.
struct Tile {
    int32_t volume;
    int32_t count;
    int64_t offset;
};

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ double sq(double a) { return a * a; }

// n / d from the hardware reciprocal refined by two Newton steps: within
// about one ulp of the rounded quotient, six instructions instead of the
// eleven of the IEEE division sequence (which also rescales denormal and
// huge operands). A zero d gives NaN; every call site either has d in the
// normal range or rejects the result (the NaN fails its t >= 0 / ordering
// tests).
__device__ __forceinline__ double fdiv(double n, double d) {
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    return n * r;
}

// 1 / sqrt(x) for finite x > 0, within a few ulp: the hardware estimate
// refined by two Newton steps (each squares the relative error, so an
// estimate within 2^-13 reaches full precision). x below 2^-960, subnormals
// included, is scaled by 2^1000 first.
__device__ __forceinline__ double rsqrt_fine(double x) {
    const bool tiny = x < 0x1p-960;
    const double xs = tiny ? x * 0x1p1000 : x;
    double z = __builtin_amdgcn_rsq(xs);
    double e = fma(-xs * z, z, 1.0);  // 1 - x z^2
    z = fma(0.5 * z, e, z);
    e = fma(-xs * z, z, 1.0);
    z = fma(0.5 * z, e, z);
    return tiny ? z * 0x1p500 : z;
}

// sqrt(x) from the hardware reciprocal square root with a Goldschmidt step
// and two corrections (within about one ulp; 11 instructions against 17 for
// the correctly rounded sequence). x below 1e-300 (including 0 and the
// clamped negative discriminants) gives 0: a tangent line, or a safety below
// 1e-150.
__device__ __forceinline__ double fsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, x);
    g = fma(d, h, g);
    d = fma(-g, g, x);
    g = fma(d, h, g);
    return x > 1e-300 ? g : 0.0;
}

// Candidate update: keep the smallest valid t; on equal t the earlier
// candidate (lower surface id) stays.
__device__ __forceinline__ void take(bool ok, double t, int id, double &best, int &sid) {
    const bool better = ok && (t < best);
    best = better ? t : best;
    sid = better ? id : sid;
}

// Roots of f(t) = A t^2 + 2 B t + C, with s = sqrt(B^2 - A C).
// Root where f goes from + to - (A t + B = -s): (-B - s) / A = C / (s - B).
__device__ __forceinline__ double root_down(double A, double B, double C, double s) {
    const bool neg = B <= 0.0;
    const double num = neg ? C : -(B + s);
    const double den = neg ? (s - B) : A;
    return fdiv(num, den);
}
// Root where f goes from - to + (A t + B = +s): (-B + s) / A = -C / (s + B).
__device__ __forceinline__ double root_up(double A, double B, double C, double s) {
    const bool pos = B >= 0.0;
    const double num = pos ? -C : (s - B);
    const double den = pos ? (s + B) : A;
    return fdiv(num, den);
}

// Near-double roots. A line through a nappe's apex (or tangent to it) has a
// double root t0: B^2 - A C vanishes in exact arithmetic but comes out as
// +-(a few ulps of B^2), whose square root would move both roots by about
// sqrt(eps) t0. Within kSnap B^2 of zero the discriminant is taken as 0, and
// the formulas above then give t0 = C / (-B) = -B / A to rounding.
constexpr double kEps = 2.220446049250313e-16;  // of doubles
constexpr double kSnap = 64.0 * kEps;
__device__ __forceinline__ double disc_sqrt(double disc, double B) {
    return disc > kSnap * (B * B) ? fsqrt(disc) : 0.0;
}
__device__ __forceinline__ bool disc_ok(double disc, double B) { return disc >= -kSnap * (B * B); }

// Edges. A candidate counts only if its hit point lies on the surface's part
// that bounds the solid (a face's rectangle or annulus, a nappe's z range, a
// segment's azimuth range). At an edge two such tests meet, and a line
// through the edge could fail both by rounding. The tests at hit points
// therefore allow a slack eps of 1e-12 x the shape's size; a hit that far
// outside a face is within a comparable distance of the neighbouring
// surface's own hit. The membership tests themselves (Contains, and "the
// point is inside" in the distance queries) stay exact.

// ---------------------------------------------------------------------- box
__device__ __forceinline__ bool box_contains(const double *c, double x, double y, double z) {
    return fabs(x) <= c[0] && fabs(y) <= c[1] && fabs(z) <= c[2];
}

__device__ __forceinline__ double box_safety(const double *c, double x, double y, double z) {
    const double ex = fabs(x) - c[0], ey = fabs(y) - c[1], ez = fabs(z) - c[2];
    const double m = fmax(ex, fmax(ey, ez));
    const double ox = fmax(ex, 0.0), oy = fmax(ey, 0.0), oz = fmax(ez, 0.0);
    const double out = fsqrt(ox * ox + oy * oy + oz * oz);
    return m <= 0.0 ? -m : out;
}

// Entering face a: the point is beyond the slab (|p_a| > D_a) and moves
// towards it; the entry point must lie within the other two slabs.
__device__ __forceinline__ double box_dist_out(const double *c, double x, double y, double z,
                                               double ux, double uy, double uz, int &sid) {
    const double ax = fabs(x) - c[0], ay = fabs(y) - c[1], az = fabs(z) - c[2];
    const bool inside = ax <= 0.0 && ay <= 0.0 && az <= 0.0;
    double best = kBig;
    sid = -1;
    {
        const double t = fdiv(ax, fabs(ux));
        const bool ok = ax > 0.0 && x * ux < 0.0 && fabs(fma(t, uy, y)) <= c[4] &&
                        fabs(fma(t, uz, z)) <= c[5];
        take(ok, t, 0, best, sid);
    }
    {
        const double t = fdiv(ay, fabs(uy));
        const bool ok = ay > 0.0 && y * uy < 0.0 && fabs(fma(t, ux, x)) <= c[3] &&
                        fabs(fma(t, uz, z)) <= c[5];
        take(ok, t, 1, best, sid);
    }
    {
        const double t = fdiv(az, fabs(uz));
        const bool ok = az > 0.0 && z * uz < 0.0 && fabs(fma(t, ux, x)) <= c[3] &&
                        fabs(fma(t, uy, y)) <= c[4];
        take(ok, t, 2, best, sid);
    }
    return inside ? 0.0 : best;
}

// Leaving: the first face the line reaches on each axis.
// The same distance without the surface that sets it, for callers that only
// need the value: the three exits taken with fmin, which skips the NaN of an
// axis the direction does not move along (fdiv by 0); the result equals
// box_dist_in's bit for bit (the smallest exit below kBig, else kBig; 0
// outside).
__device__ __forceinline__ double box_exit(const double *c, double x, double y, double z, double ux,
                                           double uy, double uz) {
    // (numerator and denominator with the direction's sign: the same quotient)
    const double tx = fdiv(copysign(c[0], ux) - x, ux);
    const double ty = fdiv(copysign(c[1], uy) - y, uy);
    const double tz = fdiv(copysign(c[2], uz) - z, uz);
    const double best = fmin(kBig, fmin(tx, fmin(ty, tz)));
    return box_contains(c, x, y, z) ? best : 0.0;
}

__device__ __forceinline__ double box_dist_in(const double *c, double x, double y, double z,
                                              double ux, double uy, double uz, int &sid) {
    const bool inside = box_contains(c, x, y, z);
    double best = kBig;
    sid = -1;
    take(ux != 0.0, fdiv(c[0] - (ux > 0.0 ? x : -x), fabs(ux)), 0, best, sid);
    take(uy != 0.0, fdiv(c[1] - (uy > 0.0 ? y : -y), fabs(uy)), 1, best, sid);
    take(uz != 0.0, fdiv(c[2] - (uz > 0.0 ? z : -z), fabs(uz)), 2, best, sid);
    return inside ? best : 0.0;
}

// --------------------------------------------------------------------- tube
// Surfaces: 0 = z planes, 1 = outer cylinder, 2 = inner cylinder.
__device__ __forceinline__ bool tube_contains(const double *c, double x, double y, double z) {
    const double rsq = x * x + y * y;
    return fabs(z) <= c[2] && rsq <= c[4] && rsq >= c[3];
}

// (r, z) profile is the rectangle [rmin, rmax] x [-dz, dz]; without a hole
// the axis bounds no surface.
__device__ __forceinline__ double tube_safety(const double *c, int hole, double x, double y,
                                              double z) {
    const double r = fsqrt(x * x + y * y);
    const double eo = r - c[1];
    const double ei = hole ? c[0] - r : -kBig;
    const double ez = fabs(z) - c[2];
    const double er = fmax(eo, ei);
    const double m = fmax(er, ez);
    const double orr = fmax(er, 0.0), oz = fmax(ez, 0.0);
    const double out = fsqrt(orr * orr + oz * oz);
    return m <= 0.0 ? -m : out;
}

// ------------------------------------------------------------ azimuth range
// A segment keeps the azimuths [phi1, phi2] and the z axis. With the inward
// normals of its two bounding half-planes, n1 = (-sin phi1, cos phi1) and
// n2 = (sin phi2, -cos phi2), a point q is in the range when a = n1.q >= 0
// and b = n2.q >= 0 if dphi <= pi (a convex range), and when a >= 0 or
// b >= 0 if dphi > pi (the complement is then the open convex wedge a < 0,
// b < 0). a and b are the signed distances from the two face planes.
__device__ __forceinline__ double wedge_a(const double *c, double x, double y) {
    return fma(c[17], y, -c[18] * x);
}
__device__ __forceinline__ double wedge_b(const double *c, double x, double y) {
    return fma(c[20], x, -c[19] * y);
}
__device__ __forceinline__ bool wedge_in(const ShapeRec &s, double x, double y) {
    const double a = wedge_a(s.c, x, y), b = wedge_b(s.c, x, y);
    return s.convex ? (a >= 0.0 && b >= 0.0) : (a >= 0.0 || b >= 0.0);
}
// The same for a candidate's hit point, with the slack eps (c21).
__device__ __forceinline__ bool wedge_in_hit(const ShapeRec &s, double x, double y) {
    const double a = wedge_a(s.c, x, y), b = wedge_b(s.c, x, y);
    const double e = -s.c[21];
    return s.convex ? (a >= e && b >= e) : (a >= e || b >= e);
}

// Leaving the range along the line (the point is in it). Convex range: the
// first plane crossed outwards. Wider range: entering the open complement
// {a < 0} and {b < 0}, which happens at the later of the starts of the two
// half-lines {t : a(t) < 0}, {t : b(t) < 0}, provided neither has ended by
// then. Surfaces 3 and 4.
__device__ __forceinline__ void wedge_exit(const ShapeRec &s, double x, double y, double ux,
                                           double uy, double &best, int &sid) {
    const double a0 = wedge_a(s.c, x, y), da = wedge_a(s.c, ux, uy);
    const double b0 = wedge_b(s.c, x, y), db = wedge_b(s.c, ux, uy);
    const double ta = fdiv(-a0, da), tb = fdiv(-b0, db);
    if (s.convex) {
        take(da < 0.0, ta, 3, best, sid);
        take(db < 0.0, tb, 4, best, sid);
    } else {
        // {t : a(t) < 0} is (ta, inf) for da < 0, (-inf, ta) for da > 0, and
        // everything or nothing for da == 0
        const double lo_a = da < 0.0 ? ta : ((da > 0.0 || a0 < 0.0) ? -kBig : kBig);
        const double hi_a = da > 0.0 ? ta : ((da < 0.0 || a0 < 0.0) ? kBig : -kBig);
        const double lo_b = db < 0.0 ? tb : ((db > 0.0 || b0 < 0.0) ? -kBig : kBig);
        const double hi_b = db > 0.0 ? tb : ((db < 0.0 || b0 < 0.0) ? kBig : -kBig);
        const double lo = fmax(lo_a, lo_b), hi = fmin(hi_a, hi_b);
        take(lo < hi && hi > 0.0 && lo >= 0.0, lo, lo_a >= lo_b ? 3 : 4, best, sid);
    }
}

__device__ __forceinline__ bool cone_contains(const double *c, int hole, double x, double y,
                                              double z);
__device__ __forceinline__ bool pcon_contains(const PconRec &P, double x, double y, double z);
__device__ __forceinline__ bool pcon_contains_hit(const PconRec &P, double x, double y, double z);

template <int BASE>
__device__ __forceinline__ bool base_contains(const ShapeRec &s, const PconRec *pc, double x,
                                              double y, double z) {
    if (BASE == kTube) return tube_contains(s.c, x, y, z);
    if (BASE == kCone) return cone_contains(s.c, s.hole, x, y, z);
    return pcon_contains(*pc, x, y, z);
}

// Membership of a face entry's hit point in the base solid, with the slack
// eps on every bound.
template <int BASE>
__device__ __forceinline__ bool base_contains_hit(const ShapeRec &s, const PconRec *pc, double x,
                                                  double y, double z) {
    const double *c = s.c;
    const double rsq = x * x + y * y;
    if (BASE == kTube) return fabs(z) <= c[5] && rsq <= c[7] && rsq >= c[6];
    if (BASE == kCone) {
        const double wo = fma(c[2], z, c[1]) + c[21];
        const double wi = fmax(fma(c[4], z, c[3]) - c[21], 0.0);
        return fabs(z) <= c[22] && rsq <= wo * wo && rsq >= wi * wi;
    }
    return pcon_contains_hit(*pc, x, y, z);
}

// Entering the range through a flat face, at a point inside the base solid
// (surfaces 3 and 4). The line's parameters in the range follow from the
// half-lines {t : a(t) >= 0} and {t : b(t) >= 0}: for a convex range their
// intersection [w_lo, w_hi], entered at w_lo when the start is outside; for a
// wider range their union, the complement of the open interval in which the
// line crosses the wedge a < 0, b < 0, re-entered where that interval ends.
// Taking the entry from these intervals, not from a point test on each
// face's half-plane, keeps a line through the axis (both planes crossed at
// one point) exact.
template <int BASE>
__device__ __forceinline__ void face_entries(const ShapeRec &s, const PconRec *pc, double x,
                                             double y, double z, double ux, double uy, double uz,
                                             double &best, int &sid) {
    const double a0 = wedge_a(s.c, x, y), da = wedge_a(s.c, ux, uy);
    const double b0 = wedge_b(s.c, x, y), db = wedge_b(s.c, ux, uy);
    const double ta = fdiv(-a0, da), tb = fdiv(-b0, db);
    double t;
    bool ok;
    int id;
    if (s.convex) {
        // {a >= 0} is [ta, inf) for da > 0, (-inf, ta] for da < 0, all or nothing for da == 0
        const double lo_a = da > 0.0 ? ta : ((da < 0.0 || a0 >= 0.0) ? -kBig : kBig);
        const double hi_a = da < 0.0 ? ta : ((da > 0.0 || a0 >= 0.0) ? kBig : -kBig);
        const double lo_b = db > 0.0 ? tb : ((db < 0.0 || b0 >= 0.0) ? -kBig : kBig);
        const double hi_b = db < 0.0 ? tb : ((db > 0.0 || b0 >= 0.0) ? kBig : -kBig);
        t = fmax(lo_a, lo_b);
        ok = t <= fmin(hi_a, hi_b) && t >= 0.0;
        id = lo_a >= lo_b ? 3 : 4;
    } else {
        // {a < 0} is (ta, inf) for da < 0, (-inf, ta) for da > 0
        const double lo_a = da < 0.0 ? ta : ((da > 0.0 || a0 < 0.0) ? -kBig : kBig);
        const double hi_a = da > 0.0 ? ta : ((da < 0.0 || a0 < 0.0) ? kBig : -kBig);
        const double lo_b = db < 0.0 ? tb : ((db > 0.0 || b0 < 0.0) ? -kBig : kBig);
        const double hi_b = db > 0.0 ? tb : ((db < 0.0 || b0 < 0.0) ? kBig : -kBig);
        t = fmin(hi_a, hi_b);
        ok = fmax(lo_a, lo_b) < t && t >= 0.0 && t < kBig;
        id = hi_a <= hi_b ? 3 : 4;
    }
    const double xh = fma(t, ux, x), yh = fma(t, uy, y), zh = fma(t, uz, z);
    take(ok && base_contains_hit<BASE>(s, pc, xh, yh, zh), t, id, best, sid);
}

// With SEG (a segment) an entry through a base surface counts only at a hit
// point within the range, and the face entries join the candidates.
template <bool SEG>
__device__ __forceinline__ double tube_dist_out(const ShapeRec &S, double x, double y, double z,
                                                double ux, double uy, double uz, int &sid) {
    const double *c = S.c;
    const int hole = S.hole;
    const double dz = c[2];
    const double rsq = x * x + y * y;
    const bool inside = fabs(z) <= dz && rsq <= c[4] && rsq >= c[3] && (!SEG || wedge_in(S, x, y));
    double best = kBig;
    sid = -1;
    {   // z planes: from beyond the slab, moving towards it, landing on the annulus
        const double az = fabs(z) - dz;
        const double t = fdiv(az, fabs(uz));
        const double xh = fma(t, ux, x), yh = fma(t, uy, y);
        const double r2 = xh * xh + yh * yh;
        const bool ok = az > 0.0 && z * uz < 0.0 && r2 >= c[6] && r2 <= c[7] &&
                        (!SEG || wedge_in_hit(S, xh, yh));
        take(ok, t, 0, best, sid);
    }
    const double A = ux * ux + uy * uy;
    const double B = x * ux + y * uy;
    {   // outer cylinder, entered from r > rmax
        const double C = rsq - c[4];
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = fdiv(C, s - B);
        const bool ok = C > 0.0 && B < 0.0 && disc_ok(disc, B) && fabs(fma(t, uz, z)) <= c[5] &&
                        (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
        take(ok, t, 1, best, sid);
    }
    if (hole) {  // inner cylinder, left from inside the hole into the material
        const double C = rsq - c[3];
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_up(A, B, C, s);
        const bool ok = disc_ok(disc, B) && t >= 0.0 && fabs(fma(t, uz, z)) <= c[5] &&
                        (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
        take(ok, t, 2, best, sid);
    }
    if (SEG) face_entries<kTube>(S, nullptr, x, y, z, ux, uy, uz, best, sid);
    return inside ? 0.0 : best;
}

// With SEG the exit is the earlier of leaving the base and leaving the range.
template <bool SEG>
__device__ __forceinline__ double tube_dist_in(const ShapeRec &S, double x, double y, double z,
                                               double ux, double uy, double uz, int &sid) {
    const double *c = S.c;
    const int hole = S.hole;
    const double dz = c[2];
    const double rsq = x * x + y * y;
    const bool inside = fabs(z) <= dz && rsq <= c[4] && rsq >= c[3] && (!SEG || wedge_in(S, x, y));
    double best = kBig;
    sid = -1;
    take(uz != 0.0, fdiv(dz - (uz > 0.0 ? z : -z), fabs(uz)), 0, best, sid);
    const double A = ux * ux + uy * uy;
    const double B = x * ux + y * uy;
    {   // leave the outer cylinder
        const double C = rsq - c[4];
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_up(A, B, C, s);
        take(disc_ok(disc, B) && t >= 0.0, t, 1, best, sid);
    }
    if (hole) {  // enter the hole's cylinder
        const double C = rsq - c[3];
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_down(A, B, C, s);
        take(disc_ok(disc, B) && t >= 0.0, t, 2, best, sid);
    }
    if (SEG) wedge_exit(S, x, y, ux, uy, best, sid);
    return inside ? best : 0.0;
}

// --------------------------------------------------------------------- cone
// Surfaces: 0 = z planes, 1 = outer nappe r = a_out + b_out z,
// 2 = inner nappe r = a_in + b_in z. On a nappe, f = r^2 - (a + b z)^2 along
// the line is the quadratic A t^2 + 2 B t + C with
//   A = ux^2 + uy^2 - (b uz)^2, B = x ux + y uy - b uz w, C = x^2 + y^2 - w^2,
// w = a + b z. Its roots include the mirror nappe (a + b z < 0); a root on the
// mirror lies outside |z| <= dz (the radii are >= 0 on the slab), so the slab
// test at the root rejects it for entries, and for exits the z plane comes
// first.
__device__ __forceinline__ bool cone_contains(const double *c, int hole, double x, double y,
                                              double z) {
    const double rsq = x * x + y * y;
    const double wo = fma(c[2], z, c[1]);
    const double wi = fma(c[4], z, c[3]);
    return fabs(z) <= c[0] && rsq <= wo * wo && (!hole || rsq >= wi * wi);
}

__device__ __forceinline__ double seg_d2(double r, double z, double r0, double z0, double er,
                                         double ez, double inv_ee) {
    const double wr = r - r0, wz = z - z0;
    const double t = fmin(fmax((wr * er + wz * ez) * inv_ee, 0.0), 1.0);
    return sq(wr - t * er) + sq(wz - t * ez);
}

// Profile: trapezoid with corners (rmin1, -dz) (rmax1, -dz) (rmax2, dz)
// (rmin2, dz). Inside it is convex, so the distance is the smallest distance
// to the edges' lines; outside it is the smallest distance to the segments.
__device__ __forceinline__ double cone_safety(const double *c, int hole, double x, double y,
                                              double z) {
    const double dz = c[0];
    const double r = fsqrt(x * x + y * y);
    const double wo = fma(c[2], z, c[1]);
    const double wi = fma(c[4], z, c[3]);
    const bool inside = fabs(z) <= dz && r <= wo && (!hole || r >= wi);
    double din = fmin(dz - fabs(z), (wo - r) * c[13]);
    din = hole ? fmin(din, (r - wi) * c[14]) : din;
    // outside: bottom and top edges, outer and inner slanted edges
    const double rb = fmin(fmax(r, c[5]), c[6]);
    const double rt = fmin(fmax(r, c[7]), c[8]);
    double d2 = fmin(sq(r - rb) + sq(z + dz), sq(r - rt) + sq(z - dz));
    d2 = fmin(d2, seg_d2(r, z, c[6], -dz, c[8] - c[6], 2.0 * dz, c[15]));
    const double di2 = seg_d2(r, z, c[5], -dz, c[7] - c[5], 2.0 * dz, c[16]);
    d2 = hole ? fmin(d2, di2) : d2;
    return inside ? din : fsqrt(d2);
}

template <bool SEG>
__device__ __forceinline__ double cone_dist_out(const ShapeRec &S, double x, double y, double z,
                                                double ux, double uy, double uz, int &sid) {
    const double *c = S.c;
    const int hole = S.hole;
    const double dz = c[0];
    const double rsq = x * x + y * y;
    const double wo = fma(c[2], z, c[1]);
    const double wi = fma(c[4], z, c[3]);
    const bool inside = fabs(z) <= dz && rsq <= wo * wo && (!hole || rsq >= wi * wi) &&
                        (!SEG || wedge_in(S, x, y));
    double best = kBig;
    sid = -1;
    {   // z planes: the face's annulus depends on which end is hit
        const double az = fabs(z) - dz;
        const double t = fdiv(az, fabs(uz));
        const double xh = fma(t, ux, x), yh = fma(t, uy, y);
        const double r2 = xh * xh + yh * yh;
        // select between the two faces' verdicts (not their constants, which
        // stay uniform scalars)
        const bool on_bot = r2 >= c[23] && r2 <= c[24];
        const bool on_top = r2 >= c[25] && r2 <= c[26];
        const bool ok = az > 0.0 && z * uz < 0.0 && (z > 0.0 ? on_top : on_bot) &&
                        (!SEG || wedge_in_hit(S, xh, yh));
        take(ok, t, 0, best, sid);
    }
    const double A0 = ux * ux + uy * uy;
    const double B0 = x * ux + y * uy;
    {   // outer nappe: entered where f goes from + to -
        const double v = c[2] * uz;
        const double A = A0 - v * v, B = B0 - v * wo, C = rsq - wo * wo;
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_down(A, B, C, s);
        const bool ok = disc_ok(disc, B) && t >= 0.0 && fabs(fma(t, uz, z)) <= c[22] &&
                        (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
        take(ok, t, 1, best, sid);
    }
    if (hole) {  // inner nappe: left from the hole where f goes from - to +
        const double v = c[4] * uz;
        const double A = A0 - v * v, B = B0 - v * wi, C = rsq - wi * wi;
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_up(A, B, C, s);
        const bool ok = disc_ok(disc, B) && t >= 0.0 && fabs(fma(t, uz, z)) <= c[22] &&
                        (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
        take(ok, t, 2, best, sid);
    }
    if (SEG) face_entries<kCone>(S, nullptr, x, y, z, ux, uy, uz, best, sid);
    return inside ? 0.0 : best;
}

template <bool SEG>
__device__ __forceinline__ double cone_dist_in(const ShapeRec &S, double x, double y, double z,
                                               double ux, double uy, double uz, int &sid) {
    const double *c = S.c;
    const int hole = S.hole;
    const double dz = c[0];
    const double rsq = x * x + y * y;
    const double wo = fma(c[2], z, c[1]);
    const double wi = fma(c[4], z, c[3]);
    const bool inside = fabs(z) <= dz && rsq <= wo * wo && (!hole || rsq >= wi * wi) &&
                        (!SEG || wedge_in(S, x, y));
    double best = kBig;
    sid = -1;
    take(uz != 0.0, fdiv(dz - (uz > 0.0 ? z : -z), fabs(uz)), 0, best, sid);
    const double A0 = ux * ux + uy * uy;
    const double B0 = x * ux + y * uy;
    {   // leave the outer nappe
        const double v = c[2] * uz;
        const double A = A0 - v * v, B = B0 - v * wo, C = rsq - wo * wo;
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_up(A, B, C, s);
        take(disc_ok(disc, B) && t >= 0.0, t, 1, best, sid);
    }
    if (hole) {  // enter the inner nappe (the hole)
        const double v = c[4] * uz;
        const double A = A0 - v * v, B = B0 - v * wi, C = rsq - wi * wi;
        const double disc = B * B - A * C;
        const double s = disc_sqrt(disc, B);
        const double t = root_down(A, B, C, s);
        take(disc_ok(disc, B) && t >= 0.0, t, 2, best, sid);
    }
    if (SEG) wedge_exit(S, x, y, ux, uy, best, sid);
    return inside ? best : 0.0;
}

// ----------------------------------------------------------------- polycone
// A sequence of connected cone sections (section 3.1). The radii are
// continuous across the planes inside, so those planes bound nothing: the
// surfaces are the two end planes (surface 0) and, per section j, its outer
// nappe (surface 5 + 2 j) and inner nappe (6 + 2 j), each a boundary only for
// z in [z_j, z_{j+1}], which every candidate checks at its hit point. The
// check allows a slack of eps: a line through a kink of the profile (a
// plane between sections) meets the two sections' nappes there, and rounding
// could otherwise put both hit points just outside their ranges. Within eps
// of the plane the two nappes are within |b_j - b_{j+1}| eps of each other.
// Nappe roots on the mirror nappe fall outside the ranges (the radii are
// >= 0 on them). The loops run over the sections, the same for every lane.
__device__ __forceinline__ bool pcon_contains(const PconRec &P, double x, double y, double z) {
    const double rsq = x * x + y * y;
    const int ns = P.nz - 1;
    bool in = false;
    for (int j = 0; j < ns; ++j) {
        const double wo = fma(P.bo[j], z, P.ao[j]);
        const double wi = fma(P.bi[j], z, P.ai[j]);
        const bool hole = (P.hole_mask >> j) & 1;
        in |= z >= P.z[j] && z <= P.z[j + 1] && rsq <= wo * wo && (!hole || rsq >= wi * wi);
    }
    return in;
}

// Membership of a candidate's hit point, with the slack eps on every bound.
__device__ __forceinline__ bool pcon_contains_hit(const PconRec &P, double x, double y, double z) {
    const double rsq = x * x + y * y;
    const int ns = P.nz - 1;
    bool in = false;
    for (int j = 0; j < ns; ++j) {
        const double wo = fma(P.bo[j], z, P.ao[j]) + P.eps;
        const double wi = fmax(fma(P.bi[j], z, P.ai[j]) - P.eps, 0.0);
        in |= z >= P.z[j] - P.eps && z <= P.z[j + 1] + P.eps && rsq <= wo * wo && rsq >= wi * wi;
    }
    return in;
}

// (u, z) in the profile polygon; u is a signed coordinate in a face's plane.
__device__ __forceinline__ bool pcon_in_profile(const PconRec &P, double u, double z) {
    const int ns = P.nz - 1;
    bool in = false;
    for (int j = 0; j < ns; ++j) {
        const double wo = fma(P.bo[j], z, P.ao[j]);
        const double wi = fma(P.bi[j], z, P.ai[j]);
        in |= z >= P.z[j] && z <= P.z[j + 1] && u <= wo && u >= wi;
    }
    return in;
}

// (SIDE: the point is known to be outside, or inside)
template <bool SEG, bool SIDE = false>
__device__ __forceinline__ double pcon_dist_out(const ShapeRec &S, const PconRec &P, double x,
                                                double y, double z, double ux, double uy,
                                                double uz, int &sid) {
    const bool inside = !SIDE && pcon_contains(P, x, y, z) && (!SEG || wedge_in(S, x, y));
    const int ns = P.nz - 1;
    double best = kBig;
    sid = -1;
    {   // bottom plane, from below moving up, landing on its annulus
        const double t = fdiv(P.z[0] - z, uz);
        const double xh = fma(t, ux, x), yh = fma(t, uy, y);
        const double r2 = xh * xh + yh * yh;
        const bool ok = z < P.z[0] && uz > 0.0 && r2 >= P.rin2_0 && r2 <= P.rout2_0 &&
                        (!SEG || wedge_in_hit(S, xh, yh));
        take(ok, t, 0, best, sid);
    }
    {   // top plane, from above moving down
        const double t = fdiv(P.z[ns] - z, uz);
        const double xh = fma(t, ux, x), yh = fma(t, uy, y);
        const double r2 = xh * xh + yh * yh;
        const bool ok = z > P.z[ns] && uz < 0.0 && r2 >= P.rin2_l && r2 <= P.rout2_l &&
                        (!SEG || wedge_in_hit(S, xh, yh));
        take(ok, t, 0, best, sid);
    }
    const double rsq = x * x + y * y;
    const double A0 = ux * ux + uy * uy;
    const double B0 = x * ux + y * uy;
    for (int j = 0; j < ns; ++j) {
        const double zlo = P.z[j] - P.eps, zhi = P.z[j + 1] + P.eps;
        {   // outer nappe: entered where f goes from + to -
            const double w = fma(P.bo[j], z, P.ao[j]);
            const double v = P.bo[j] * uz;
            const double A = A0 - v * v, B = B0 - v * w, C = rsq - w * w;
            const double disc = B * B - A * C;
            const double s = disc_sqrt(disc, B);
            const double t = root_down(A, B, C, s);
            const double zh = fma(t, uz, z);
            const bool ok = disc_ok(disc, B) && t >= 0.0 && zh >= zlo && zh <= zhi &&
                            (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
            take(ok, t, 5 + 2 * j, best, sid);
        }
        if ((P.hole_mask >> j) & 1) {  // inner nappe: left from the hole
            const double w = fma(P.bi[j], z, P.ai[j]);
            const double v = P.bi[j] * uz;
            const double A = A0 - v * v, B = B0 - v * w, C = rsq - w * w;
            const double disc = B * B - A * C;
            const double s = disc_sqrt(disc, B);
            const double t = root_up(A, B, C, s);
            const double zh = fma(t, uz, z);
            const bool ok = disc_ok(disc, B) && t >= 0.0 && zh >= zlo && zh <= zhi &&
                            (!SEG || wedge_in_hit(S, fma(t, ux, x), fma(t, uy, y)));
            take(ok, t, 6 + 2 * j, best, sid);
        }
    }
    if (SEG) face_entries<kPcon>(S, &P, x, y, z, ux, uy, uz, best, sid);
    return inside ? 0.0 : best;
}

template <bool SEG, bool SIDE = false>
__device__ __forceinline__ double pcon_dist_in(const ShapeRec &S, const PconRec &P, double x,
                                               double y, double z, double ux, double uy, double uz,
                                               int &sid) {
    const bool inside = SIDE || (pcon_contains(P, x, y, z) && (!SEG || wedge_in(S, x, y)));
    const int ns = P.nz - 1;
    double best = kBig;
    sid = -1;
    take(uz < 0.0, fdiv(P.z[0] - z, uz), 0, best, sid);
    take(uz > 0.0, fdiv(P.z[ns] - z, uz), 0, best, sid);
    const double rsq = x * x + y * y;
    const double A0 = ux * ux + uy * uy;
    const double B0 = x * ux + y * uy;
    for (int j = 0; j < ns; ++j) {
        const double zlo = P.z[j] - P.eps, zhi = P.z[j + 1] + P.eps;
        {   // leave the outer nappe
            const double w = fma(P.bo[j], z, P.ao[j]);
            const double v = P.bo[j] * uz;
            const double A = A0 - v * v, B = B0 - v * w, C = rsq - w * w;
            const double disc = B * B - A * C;
            const double s = disc_sqrt(disc, B);
            const double t = root_up(A, B, C, s);
            const double zh = fma(t, uz, z);
            take(disc_ok(disc, B) && t >= 0.0 && zh >= zlo && zh <= zhi, t, 5 + 2 * j, best, sid);
        }
        if ((P.hole_mask >> j) & 1) {  // enter the hole
            const double w = fma(P.bi[j], z, P.ai[j]);
            const double v = P.bi[j] * uz;
            const double A = A0 - v * v, B = B0 - v * w, C = rsq - w * w;
            const double disc = B * B - A * C;
            const double s = disc_sqrt(disc, B);
            const double t = root_down(A, B, C, s);
            const double zh = fma(t, uz, z);
            take(disc_ok(disc, B) && t >= 0.0 && zh >= zlo && zh <= zhi, t, 6 + 2 * j, best, sid);
        }
    }
    if (SEG) wedge_exit(S, x, y, ux, uy, best, sid);
    return inside ? best : 0.0;
}

// Squared distance from (r, z) to the profile's edges: the two end edges,
// the outer edges and the inner edges; an inner edge on the axis (both radii
// 0) bounds no surface and is skipped unless `axis` is set (a face's
// polygon, whose edge on the axis is real).
__device__ __forceinline__ double pcon_edges_d2(const PconRec &P, double r, double z, bool axis) {
    const int ns = P.nz - 1;
    const double rb = fmin(fmax(r, P.rin[0]), P.rout[0]);
    const double rt = fmin(fmax(r, P.rin[ns]), P.rout[ns]);
    double d2 = fmin(sq(r - rb) + sq(z - P.z[0]), sq(r - rt) + sq(z - P.z[ns]));
    for (int j = 0; j < ns; ++j) {
        const double h = P.z[j + 1] - P.z[j];
        d2 = fmin(d2, seg_d2(r, z, P.rout[j], P.z[j], P.rout[j + 1] - P.rout[j], h, P.inv_eo[j]));
        if (axis || ((P.hole_mask >> j) & 1))
            d2 = fmin(d2, seg_d2(r, z, P.rin[j], P.z[j], P.rin[j + 1] - P.rin[j], h, P.inv_ei[j]));
    }
    return d2;
}

// A solid of revolution: the planar distance from (r, z) to the profile's
// edges, inside and outside alike.
__device__ __forceinline__ double pcon_safety(const PconRec &P, double x, double y, double z) {
    return fsqrt(pcon_edges_d2(P, fsqrt(x * x + y * y), z, false));
}

__device__ __forceinline__ double pcon_face_d2(const PconRec &P, double u, double z) {
    return pcon_in_profile(P, u, z) ? 0.0 : pcon_edges_d2(P, u, z, true);
}

// ------------------------------------------------------ segment safety
// Squared distance from (u, z) to a face, the profile polygon laid in the
// half-plane at phi_i with u along e_i (0 on or inside the polygon). The
// tube's profile is the rectangle [rmin, rmax] x [-dz, dz]; the cone's is the
// trapezoid, its inner edge included even on the axis (there the two faces
// meet).
__device__ __forceinline__ double tube_face_d2(const double *c, double u, double z) {
    const double du = fmax(fmax(c[0] - u, u - c[1]), 0.0);
    const double dz = fmax(fabs(z) - c[2], 0.0);
    return du * du + dz * dz;
}

__device__ __forceinline__ double cone_face_d2(const double *c, double u, double z) {
    const double dz = c[0];
    const double wo = fma(c[2], z, c[1]);
    const double wi = fma(c[4], z, c[3]);
    const bool in = fabs(z) <= dz && u <= wo && u >= wi;
    const double rb = fmin(fmax(u, c[5]), c[6]);
    const double rt = fmin(fmax(u, c[7]), c[8]);
    double d2 = fmin(sq(u - rb) + sq(z + dz), sq(u - rt) + sq(z - dz));
    d2 = fmin(d2, seg_d2(u, z, c[6], -dz, c[8] - c[6], 2.0 * dz, c[15]));
    d2 = fmin(d2, seg_d2(u, z, c[5], -dz, c[7] - c[5], 2.0 * dz, c[16]));
    return in ? 0.0 : d2;
}

// Safety of a segment: the boundary is the base's surfaces within the range
// and the two faces.
//   Outside the solid: the base's Safety if p is in the range (the nearest
//   point of a surface of revolution has p's own azimuth), and the distance
//   to each face, sqrt(v_i^2 + d2_i) with v_i the distance from the face's
//   plane and d2_i that of (u_i, z) to the face polygon (this also covers
//   the base surfaces' edges when p is out of the range).
//   Inside: the base's Safety and, per face, |v_i| when the foot of the
//   perpendicular lies on the face's half-plane (u_i >= 0) or else r. The
//   foot can fall short of the face only into the hole, where the base's
//   inner surface is nearer than |v_i|; off the half-plane the face is at
//   least r away, exactly r where the profile reaches the axis, and with a
//   hole the inner surface is nearer than r.
template <int BASE>
__device__ __forceinline__ double seg_safety(const ShapeRec &S, const PconRec *pc, double x,
                                             double y, double z) {
    const double *c = S.c;
    const double base = BASE == kTube   ? tube_safety(c, S.hole, x, y, z)
                        : BASE == kCone ? cone_safety(c, S.hole, x, y, z)
                                        : pcon_safety(*pc, x, y, z);
    const bool in_base = base_contains<BASE>(S, pc, x, y, z);
    const double a = wedge_a(c, x, y), b = wedge_b(c, x, y);
    const bool in_range = S.convex ? (a >= 0.0 && b >= 0.0) : (a >= 0.0 || b >= 0.0);
    const double u1 = fma(c[18], y, c[17] * x), u2 = fma(c[20], y, c[19] * x);
    const double r = fsqrt(x * x + y * y);
    const double f_in = fmin(u1 >= 0.0 ? fabs(a) : r, u2 >= 0.0 ? fabs(b) : r);
    const double d1 = BASE == kTube   ? tube_face_d2(c, u1, z)
                      : BASE == kCone ? cone_face_d2(c, u1, z)
                                      : pcon_face_d2(*pc, u1, z);
    const double d2 = BASE == kTube   ? tube_face_d2(c, u2, z)
                      : BASE == kCone ? cone_face_d2(c, u2, z)
                                      : pcon_face_d2(*pc, u2, z);
    const double f_out = fsqrt(fmin(fma(a, a, d1), fma(b, b, d2)));
    return (in_base && in_range) ? fmin(base, f_in) : fmin(in_range ? base : kBig, f_out);
}

// ------------------------------------------------------ dispatch on kind
// `pc` is the shape's polycone record (read only for the polycone kinds).
template <int KIND>
__device__ __forceinline__ bool shape_contains(const ShapeRec &s, const PconRec *pc, double x,
                                               double y, double z) {
    if (KIND == kBox) return box_contains(s.c, x, y, z);
    if (KIND == kTube) return tube_contains(s.c, x, y, z);
    if (KIND == kCone) return cone_contains(s.c, s.hole, x, y, z);
    if (KIND == kTubs) return tube_contains(s.c, x, y, z) && wedge_in(s, x, y);
    if (KIND == kCons) return cone_contains(s.c, s.hole, x, y, z) && wedge_in(s, x, y);
    if (KIND == kPcon) return pcon_contains(*pc, x, y, z);
    return pcon_contains(*pc, x, y, z) && wedge_in(s, x, y);
}

template <int KIND>
__device__ __forceinline__ double shape_safety(const ShapeRec &s, const PconRec *pc, double x,
                                               double y, double z) {
    if (KIND == kBox) return box_safety(s.c, x, y, z);
    if (KIND == kTube) return tube_safety(s.c, s.hole, x, y, z);
    if (KIND == kCone) return cone_safety(s.c, s.hole, x, y, z);
    if (KIND == kTubs) return seg_safety<kTube>(s, pc, x, y, z);
    if (KIND == kCons) return seg_safety<kCone>(s, pc, x, y, z);
    if (KIND == kPcon) return pcon_safety(*pc, x, y, z);
    return seg_safety<kPcon>(s, pc, x, y, z);
}

template <int KIND>
__device__ __forceinline__ double shape_dist_out(const ShapeRec &s, const PconRec *pc, double x,
                                                 double y, double z, double ux, double uy,
                                                 double uz, int &sid) {
    if (KIND == kBox) return box_dist_out(s.c, x, y, z, ux, uy, uz, sid);
    if (KIND == kTube) return tube_dist_out<false>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kCone) return cone_dist_out<false>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kTubs) return tube_dist_out<true>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kCons) return cone_dist_out<true>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kPcon) return pcon_dist_out<false>(s, *pc, x, y, z, ux, uy, uz, sid);
    return pcon_dist_out<true>(s, *pc, x, y, z, ux, uy, uz, sid);
}

template <int KIND>
__device__ __forceinline__ double shape_dist_in(const ShapeRec &s, const PconRec *pc, double x,
                                                double y, double z, double ux, double uy,
                                                double uz, int &sid) {
    if (KIND == kBox) return box_dist_in(s.c, x, y, z, ux, uy, uz, sid);
    if (KIND == kTube) return tube_dist_in<false>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kCone) return cone_dist_in<false>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kTubs) return tube_dist_in<true>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kCons) return cone_dist_in<true>(s, x, y, z, ux, uy, uz, sid);
    if (KIND == kPcon) return pcon_dist_in<false>(s, *pc, x, y, z, ux, uy, uz, sid);
    return pcon_dist_in<true>(s, *pc, x, y, z, ux, uy, uz, sid);
}

// `kind` is uniform across the wavefront wherever these are called. KSET
// bounds the kinds a geometry holds (kSetBasic: box, tube, cone; kSetSeg:
// and their segments; kSetAll: and polycones), so that kernels for simpler
// geometries carry no code for the kinds they never meet: the navigator's
// loop body stays small, which the instruction cache rewards.
enum : int { kSetBasic = 0, kSetSeg = 1, kSetAll = 2 };

#define GN_KIND_SWITCH(CALL) GN_KIND_SWITCH_ON(s.kind, CALL)
#define GN_KIND_SWITCH_ON(KIND, CALL)       \
    if (KSET == kSetBasic) {                \
        switch (KIND) {                     \
            case kBox: return CALL(kBox);   \
            case kTube: return CALL(kTube); \
            default: return CALL(kCone);    \
        }                                   \
    }                                       \
    if (KSET == kSetSeg) {                  \
        switch (KIND) {                     \
            case kBox: return CALL(kBox);   \
            case kTube: return CALL(kTube); \
            case kCone: return CALL(kCone); \
            case kTubs: return CALL(kTubs); \
            default: return CALL(kCons);    \
        }                                   \
    }                                       \
    switch (KIND) {                         \
        case kBox: return CALL(kBox);       \
        case kTube: return CALL(kTube);     \
        case kCone: return CALL(kCone);     \
        case kTubs: return CALL(kTubs);     \
        case kCons: return CALL(kCons);     \
        case kPcon: return CALL(kPcon);     \
        default: return CALL(kPcons);       \
    }

template <int KSET = kSetAll>
__device__ __forceinline__ bool any_contains(const ShapeRec &s, const PconRec *pc, double x,
                                             double y, double z) {
#define GN_CALL(K) shape_contains<K>(s, pc, x, y, z)
    GN_KIND_SWITCH(GN_CALL)
#undef GN_CALL
}

template <int KSET = kSetAll>
__device__ __forceinline__ double any_safety(const ShapeRec &s, const PconRec *pc, double x,
                                             double y, double z) {
#define GN_CALL(K) shape_safety<K>(s, pc, x, y, z)
    GN_KIND_SWITCH(GN_CALL)
#undef GN_CALL
}

template <int KSET = kSetAll>
__device__ __forceinline__ double any_dist_out(const ShapeRec &s, const PconRec *pc, double x,
                                               double y, double z, double ux, double uy,
                                               double uz, int &sid) {
#define GN_CALL(K) shape_dist_out<K>(s, pc, x, y, z, ux, uy, uz, sid)
    GN_KIND_SWITCH(GN_CALL)
#undef GN_CALL
}

template <int KSET = kSetAll>
__device__ __forceinline__ double any_dist_in(const ShapeRec &s, const PconRec *pc, double x,
                                              double y, double z, double ux, double uy,
                                              double uz, int &sid) {
#define GN_CALL(K) shape_dist_in<K>(s, pc, x, y, z, ux, uy, uz, sid)
    GN_KIND_SWITCH(GN_CALL)
#undef GN_CALL
}

// Number of kind classes a kind set tells apart (kinds beyond them take the
// last class's code, as in the switch above), and the class of a kind.
template <int KSET>
__device__ __forceinline__ constexpr int kind_classes() {
    return KSET == kSetBasic ? 3 : (KSET == kSetSeg ? 5 : 7);
}
template <int KSET>
__device__ __forceinline__ int kind_class(int kind) {
    return kind < kind_classes<KSET>() - 1 ? kind : kind_classes<KSET>() - 1;
}

// DistFromOutside for a class known to be uniform over the wavefront (a
// scalar branch instead of one path per kind present).
template <int KSET>
__device__ __forceinline__ double class_dist_out(int cls, const ShapeRec &s, const PconRec *pc, double x,
                                                 double y, double z, double ux, double uy, double uz,
                                                 int &sid) {
#define GN_CALL(K) shape_dist_out<K>(s, pc, x, y, z, ux, uy, uz, sid)
    GN_KIND_SWITCH_ON(cls, GN_CALL)
#undef GN_CALL
}
template <int KSET>
__device__ __forceinline__ double class_safety(int cls, const ShapeRec &s, const PconRec *pc, double x, double y,
                                               double z) {
#define GN_CALL(K) shape_safety<K>(s, pc, x, y, z)
    GN_KIND_SWITCH_ON(cls, GN_CALL)
#undef GN_CALL
}
#undef GN_KIND_SWITCH
#undef GN_KIND_SWITCH_ON

// The mother's DistFromInside for the navigators; SURF false: the surface
// that sets it is not wanted (sid = -1), and a box mother takes box_exit.
template <bool SURF, int KSET>
__device__ __forceinline__ double mother_step(const VolumeRec &v, double x, double y, double z, double ux,
                                              double uy, double uz, int &sid) {
    if (!SURF && v.mother.kind == kBox) {
        sid = -1;
        return box_exit(v.mother.c, x, y, z, ux, uy, uz);
    }
    return any_dist_in<KSET>(v.mother, v.pcon, x, y, z, ux, uy, uz, sid);
}

// Outward-or-inward normal (any scale/sign) of surface `sid` at local point h.
__device__ __forceinline__ void surface_normal(const ShapeRec &s, const PconRec *pc, int sid,
                                               double hx, double hy, double hz, double &nx,
                                               double &ny, double &nz) {
    nx = ny = nz = 0.0;
    if (s.kind == kBox) {
        nx = sid == 0 ? 1.0 : 0.0;
        ny = sid == 1 ? 1.0 : 0.0;
        nz = sid == 2 ? 1.0 : 0.0;
        return;
    }
    if (sid == 0) { nz = 1.0; return; }
    if (sid < 0) return;
    if (sid == 3) {  // segment face planes: n1, n2
        nx = -s.c[18];
        ny = s.c[17];
        return;
    }
    if (sid == 4) {
        nx = s.c[20];
        ny = -s.c[19];
        return;
    }
    nx = hx;
    ny = hy;
    if (s.kind == kPcon || s.kind == kPcons) {  // nappe of section j: r = a + b z
        const int j = (sid - 5) >> 1;
        const bool outer = ((sid - 5) & 1) == 0;
        const double a = outer ? pc->ao[j] : pc->ai[j];
        const double b = outer ? pc->bo[j] : pc->bi[j];
        nz = -b * fma(b, hz, a);
        return;
    }
    if (s.kind == kCone || s.kind == kCons) {
        const double a = sid == 1 ? s.c[1] : s.c[3];
        const double b = sid == 1 ? s.c[2] : s.c[4];
        nz = -b * fma(b, hz, a);
    }
}

// ----------------------------------------------------------- navigator
// Per-track navigator of Fig. 1b, sequential form (the adjoint's forward
// recomputation, and the forward navigators with culling off): the mother's
// DistFromInside, then each daughter's DistFromOutside in its own frame,
// keeping the smallest (ties to the mother, then the lowest index).
// Daughters are walked in lockstep by the whole wavefront, so the daughter
// record and its kind are uniform (scalar loads, scalar branch).
//
// With COUNT, the work done is tallied into census[kCensusSlots] (one atomic
// per wavefront and event, adding the number of active lanes): slots
// 2 * kind + hole count daughter evaluations, slot kCensusCull culling
// tests, slot kCensusTracks tracks.
__device__ __forceinline__ void census_add(unsigned long long *census, int slot) {
    const unsigned long long act = __ballot(1);
    if ((int)__lane_id() == __ffsll((unsigned long long)act) - 1)
        atomicAdd(&census[slot], (unsigned long long)__popcll(act));
}

template <bool HAS_OFFS, bool TRACK_SURF, bool COUNT = false, int KSET = kSetAll>
__device__ __forceinline__ void nav_track(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                          const double *__restrict__ offs, double x, double y,
                                          double z, double ux, double uy, double uz, double &best,
                                          int &hit, int &bsid,
                                          unsigned long long *census = nullptr) {
    int sid;
    if (COUNT) census_add(census, kCensusTracks);
    best = mother_step<TRACK_SURF, KSET>(v, x, y, z, ux, uy, uz, sid);
    hit = -1;
    bsid = sid;
    const int nd = v.nd;
    for (int k = 0; k < nd; ++k) {
        const DaughterRec &D = dau[k];
        double wx = x - D.tr[0], wy = y - D.tr[1], wz = z - D.tr[2];
        if (HAS_OFFS) {
            wx -= offs[3 * k + 0];
            wy -= offs[3 * k + 1];
            wz -= offs[3 * k + 2];
        }
        if (COUNT) census_add(census, 2 * D.shape.kind + D.shape.hole);
        const double *R = D.rot;
        // local = R^T w
        const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
        const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
        const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
        const double lux = fma(R[6], uz, fma(R[3], uy, R[0] * ux));
        const double luy = fma(R[7], uz, fma(R[4], uy, R[1] * ux));
        const double luz = fma(R[8], uz, fma(R[5], uy, R[2] * ux));
        const double s = any_dist_out<KSET>(D.shape, D.pcon, lx, ly, lz, lux, luy, luz, sid);
        const bool better = s < best;
        best = better ? s : best;
        hit = better ? k : hit;
        if (TRACK_SURF) bsid = better ? sid : bsid;
    }
    best = best == 0.0 ? 0.0 : best;  // a step of -0 is reported as +0
}

// ------------------------------------------------ compacted navigator
// A (track, daughter) pair needs evaluating only when the track's
// half-line from p passes within the daughter's culling radius (its
// bounding radius enlarged by 1e-6 relative + 1e-6) of the sphere's centre
// T; otherwise the daughter cannot be entered at any t >= 0, so it could
// neither lower the step nor win a tie. (The mother's exit would bound the
// half-line further, but the daughters lie inside the mother and no line
// comes back near them after leaving a convex mother: on the batched
// workload that bound removes no pair.) Skipping a daughter for a whole
// wavefront unless some lane needs it would leave all 64 lanes evaluating it
// for the one lane or two that do (with random tracks about one lane in 64).
// The compacted form separates the two: the wavefront first runs the culling
// tests of its tracks against every daughter (see "culling" below) and
// appends each (track, daughter) pair that passes to a queue in LDS; then
// each lane takes one queued pair and evaluates that daughter's
// DistFromOutside for that track, so a batch of 64 pairs costs one pass (the
// lanes of different kinds take their kinds' code in turn).
//
// The step of a track is the minimum over its candidates of (s, index),
// compared lexicographically with the mother as index -1: the result of
// the sequential loop, whose strict < keeps the earlier of equal steps.
// Each track's running minimum sits in LDS as a 64-bit key (an
// order-preserving map of the double, -0 taken as +0, so that a step of -0
// is reported as +0 as in the sequential loop) and an index (packed with the
// surface that set the step, see hit_pack); a batch merges into it with a
// 64-bit LDS min on the key, then, for the pairs whose key equals the new
// minimum, an integer min on the index (reset first when the batch lowered
// the key). After every batch the slot holds the lexicographic minimum of
// all candidates merged so far, whatever the order of the batches.
//
// The queue holds 64 pairs, each with its track's six coordinates: a lane
// that appends a pair has its track in registers, and the batch would
// otherwise read it from global memory, where the six component arrays put
// each track on six cache lines, long evicted from L2 by the time its batch
// runs. A full queue is run at once (a batch of 64 pairs, every lane busy);
// what is left at the end of the tile makes the last batch. All LDS traffic
// of the queue and the minima is the wavefront's own, whose LDS instructions
// execute in program order, so no barrier is needed.
constexpr int kQueueCap = 64;
constexpr int kListCap = 256;  // pairs of a round, 64 for each of the four daughters tested together at least
template <int U>
struct NavScratch {
    unsigned long long key[U * 64];   // running minimum per track: key of the step
    int hit[U * 64];                  // and the packed index of its candidate
    // the queued pairs: (daughter << 10) | round * 64 + lane, and the track
    unsigned int pair[kQueueCap];
    double x[kQueueCap], y[kQueueCap], z[kQueueCap], ux[kQueueCap], uy[kQueueCap], uz[kQueueCap];
    // the volume's second culling block (tiles of a few rounds; volumes of
    // box, tube and cone, whose kernels have the registers): read from global
    // memory in every round, it would be waited for behind the next round's
    // tracks (512 baskets of 64 volumes 76.7 to 75.0 us)
    // (stored and loaded 16 bytes at a time)
    static constexpr bool kSecond = U == 2 || U == 4;
    alignas(kSecond ? 16 : 4) unsigned int second[kSecond ? 64 : 1][4];
    static_assert(U * 64 <= 1024, "track index within the tile: 10 bits");
};

// The key of a step: steps are >= 0 (or -0, taken as +0), so their bits less
// the sign order them; one more, so that 0 is left for a mother step that is
// not a number, which is never beaten. A daughter's, larger than every
// number's, never wins. (As in the sequential loop. 6 VALU instructions for
// the mother's and 3 for a daughter's, 16 and 13 for a map of all doubles.)
__device__ __forceinline__ unsigned long long step_key(double s) {
    return ((unsigned long long)__double_as_longlong(s) & 0x7fffffffffffffffull) + 1ull;
}
__device__ __forceinline__ unsigned long long mother_key(double s) { return s == s ? step_key(s) : 0ull; }
__device__ __forceinline__ double key_step(unsigned long long k) {
    return __longlong_as_double((long long)(k - 1ull));
}

// Accesses to the running minima, which other lanes of the wavefront update
// atomically.
template <typename T>
__device__ __forceinline__ T lds_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename T>
__device__ __forceinline__ void lds_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Number of set bits of m below this lane.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// DistFromOutside of daughter k (record D) for a mother-frame track;
// sid receives the surface that set it. With a class cls >= 0 (uniform over
// the wavefront), the daughter is known to be of that kind class.
template <bool HAS_OFFS, int KSET>
__device__ __forceinline__ double daughter_dist_out(const DaughterRec &D,
                                                    const double *__restrict__ offs, int k, double x,
                                                    double y, double z, double ux, double uy,
                                                    double uz, int &sid, int cls = -1) {
    double wx = x - D.tr[0], wy = y - D.tr[1], wz = z - D.tr[2];
    if (HAS_OFFS) {
        wx -= offs[3 * k + 0];
        wy -= offs[3 * k + 1];
        wz -= offs[3 * k + 2];
    }
    const double *R = D.rot;
    const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
    const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
    const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
    const double lux = fma(R[6], uz, fma(R[3], uy, R[0] * ux));
    const double luy = fma(R[7], uz, fma(R[4], uy, R[1] * ux));
    const double luz = fma(R[8], uz, fma(R[5], uy, R[2] * ux));
    if (cls >= 0) return class_dist_out<KSET>(cls, D.shape, D.pcon, lx, ly, lz, lux, luy, luz, sid);
    return any_dist_out<KSET>(D.shape, D.pcon, lx, ly, lz, lux, luy, luz, sid);
}

// A tile's six track arrays from its first track on: uniform pointers, so
// that a lane's track, an unsigned index below 1024 off them, is loaded with
// a scalar base address and a 32-bit vector offset (no 64-bit address per
// lane and array).
struct TileTracks {
    const double *x, *y, *z, *ux, *uy, *uz;
};
// element j (< 2^29) of a, its byte offset formed in 32 bits
template <typename T>
__device__ __forceinline__ T &at32(T *a, unsigned int j) {
    return *reinterpret_cast<T *>(reinterpret_cast<char *>(a) + j * (unsigned int)sizeof(T));
}
template <typename T>
__device__ __forceinline__ const T &at32(const T *a, unsigned int j) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(a) + j * (unsigned int)sizeof(T));
}
__device__ __forceinline__ TileTracks tile_tracks(const TracksDev &t, int64_t base) {
    TileTracks r;
    r.x = t.x + base;
    r.y = t.y + base;
    r.z = t.z + base;
    r.ux = t.ux + base;
    r.uy = t.uy + base;
    r.uz = t.uz + base;
    return r;
}

// A hit slot holds the candidate's index k (-1 for the mother) and the
// surface that set its step (sid, -1 .. 254) as k * 256 + sid + 1: ordered
// by k, since each index has one candidate per track, and the adjoint reads
// the winner's surface back without evaluating it again.
__device__ __forceinline__ int hit_pack(int k, int sid) { return k * 256 + (sid + 1); }
__device__ __forceinline__ int hit_index(int v) { return v >> 8; }
__device__ __forceinline__ int hit_surface(int v) { return (v & 255) - 1; }

// Merges a candidate (its step's key and packed hit) into running minimum j
// of S, the wavefront's own. Lanes of one call may share a minimum; whatever
// the order of calls, it ends at the lexicographic minimum of all candidates
// merged. merge_step: the same for candidate (s, k) with surface sid.
template <typename Scratch>
__device__ __forceinline__ void merge_key(Scratch &S, int j, unsigned long long key, int hp) {
    const unsigned long long before = lds_load(&S.key[j]);
    __hip_atomic_fetch_min(&S.key[j], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    const unsigned long long now = lds_load(&S.key[j]);
    if (now < before) lds_store(&S.hit[j], 0x7fffffff);
    if (key == now) __hip_atomic_fetch_min(&S.hit[j], hp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename Scratch>
__device__ __forceinline__ void merge_step(Scratch &S, int j, double s, int k, int sid) {
    merge_key(S, j, step_key(s), hit_pack(k, sid));
}

// Runs the qn queued pairs as one batch, one pair per lane.
template <int U, bool HAS_OFFS, bool COUNT, int KSET, bool SURF>
__device__ __forceinline__ void nav_batch(const DaughterRec *__restrict__ dau,
                                          const double *__restrict__ offs, NavScratch<U> &S, int qn, int lane,
                                          unsigned long long *census) {
    const bool on = lane < qn;
    const unsigned int q = on ? S.pair[lane] : 0u;
    const int j = (int)(q & 1023u);
    const int k = (int)(q >> 10);
    if (COUNT) {
        const int c = 2 * dau[k].shape.kind + dau[k].shape.hole;
        for (int cc = 0; cc < 2 * (kPcons + 1); ++cc) {
            const unsigned long long m = __ballot(on && c == cc);
            if (m != 0ull && lane == __ffsll(m) - 1) atomicAdd(&census[cc], (unsigned long long)__popcll(m));
        }
    }
    if (on) {
        int sid;
        const double s = daughter_dist_out<HAS_OFFS, KSET>(dau[k], offs, k, S.x[lane], S.y[lane], S.z[lane],
                                                           S.ux[lane], S.uy[lane], S.uz[lane], sid);
        merge_step(S, j, s, k, SURF ? sid : -1);  // (a surface not wanted is not tracked)
    }
}

// ------------------------------------------------------------- culling
// The tests ask, for the 64 tracks of a wavefront and a block of 32
// daughters, which half-lines pass within a daughter's culling radius r of
// its centre T. With w = p - T and e = d / |d|, that is |w|^2 - r^2 <=
// min(w.e, 0)^2, two inner products per pair: a contraction over K = 16,
// run as two v_mfma_f32_32x32x16_f16 per 32 tracks (one for |w|^2 - r^2, one
// for w.e), daughters along the rows, tracks along the columns. What is left
// per pair is one fma and one v_alignbit that shifts the sign into the
// lane's mask: two VALU instructions, where the tests took nine in FP64
// (bound by VALU issue: 55 % of the batched navigator's instructions). Two
// products and 32 VALU instructions for 1024 pairs measured 154 cycles of a
// SIMD, 9 x 16 FP64 instructions about 700.
//
// The test is a filter: a pair that passes is evaluated in FP64, a pair that
// is dropped must be one whose half-line misses the sphere. So every error
// of the filter goes one way:
//  - Lengths are taken in units where the sphere that bounds the starts (the
//    mother's, or the daughters', see VolumeRec) has the radius kCullR = 256, and
//    every factor as two half-precision pieces (round
//    toward zero, 21 bits) whose products are exact in the FP32 accumulator,
//    the product of two second pieces left out.
//  - r^2 is widened by delta = 2^-15 ((256 + L)^2 + |T|^2), L the shift
//    below. With W = 256 + L + |T| (so delta >= 2^-16 W^2), the first
//    product is off by at most 2^-18.8 W^2 and w.e by 2^-18.3 W (a sum of
//    products off by 2^-22 of its terms' magnitudes was measured, four times
//    that is allowed for), together 2^-16.8 W^2.
//  - min(w.e, 0)^2 costs an instruction that w.e |w.e| does not, which is the
//    same for w.e <= 0 and wrongly negative otherwise. The start is
//    therefore moved back along the line by L, more than any radius: a
//    half-line that meets a sphere then has w.e <= 0 there, and the test is
//    exact for it; a line that meets a sphere up to L behind its start
//    passes as well.
//  - A daughter whose centre or radius is over kCullMax (out of the mother's
//    reach) always passes. The radii that the volume's bounds (cull_back, the
//    safety's) are formed from are those within kCullMax, told by the same
//    product of doubles.
// A track that starts outside the mother has step 0 from the mother, which
// no daughter can beat: it is left out, so every start is within 256. With the
// daughters' sphere a start outside it is where its line enters it.
//
// The widening delta is at least two units squared: the tests take a daughter for
// a sphere of 1.4 units or more. In the mother's units that is 0.55 % of its
// radius, and a detector in a mother 30 times its size passed 1.45 pairs per track
// for 0.135 (2^22 tracks 164 us; in a mother of its own size 49.5, and with the
// daughters' units here 50.9). Volumes that lose that much take the daughters'
// units, and where those do not resolve them either, the tests in FP64.
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

// a and b as half-precision pairs: hi the values toward zero, lo what is left.
__device__ __forceinline__ unsigned int half_pair(float a, float b) {
    return __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_pkrtz(a, b));
}
__device__ __forceinline__ void half_split(float a, float b, unsigned int &hi, unsigned int &lo) {
    hi = half_pair(a, b);
    float ra, rb;  // a and b less their halves of hi, one mixed fma each
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(hi), "v"(a));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(hi), "v"(b));
    lo = half_pair(ra, rb);
}

// The K = 16 slots, as pairs: lanes 0..31 hold slots 0..7 of row (column)
// lane, lanes 32..63 slots 8..15 of row (column) lane - 32.
//   daughter (hi, lo the pieces of -2 T, n of (|T|^2 - r^2 - delta) / 64, s of -2 r):
//     hi.x hi.y | hi.z 64 | hi.x hi.y | hi.z 64 | lo.x lo.y | lo.z s.hi | n.hi n.lo | s.hi s.lo
//   track (of a vector v, a constant c / 64 and a length f):
//     hi.x hi.y | hi.z c.hi | lo.x lo.y | lo.z c.lo | hi.x hi.y | hi.z f.hi | 64 64 | f.lo f.hi
// and for w.e, whose daughters are the same, zeros in the last four slots.
// Their product is -2 T.v + c + |T|^2 - r^2 - delta - 2 r f.
//
// Row 8 i + 4 h + j (i, j < 4, h < 2) holds the daughter whose mask bit
// cull_merge makes of lane half h and result 4 i + j: the block's first 16
// daughters are in the last 8 results of the lanes.
template <bool HAS_OFFS, bool NEAR = false>  // NEAR: in the safety's units
__device__ __forceinline__ uint4v cull_operand(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                               const double *__restrict__ offs, int k0, int lane) {
    const int row = lane & 31;
    const int bit = 15 - ((row >> 3) * 4 + (row & 3));
    const int k = k0 + ((bit & 8) << 1) + ((row & 4) << 1) + (bit & 7);
    float tx = 0.0f, ty = 0.0f, tz = 0.0f, r = 0.0f;
    float n = kCullFar;  // past the last daughter: never passes
    if (k < v.nd) {
        const DaughterRec &D = dau[k];
        double cx = D.tr[0], cy = D.tr[1], cz = D.tr[2];
        if (HAS_OFFS) {
            cx += offs[3 * k + 0];
            cy += offs[3 * k + 1];
            cz += offs[3 * k + 2];
        }
        const double s = NEAR ? v.near_s : v.cull_s;
        const float back = NEAR ? v.near_back : v.cull_back;
        tx = (float)((NEAR ? cx : cx - v.cx) * s);
        ty = (float)((NEAR ? cy : cy - v.cy) * s);
        tz = (float)((NEAR ? cz : cz - v.cz) * s);
        const double rs = D.cull_r * s;
        r = (float)rs;
        const float tt = fmaf(tz, tz, fmaf(ty, ty, tx * tx));
        const float reach = kCullR + back;
        n = fmaf(-0x1p-15f, fmaf(reach, reach, tt), fmaf(-r, r, tt));
        bool near = s > 0.0 && fabsf(tx) <= kCullMax && fabsf(ty) <= kCullMax && fabsf(tz) <= kCullMax &&
                    rs <= (double)kCullMax;
        // (within the sphere that the starts are moved to)
        if (!NEAR && v.moved) near = __builtin_amdgcn_sqrtf(tt) + r <= kCullR - 0.125f;
        if (!near) {  // (or not a number): always passes
            tx = ty = tz = r = 0.0f;
            n = -kCullFar;
        }
    }
    unsigned int hxy, lxy, hzr, lzr, nn, rr, dummy;
    half_split(-2.0f * tx, -2.0f * ty, hxy, lxy);
    half_split(-2.0f * tz, -2.0f * r, hzr, lzr);
    half_split(n * 0.015625f, 0.0f, nn, dummy);
    const unsigned int n2 = (nn & 0xffffu) | (dummy << 16);
    const unsigned int hz64 = (hzr & 0xffffu) | 0x54000000u;  // (64 in half precision: 0x5400)
    const unsigned int lzsh = (lzr & 0xffffu) | (hzr & 0xffff0000u);
    rr = (hzr >> 16) | (lzr & 0xffff0000u);
    const bool upper = lane >= 32;
    return uint4v{upper ? lxy : hxy, upper ? lzsh : hz64, upper ? n2 : hxy, upper ? rr : hz64};
}

// The two column operands (tracks 0..31 and 32..63) from the 16 slots that
// each lane forms of its own track: the halves of the wavefront swap.
__device__ __forceinline__ void cull_swap(const unsigned int (&lo)[4], const unsigned int (&hi)[4], uint4v (&col)[2]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint2v r = __builtin_amdgcn_permlane32_swap(lo[i], hi[i], false, false);
        col[0][i] = r.x;  // lower lanes' lo | lower lanes' hi
        col[1][i] = r.y;  // upper lanes' lo | upper lanes' hi
    }
}

// Columns of a vector and a constant (the length 0); `ones` is the pair that
// meets n, (64, 64) or zeros. The split vector stays in v (z in the low
// halves of its second pairs).
struct CullVector {
    unsigned int xy_hi, xy_lo, z_hi, z_lo;
};
__device__ __forceinline__ void cull_columns(float x, float y, float z, float c, unsigned int ones, CullVector &v,
                                             uint4v (&col)[2]) {
    half_split(x, y, v.xy_hi, v.xy_lo);
    half_split(z, c * 0.015625f, v.z_hi, v.z_lo);
    cull_swap({v.xy_hi, v.z_hi, v.xy_lo, v.z_lo}, {v.xy_hi, v.z_hi & 0xffffu, ones, 0u}, col);
}
// The same vector's columns with another constant, and a length.
__device__ __forceinline__ void cull_columns(const CullVector &v, float c, float f, uint4v (&col)[2]) {
    unsigned int h, l;
    half_split(c * 0.015625f, f, h, l);
    cull_swap({v.xy_hi, __builtin_amdgcn_perm(h, v.z_hi, 0x05040100u), v.xy_lo,
               __builtin_amdgcn_perm(l, v.z_lo, 0x05040100u)},
              {v.xy_hi, __builtin_amdgcn_perm(h, v.z_hi, 0x07060100u), 0x54005400u,
               __builtin_amdgcn_perm(h, l, 0x07060302u)},
              col);
}

// A wavefront's column operands: of |w|^2 - r^2 (p) and of w.e (e).
struct CullTracks {
    uint4v p[2], e[2];
};

// A start relative to the centre of the sphere that holds the daughters, if that is
// outside the sphere where its half-line enters it; true if it never does (the
// start is then the centre, and the caller lets no daughter of the sphere pass).
// In FP64: the sphere holds the culling spheres with 0.1 units to spare, 51 units^2
// of a line's squared distance, and the rounding of the discriminant is below 4 eps
// times the squared distance of the start, 4 units^2 at the farthest, 2^26 units.
__device__ __forceinline__ bool cull_enter(const VolumeRec &v, double &x, double &y, double &z, double ux, double uy,
                                           double uz) {
    x -= v.cx;
    y -= v.cy;
    z -= v.cz;
    const double dd = fma(uz, uz, fma(uy, uy, ux * ux));
    const double b = fma(z, uz, fma(y, uy, x * ux));
    const double g = fma(z, z, fma(y, y, x * x)) - v.out2;
    const double disc = fma(b, b, -g * dd);
    const bool out = g > 0.0, miss = out && !(b < 0.0 && disc >= 0.0);
    const double t = out && !miss ? fdiv(g, fsqrt(disc) - b) : 0.0;
    x = miss ? 0.0 : fma(t, ux, x);
    y = miss ? 0.0 : fma(t, uy, y);
    z = miss ? 0.0 : fma(t, uz, z);
    return miss;
}

// Starts moved back by v.cull_back along the unit direction. A zero
// direction, or one whose |d|^2 overflows or is not a number, gives e = 0
// (the test then takes the start point); the FP32 root serves unless a lane
// that counts (`on`) has |d|^2 near the ends of its range.
template <bool MOVED>
__device__ __forceinline__ void cull_tracks(const VolumeRec &v, double x, double y, double z, double ux, double uy,
                                            double uz, bool on, CullTracks &c) {
    float ex = (float)ux, ey = (float)uy, ez = (float)uz;
    const float dd = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
    const bool odd = !(dd > 1e-30f && dd < 1e30f);
    const float il = __builtin_amdgcn_rsqf(dd);
    ex *= il;
    ey *= il;
    ez *= il;
    if (__builtin_amdgcn_ballot_w64(on && odd) != 0ull) {
        const double d2 = fma(uz, uz, fma(uy, uy, ux * ux));
        const bool has = d2 > 0.0 && d2 < __builtin_inf();
        const double il2 = rsqrt_fine(d2);
        if (odd) {
            ex = has ? (float)(ux * il2) : 0.0f;
            ey = has ? (float)(uy * il2) : 0.0f;
            ez = has ? (float)(uz * il2) : 0.0f;
        }
    }
    const float back = -v.cull_back;
    const double s = v.cull_s;
    bool miss = false;
    if (MOVED && v.moved) miss = cull_enter(v, x, y, z, ux, uy, uz);
    const float px = fmaf(back, ex, (float)(x * s)), py = fmaf(back, ey, (float)(y * s)),
                pz = fmaf(back, ez, (float)(z * s));
    float pp = fmaf(pz, pz, fmaf(py, py, px * px));
    if (MOVED && miss) pp = kCullMiss;
    CullVector split;
    cull_columns(px, py, pz, pp, 0x54005400u, split, c.p);
    cull_columns(0.5f * ex, 0.5f * ey, 0.5f * ez, fmaf(pz, ez, fmaf(py, ey, px * ex)), 0u, split, c.e);
}

__device__ __forceinline__ float16v cull_product(const uint4v &a, const uint4v &b) {
    const float16v zero = {};
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), zero,
                                                  0, 0, 0);
}

// The signs of a product's 16 results in a lane (column lane % 32; result i
// is row 8 (i / 4) + 4 (lane / 32) + i % 4), result i at bit 15 - i; of the
// last 8 alone where the other rows hold no daughters. (A branch for each
// group of 4 results cost more than it skipped: 54.9 to 56.4 us at 32
// daughters and 2^22 tracks.)
template <int N, typename F>
__device__ __forceinline__ unsigned int cull_signs(F result) {
    unsigned int m = 0u;
#pragma unroll
    for (int i = 16 - N; i < 16; ++i) m = __builtin_amdgcn_alignbit(m, __float_as_uint(result(i)), 31);
    return m;
}

// The masks of the two halves' columns as each lane's own track's 32 rows:
// bit k is daughter k of the block (the bytes of the lower lanes' rows and
// the upper ones' in turn).
__device__ __forceinline__ unsigned int cull_merge(unsigned int m0, unsigned int m1) {
    const uint2v r = __builtin_amdgcn_permlane32_swap(m0, m1, false, false);
    return __builtin_amdgcn_perm(r.y, r.x, 0x05010400u);
}
template <int N>
__device__ __forceinline__ unsigned int cull_mask_of(const uint4v &a, const CullTracks &c) {
    unsigned int m[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float16v g = cull_product(a, c.p[t]);
        const float16v b = cull_product(a, c.e[t]);
        m[t] = cull_signs<N>([&](int i) { return fmaf(b[i], fabsf(b[i]), g[i]); });
        __builtin_amdgcn_sched_barrier(0);
    }
    return cull_merge(m[0], m[1]);
}
// (left: daughters from the block's first on)
__device__ __forceinline__ unsigned int cull_mask(const uint4v &a, const CullTracks &c, int left) {
    return left <= 16 ? cull_mask_of<8>(a, c) : cull_mask_of<16>(a, c);
}

struct Track {
    double x, y, z, ux, uy, uz;
};
// Where the (up to four) rounds of an adjoint workgroup's wavefront start.
struct Rounds {
    int odd, pair;
    __device__ __forceinline__ int at(int u) const { return (u & 1) * odd + (u >> 1) * pair; }
};

// Navigates the tracks base + u * 64 + lane (u < U, index below `count` > 0
// past base) of one volume, leaving each track's step (as a key) and hit
// index in S; with SURF, the hit slot also carries the surface that set the
// step (for the adjoint). Each round's tracks are requested a round ahead
// (with the tests on the matrix cores the wavefronts otherwise waited for
// memory 75 % of their time).
//
// Without FINAL the last batch is left to the caller: the queue's length is
// returned.
//
// With TABLE the culling operands are read from `cul` (the volume's blocks,
// or the blocks of this call's offsets); else they are formed from the
// daughter records and the offsets, once per wavefront for the first block
// and once per round for the others.
//
// With TILE the rounds follow one another; else round u starts rounds.at(u)
// tracks past base, and `count` counts the tracks from base on.
//
// With MOVED the volume's units may be moved ones.
template <int U, bool HAS_OFFS, bool COUNT, int KSET, bool SURF, bool FINAL, bool TABLE, bool TILE, bool MOVED>
__device__ __forceinline__ int nav_compact_core(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                                const CullBlock *__restrict__ cul,
                                                const double *__restrict__ offs, const TracksDev &t,
                                                int64_t base, int count, const Rounds &rounds, NavScratch<U> &S,
                                                int lane, unsigned long long *census) {
    int qn = 0;  // queue length (uniform)
    const int nd = v.nd;
    const TileTracks tt = tile_tracks(t, base);
    auto operand = [&](int k0) -> uint4v {
        if (TABLE) return *reinterpret_cast<const uint4v *>(cul[k0 / kCullBlock].a[lane]);
        return cull_operand<HAS_OFFS>(v, dau, offs, k0, lane);
    };
    auto place = [&](int j, int u) { return TILE ? j : rounds.at(u) + (j & 63); };  // (track j, of round u)
    auto load = [&](int j, int u) -> Track {  // (a lane past the end: the last track)
        const int at = place(j, u);
        const unsigned int ju = (unsigned int)(at < count ? at : count - 1);
        return Track{at32(tt.x, ju), at32(tt.y, ju), at32(tt.z, ju), at32(tt.ux, ju), at32(tt.uy, ju), at32(tt.uz, ju)};
    };
    Track next = load(lane, 0);
    uint4v first = {};
    if (nd > 0) first = operand(0);
    constexpr bool SECOND = NavScratch<U>::kSecond && KSET == kSetBasic;
    static_assert(!SECOND || alignof(NavScratch<U>) >= alignof(uint4v), "16-byte accesses of the second block");
    if (SECOND && nd > kCullBlock) *reinterpret_cast<uint4v *>(S.second[lane]) = operand(kCullBlock);
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        if (TILE && u * 64 >= count) break;
        const int j = u * 64 + lane;
        const bool act = place(j, u) < count;
        uint4v a = first;
        Track p = next;
        if (U > 1 && (!TILE || (u + 1) * 64 < count) && u + 1 < U) next = load(j + 64, u + 1);
        if (!TILE && rounds.at(u) >= count) continue;
        int sid;
        const double ms = mother_step<SURF, KSET>(v, p.x, p.y, p.z, p.ux, p.uy, p.uz, sid);
        lds_store(&S.key[j], mother_key(ms));
        lds_store(&S.hit[j], hit_pack(-1, sid));
        if (COUNT) {
            const int n = __popcll(__builtin_amdgcn_ballot_w64(act));
            if (lane == 0) {
                atomicAdd(&census[kCensusTracks], (unsigned long long)n);
                atomicAdd(&census[kCensusCull], (unsigned long long)n * (unsigned long long)nd);
            }
        }
        // a step of 0 from the mother (a start outside it), or one that is
        // not a number, is not beaten
        const bool on = act && ms > 0.0;
        if (nd == 0 || __builtin_amdgcn_ballot_w64(on) == 0ull) continue;
        CullTracks c;
        cull_tracks<MOVED>(v, p.x, p.y, p.z, p.ux, p.uy, p.uz, on, c);
        for (int k0 = 0; k0 < nd; k0 += kCullBlock) {
            if (SECOND && k0 == kCullBlock) {
                a = *reinterpret_cast<const uint4v *>(S.second[lane]);
            } else if (k0 > 0) {
                // waited for here: a wait where the paths join would be for
                // the next round's tracks as well, in the first block too
                a = operand(k0);
                asm volatile("" : "+v"(a));
            }
            unsigned int m = cull_mask(a, c, nd - k0);
            if (!on) m = 0u;
            // each lane with a daughter left appends its lowest, while there is room
            for (;;) {
                const unsigned long long more = __builtin_amdgcn_ballot_w64(m != 0u);
                if (more == 0ull) break;
                const int at = qn + lanes_below(more);
                if (m != 0u && at < kQueueCap) {
                    S.pair[at] = ((unsigned int)(k0 + __builtin_ctz(m)) << 10) | (unsigned int)j;
                    S.x[at] = p.x;
                    S.y[at] = p.y;
                    S.z[at] = p.z;
                    S.ux[at] = p.ux;
                    S.uy[at] = p.uy;
                    S.uz[at] = p.uz;
                    m &= m - 1u;
                }
                qn += __popcll(more);
                if (qn >= kQueueCap) {
                    nav_batch<U, HAS_OFFS, COUNT, KSET, SURF>(dau, offs, S, kQueueCap, lane, census);
                    qn = 0;
                    // the tracks and the operands are read and formed again
                    // rather than kept live through the evaluations (from an
                    // address that is not formed ahead of them either): 104
                    // to 91 VGPRs
                    int again = j;
                    asm volatile("" : "+v"(again));
                    p = load(again, u);
                    if (U > 1) next = load(again + 64, u + 1);
                    if (TABLE) first = operand(0);
                    if (U == 1 || k0 + kCullBlock < nd)
                        cull_tracks<MOVED>(v, p.x, p.y, p.z, p.ux, p.uy, p.uz, on, c);
                }
            }
        }
    }
    if (FINAL && qn > 0) nav_batch<U, HAS_OFFS, COUNT, KSET, SURF>(dau, offs, S, qn, lane, census);
    return qn;
}

// ------------------------------------------------- culling in FP64
// Row of daughter k: its centre T (moved by the offset) and the threshold of
// the expanded test, which evaluates the squared distance from T to the
// half-line less |T|^2 as |p|^2 - 2 p.T - b^2, b = min((p - T).e, 0): every term is
// at most (|p| + |T|)^2, so its rounding is below 16 eps (2 R + 2 |T|)^2 for a
// start inside the mother (R its bounding radius).
template <bool HAS_OFFS>
__device__ __forceinline__ void exact_row(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                          const double *__restrict__ offs, int k, double *row) {
    if (k >= v.nd) {  // never passes
        row[0] = row[1] = row[2] = 0.0;
        row[3] = -__builtin_inf();
        return;
    }
    const DaughterRec &D = dau[k];
    double cx = D.tr[0], cy = D.tr[1], cz = D.tr[2];
    if (HAS_OFFS) {
        cx += offs[3 * k + 0];
        cy += offs[3 * k + 1];
        cz += offs[3 * k + 2];
    }
    const double tt = fma(cz, cz, fma(cy, cy, cx * cx));
    const double span = fma(2.0, fsqrt(tt), 3.0 * v.bound_r);
    row[0] = cx;
    row[1] = cy;
    row[2] = cz;
    row[3] = fma(64.0 * kEps * span, span, fma(D.cull_r, D.cull_r, -tt));
}

// What the tests take of a track: e = d / |d| (0 for a zero direction, or one whose
// |d|^2 overflows: the start point is tested), p.e, |p|^2 and -2 p.
struct ExactTrack {
    double ex, ey, ez, pe, pp, mx, my, mz;
};
__device__ __forceinline__ ExactTrack exact_track(double x, double y, double z, double ux, double uy, double uz) {
    ExactTrack t;
    const double dd = fma(uz, uz, fma(uy, uy, ux * ux));
    const double il = (dd > 0.0 && dd < __builtin_inf()) ? rsqrt_fine(dd) : 0.0;
    t.ex = ux * il;
    t.ey = uy * il;
    t.ez = uz * il;
    t.pe = fma(z, t.ez, fma(y, t.ey, x * t.ex));
    t.pp = fma(z, z, fma(y, y, x * x));
    t.mx = -2.0 * x;
    t.my = -2.0 * y;
    t.mz = -2.0 * z;
    return t;
}

// The lanes that pass daughters g to g + 3: a track's half-line meets the culling
// sphere (kLineTests), it holds the point (kHoldTests), or comes nearer to it than
// `reach` (kNearTests). A lane that is left out has |p|^2 = inf and passes none.
// The rows are loaded together (scalar loads), the four tests independent.
// Without TABLE w = p - T - offset is formed explicitly, as the evaluation forms it.
enum : int { kLineTests, kHoldTests, kNearTests };
template <int WHAT, bool HAS_OFFS, bool TABLE>
__device__ __forceinline__ void exact_tests(const ExactTrack &t, const CullBlock *__restrict__ cul,
                                            const DaughterRec *__restrict__ dau, const double *__restrict__ offs,
                                            int g, int nd, double x, double y, double z, double reach,
                                            unsigned long long (&pass)[4]) {
    double r[4][5], o[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = g + i < nd ? g + i : 0;
        if (TABLE) {
#pragma unroll
            for (int c = 0; c < 4; ++c) r[i][c] = cul[g / kCullBlock].exact[g % kCullBlock + i][c];
            if (WHAT == kNearTests) r[i][4] = dau[k].cull_r;
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[i][c] = dau[k].tr[c];
                o[i][c] = HAS_OFFS ? offs[3 * k + c] : 0.0;
            }
            r[i][3] = dau[k].cull_r;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double f, b = 0.0, lim;
        if (TABLE) {
            f = fma(r[i][2], t.mz, fma(r[i][1], t.my, fma(r[i][0], t.mx, t.pp)));
            if (WHAT == kLineTests) b = fma(-r[i][2], t.ez, fma(-r[i][1], t.ey, fma(-r[i][0], t.ex, t.pe)));
            // (|w| < reach + r: r^2 and the shift are in the row)
            lim = WHAT == kNearTests ? fma(r[i][4], 2.0 * reach, r[i][3]) + reach * reach : r[i][3];
        } else {
            const double wx = x - r[i][0] - o[i][0], wy = y - r[i][1] - o[i][1], wz = z - r[i][2] - o[i][2];
            f = fma(wz, wz, fma(wy, wy, wx * wx));
            if (WHAT == kLineTests) b = fma(wz, t.ez, fma(wy, t.ey, wx * t.ex));
            lim = WHAT == kNearTests ? r[i][3] + reach : r[i][3];
            lim = fma(lim, lim, 64.0 * kEps * f);
        }
        if (WHAT == kLineTests) {
            b = fmin(b, 0.0);
            f = fma(-b, b, f);
        }
        pass[i] = __builtin_amdgcn_ballot_w64(TABLE ? f <= lim : f <= lim && t.pp < __builtin_inf());
        if (!TABLE && g + i >= nd) pass[i] = 0ull;
    }
}

// The navigator of nav_compact_core with these tests, four daughters at a time,
// for volumes with many pairs per track. A round's pairs go into a list
// ((daughter << 6) | lane), daughter by daughter, and from there to the queue with
// their tracks, which are read again (just read: cache hits): a batch then holds
// few daughters, whose records its lanes share, and runs few kinds' code. (The
// queue of nav_compact_core takes each lane's lowest daughter, which fills it in
// fewer steps but mixes the daughters, and its moved starts let large spheres
// behind a start pass. 32 daughters whose spheres meet 3, 10, 20 % of the lines, 2^20
// tracks, nav_compact_core / here: boxes, tubes and cones 41 / 50, 117 / 89, 229 / 149
// us; every kind 150 / 146, 493 / 291, 975 / 431.) What is left of the list at the end
// of a round stays queued.
template <int U, bool HAS_OFFS, bool COUNT, int KSET, bool SURF, bool FINAL, bool TABLE, bool TILE>
__device__ __forceinline__ int nav_exact_core(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                              const CullBlock *__restrict__ cul, const double *__restrict__ offs,
                                              const TracksDev &t, int64_t base, int count, const Rounds &rounds,
                                              NavScratch<U> &S, unsigned short *list, int lane,
                                              unsigned long long *census) {
    int qn = 0;  // queue length (uniform)
    const int nd = v.nd;
    const TileTracks tt = tile_tracks(t, base);
    auto load = [&](int j, int u) -> Track {  // (a lane past the end: the last track)
        const int at = TILE ? j : rounds.at(u) + (j & 63);
        const unsigned int ju = (unsigned int)(at < count ? at : count - 1);
        return Track{at32(tt.x, ju), at32(tt.y, ju), at32(tt.z, ju), at32(tt.ux, ju), at32(tt.uy, ju), at32(tt.uz, ju)};
    };
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        const int start = TILE ? u * 64 : rounds.at(u);
        if (start >= count) continue;
        const int j = u * 64 + lane;
        const bool act = start + lane < count;
        Track p = load(j, u);
        int sid;
        const double ms = mother_step<SURF, KSET>(v, p.x, p.y, p.z, p.ux, p.uy, p.uz, sid);
        lds_store(&S.key[j], mother_key(ms));
        lds_store(&S.hit[j], hit_pack(-1, sid));
        if (COUNT) {
            const int n = __popcll(__builtin_amdgcn_ballot_w64(act));
            if (lane == 0) {
                atomicAdd(&census[kCensusTracks], (unsigned long long)n);
                atomicAdd(&census[kCensusCull], (unsigned long long)n * (unsigned long long)nd);
            }
        }
        const bool on = act && ms > 0.0;
        if (__builtin_amdgcn_ballot_w64(on) == 0ull) continue;
        auto constants = [&]() {
            ExactTrack c = exact_track(p.x, p.y, p.z, p.ux, p.uy, p.uz);
            if (!on) c.pp = __builtin_inf();
            return c;
        };
        ExactTrack c = constants();
        int ln = 0;  // pairs in the list
        for (int g = 0;; g += 4) {
            unsigned long long pass[4] = {0ull, 0ull, 0ull, 0ull};
            int more = 0;
            if (g < nd) {
                exact_tests<kLineTests, HAS_OFFS, TABLE>(c, cul, dau, offs, g, nd, p.x, p.y, p.z, 0.0, pass);
                if (((pass[0] | pass[1]) | (pass[2] | pass[3])) == 0ull) continue;
                more = __popcll(pass[0]) + __popcll(pass[1]) + __popcll(pass[2]) + __popcll(pass[3]);
            }
            if (g >= nd || ln + more > kListCap) {
                for (int lt = 0; lt < ln;) {
                    const int n = ln - lt < kQueueCap - qn ? ln - lt : kQueueCap - qn;
                    if (lane >= qn && lane < qn + n) {
                        const unsigned int e = list[lt + lane - qn];
                        const int je = u * 64 + (int)(e & 63u);
                        const Track q = load(je, u);
                        S.pair[lane] = ((e >> 6) << 10) | (unsigned int)je;
                        S.x[lane] = q.x;
                        S.y[lane] = q.y;
                        S.z[lane] = q.z;
                        S.ux[lane] = q.ux;
                        S.uy[lane] = q.uy;
                        S.uz[lane] = q.uz;
                    }
                    qn += n;
                    lt += n;
                    if (qn == kQueueCap) {
                        nav_batch<U, HAS_OFFS, COUNT, KSET, SURF>(dau, offs, S, kQueueCap, lane, census);
                        qn = 0;
                    }
                }
                ln = 0;
                if (g >= nd) break;
                int again = j;
                asm volatile("" : "+v"(again));  // (see nav_compact_core)
                p = load(again, u);
                c = constants();
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (__builtin_amdgcn_inverse_ballot_w64(pass[i]))
                    list[ln + lanes_below(pass[i])] = (unsigned short)(((g + i) << 6) | lane);
                ln += __popcll(pass[i]);
            }
        }
    }
    if (FINAL && qn > 0) nav_batch<U, HAS_OFFS, COUNT, KSET, SURF>(dau, offs, S, qn, lane, census);
    return qn;
}

// The form that TESTS (kMatrixTests or kAnyTests) and the volume call for; `exact`:
// in FP64, with kAnyTests.
template <int U, bool HAS_OFFS, bool COUNT, int KSET, int TESTS, bool SURF = true, bool FINAL = true,
          bool TABLE = !HAS_OFFS, bool TILE = true>
__device__ __forceinline__ int nav_core(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                        const CullBlock *__restrict__ cul, const double *__restrict__ offs,
                                        const TracksDev &t, int64_t base, int count, NavScratch<U> &S,
                                        unsigned short *list, bool exact, int lane,
                                        unsigned long long *census = nullptr, const Rounds &rounds = Rounds{0, 0}) {
    if (TESTS == kAnyTests && exact)
        return nav_exact_core<U, HAS_OFFS, COUNT, KSET, SURF, FINAL, TABLE, TILE>(v, dau, cul, offs, t, base, count,
                                                                                 rounds, S, list, lane, census);
    return nav_compact_core<U, HAS_OFFS, COUNT, KSET, SURF, FINAL, TABLE, TILE, TESTS == kAnyTests>(
        v, dau, cul, offs, t, base, count, rounds, S, lane, census);
}

// Writes step, hit and (when HITPT) the hit point of the tile's tracks
// from their running minima.
template <int U, bool HITPT>
__device__ __forceinline__ void nav_write(const NavScratch<U> &S, const TracksDev &t, int64_t base,
                                          int count, int lane, double *__restrict__ step,
                                          int32_t *__restrict__ hit, double *__restrict__ hitpt) {
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        const int j = u * 64 + lane;
        if (j < count) {
            const unsigned int ju = (unsigned int)j;
            const double s = key_step(lds_load(&S.key[j]));
            at32(step + base, ju) = s;
            at32(hit + base, ju) = hit_index(lds_load(&S.hit[j]));
            if (HITPT) {
                const int64_t n = t.n;
                const TileTracks tt = tile_tracks(t, base);
                at32(hitpt + base, ju) = fma(s, at32(tt.ux, ju), at32(tt.x, ju));
                at32(hitpt + n + base, ju) = fma(s, at32(tt.uy, ju), at32(tt.y, ju));
                at32(hitpt + 2 * n + base, ju) = fma(s, at32(tt.uz, ju), at32(tt.z, ju));
            }
        }
    }
}

// The navigator of one wavefront's tile, writing its outputs.
template <int U, bool HAS_OFFS, bool HITPT, bool COUNT, int KSET, int TESTS>
__device__ __forceinline__ void nav_compact(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                            const CullBlock *__restrict__ cul,
                                            const double *__restrict__ offs, const TracksDev &t,
                                            int64_t base, int count, NavScratch<U> &S, unsigned short *list,
                                            bool exact, int lane, double *__restrict__ step, int32_t *__restrict__ hit,
                                            double *__restrict__ hitpt,
                                            unsigned long long *census = nullptr) {
    nav_core<U, HAS_OFFS, COUNT, KSET, TESTS, false>(v, dau, cul, offs, t, base, count, S, list, exact, lane, census);
    nav_write<U, HITPT>(S, t, base, count, lane, step, hit, hitpt);
}

// --------------------------------------------- workgroup-pooled last batch
// A tile's last batch holds a few dozen pairs (about 0.12 per track on the
// toy detectors), whose lanes meet every daughter kind the volume holds, so
// that the batch runs each kind's code in turn, each on a few lanes.
// Instead, the W wavefronts of a workgroup pool their last queues: each
// sorts its own queue by kind class; after a barrier the workgroup's pairs
// of each class are cut into batches of 64, and the batches, in class order,
// are dealt to the wavefronts in turn, so that each batch runs one class's
// code. A pair's result (key and packed hit) goes back to its place in the
// owner's queue, over the track it was formed from; after a second barrier
// each wavefront merges its own queue's results into its running minima, as
// a batch of its own would. Without `shared` (uniform over the workgroup:
// its wavefronts' work is too uneven to wait for each other) each wavefront
// runs its own last batch alone, with no barrier. (Sorting a single
// wavefront's queue by class saves nothing: its classes still run one after
// another.)
constexpr int kClassSlots = 8;
template <int W>
struct PoolInfo {
    int cnt[W][kClassSlots];             // pairs of each kind class in each wavefront's queue
    unsigned char order[W][kQueueCap];   // the queue's places, sorted by class
    int first[W];                        // its volume's first daughter record
};

template <int U, int W, bool HAS_OFFS, int KSET, bool SURF>
__device__ __forceinline__ void pool_flush(const DaughterRec *__restrict__ dau_all,
                                           const double *__restrict__ offs, NavScratch<U> *scr, PoolInfo<W> &P,
                                           bool shared, int wave, int first, int qn, int lane) {
    constexpr int NK = kind_classes<KSET>();
    static_assert(NK <= kClassSlots, "class slots");
    static_assert(kQueueCap == 64, "one pair per lane");
    wave = __builtin_amdgcn_readfirstlane(wave);  // (uniform: the batch loop runs on scalars)
    NavScratch<U> &S = scr[wave];
    if (!shared) {
        nav_batch<U, HAS_OFFS, false, KSET, SURF>(dau_all + first, offs, S, qn, lane, nullptr);
        return;
    }
    // the queue's places by class (stable)
    {
        const bool on = lane < qn;
        const int c0 = on ? kind_class<KSET>(dau_all[first + (int)(S.pair[lane] >> 10)].shape.kind) : -1;
        int d = 0, off = 0;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(c0 == c);
            if (c0 == c) d = off + lanes_below(m);
            const int n = __popcll(m);
            if (lane == c) P.cnt[wave][c] = n;
            off += n;
        }
        if (on) P.order[wave][d] = (unsigned char)lane;
        if (lane == 0) P.first[wave] = first;
    }
    __syncthreads();
    // per class: each wavefront's share and the number of batches (uniform
    // values)
    int cn[W][NK], nbc[NK], nb = 0;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            cn[w][c] = __builtin_amdgcn_readfirstlane(P.cnt[w][c]);
            n += cn[w][c];
        }
        nbc[c] = (n + 63) >> 6;
        nb += nbc[c];
    }
    for (int b = wave; b < nb; b += W) {
        // the batch's class and its part within the class
        int c = 0, p = b;
#pragma unroll
        for (int cc = 0; cc < NK - 1; ++cc)
            if (c == cc && p >= nbc[cc]) {
                p -= nbc[cc];
                c = cc + 1;
            }
        const int l = p * 64 + lane;  // the lane's pair within the class
        // the class's pairs run through the wavefronts' sorted queues in
        // order: the owner and the pair's rank in its queue
        int own = 0, rank = 0, pre = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            int before = 0, n = 0;
#pragma unroll
            for (int cc = 0; cc < NK; ++cc) {
                if (cc < c) before += cn[w][cc];
                if (cc == c) n = cn[w][cc];
            }
            if (l >= pre && l < pre + n) {
                own = w;
                rank = before + (l - pre);
            }
            pre += n;
        }
        if (l < pre) {
            NavScratch<U> &O = scr[own];
            const int at = P.order[own][rank];
            const int k = (int)(O.pair[at] >> 10);
            int sid;
            const double s = daughter_dist_out<HAS_OFFS, KSET>(dau_all[P.first[own] + k], offs, k, O.x[at], O.y[at],
                                                               O.z[at], O.ux[at], O.uy[at], O.uz[at], sid, c);
            O.x[at] = __longlong_as_double((long long)step_key(s));
            O.y[at] = __longlong_as_double((long long)hit_pack(k, SURF ? sid : -1));
        }
    }
    __syncthreads();
    // each wavefront merges its own pairs' results
    if (lane < qn)
        merge_key(S, (int)(S.pair[lane] & 1023u), (unsigned long long)__double_as_longlong(S.x[lane]),
                  (int)__double_as_longlong(S.y[lane]));
}

// The navigator of the W tiles of a workgroup (wavefront `wave` holds
// `count` tracks from `base` of volume v (culling blocks `cul`); count may be 0, the wavefront then only taking part in the pooled flush),
// the last flush pooled over the workgroup when `shared`.
template <int U, int W, bool HAS_OFFS, bool HITPT, int KSET, int TESTS>
__device__ __forceinline__ void nav_compact_pooled(const VolumeRec &v, const DaughterRec *__restrict__ dau_all,
                                                   const CullBlock *__restrict__ cul, int first,
                                                   const double *__restrict__ offs, const TracksDev &t,
                                                   int64_t base, int count, NavScratch<U> *scr,
                                                   unsigned short *list, PoolInfo<W> &P, bool shared, int wave, int lane,
                                                   double *__restrict__ step, int32_t *__restrict__ hit,
                                                   double *__restrict__ hitpt) {
    int qn = 0;
    if (count > 0)
        qn = nav_core<U, HAS_OFFS, false, KSET, TESTS, false, false>(v, dau_all + first, cul, offs, t, base, count,
                                                                    scr[wave], list, (v.exact & kLineTasks) != 0, lane);
    pool_flush<U, W, HAS_OFFS, KSET, false>(dau_all, offs, scr, P, shared, wave, first, qn, lane);
    nav_write<U, HITPT>(scr[wave], t, base, count, lane, step, hit, hitpt);
}

// ---------------------------- compacted navigator safety and localization
// The same for the navigator's other two tasks. Safety: a daughter is queued for a point when |w| < s + r
// with s the mother's Safety (the daughter's is at least |w| - r, so
// otherwise it cannot go below the mother's, hence not below the minimum);
// the minimum is merged as a 64-bit key like the step (-0 as +0).
// Localization: a daughter is queued for a point inside the mother when
// |w| <= r; the lowest index of a queued daughter that contains the point
// wins (an integer LDS min). Both tests are the first product of the
// navigator's culling tests alone (|w|^2 - r^2 - delta, less 2 r s + s^2 for
// the safety), one VALU instruction per pair after it, with the same
// operands of the daughters: a start's bound 256 + L holds for the point and
// for s here, and a point where it does not (far outside the mother)
// takes every daughter. The sequential loops report -0 as +0 too, so both
// forms give the same bits.
//
// The mother's Safety alone lets 1.7 pairs per point pass on the toy detector
// (14 for the point of a wavefront that has the most, and its lanes append
// one after another). The nearest daughter bounds the minimum better. With G
// the smallest |w|^2 - r^2 - delta over the daughters, G > 0 puts the point
// outside every sphere, and the nearest daughter's Safety is at most |w| - b
// where a ball of radius b about its centre is solid (the way to the centre
// meets the surface; (|w| - b)^2 <= |w|^2 - b^2), sqrt(|w|^2 + a^2) where its
// hole is a full circle of radius a at z = 0, and |w| + q with q the distance
// of any of its surface's points from the centre. With the volume's largest
// r^2 + c (c = -b^2 or a^2) the minimum is at most sqrt(G + max(r^2 + c)): one
// v_min3 per two pairs and the products once more with s replaced, for 0.83
// pairs per point and 4.6 appends (a CPU simulation), one batch per
// wavefront where there were two.
// Scratch of the safety, per wavefront: running minima, the queue of
// (daughter << 10) | point, and the points, which the queued pairs read back.
constexpr int kPointQueue = 256;
struct PointScratch {
    unsigned long long key[64];
    unsigned int queue[kPointQueue];
    double px[64], py[64], pz[64];
};

// Where the queued pairs read their daughter's record. From the geometry's
// table, one pair per lane, a batch takes a dozen 16-byte loads of up to 64
// cache lines each, and they were what bound the safety: 185,000 lookups of
// the vector cache per CU in the 190,000 cycles of 2^22 points (toy detector),
// 0.55 of the VALU's slots used. From a copy in the workgroup's LDS, in 16-byte
// parts whose odd number per record spreads the records over the banks: 75.4
// to 60.5 us (10^6 points 22.0 to 18.3; 64 daughters, 2^20, 30.8 to 26.8; 8,
// 17.2 to 15.5; every kind 52.0 to 48.9). Boxes, tubes and cones need the front
// 19 parts only (the Safety reads c[0] to c[16]): with a queue of 256 pairs
// seven workgroups of 32 daughters fit a CU, as many as the registers allow.
struct GlobalRecords {
    const DaughterRec *__restrict__ dau;
    static __device__ __forceinline__ void ready() {}
    __device__ __forceinline__ const DaughterRec &operator[](int k) const { return dau[k]; }
};
template <int KSET>
struct LdsRecords {  // (the front Q parts of each record)
    static constexpr int Q = KSET == kSetBasic ? 19 : (int)sizeof(DaughterRec) / 16;
    static_assert(Q % 2 == 1 && Q * 16 >= (int)(offsetof(DaughterRec, shape) + offsetof(ShapeRec, c[17])), "");
    const uint4v *at;
    static __device__ __forceinline__ void ready() { __syncthreads(); }
    __device__ __forceinline__ const DaughterRec &operator[](int k) const {
        return *reinterpret_cast<const DaughterRec *>(at + k * Q);
    }
};
// Copies them, the workgroup's threads side by side, four loads at a time; read
// after ready().
template <int KSET>
__device__ __forceinline__ void lds_records(const DaughterRec *__restrict__ dau, int nd, uint4v *to) {
    constexpr int Q = LdsRecords<KSET>::Q, P = (int)sizeof(DaughterRec) / 16, N = 4;
    const uint4v *from = reinterpret_cast<const uint4v *>(dau);
    const int n = nd * Q, step = (int)blockDim.x;
    for (int i0 = (int)threadIdx.x; i0 < n; i0 += N * step) {
        uint4v r[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const int i = i0 + c * step < n ? i0 + c * step : i0;
            r[c] = from[i / Q * P + i % Q];
        }
#pragma unroll
        for (int c = 0; c < N; ++c)
            if (i0 + c * step < n) to[i0 + c * step] = r[c];
    }
}

template <bool HAS_OFFS, int KSET, typename Records>
__device__ __forceinline__ void point_flush(const Records &dau, const double *__restrict__ offs, PointScratch &S,
                                            int qn, int lane) {
    for (int e0 = 0; e0 < qn; e0 += 64) {
        const int e = e0 + lane;
        if (e < qn) {
            const unsigned int q = S.queue[e];
            const int j = (int)(q & 1023u);
            const int k = (int)(q >> 10);
            const DaughterRec &D = dau[k];
            double wx = lds_load(&S.px[j]) - D.tr[0], wy = lds_load(&S.py[j]) - D.tr[1],
                   wz = lds_load(&S.pz[j]) - D.tr[2];
            if (HAS_OFFS) {
                wx -= offs[3 * k + 0];
                wy -= offs[3 * k + 1];
                wz -= offs[3 * k + 2];
            }
            const double *R = D.rot;
            const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
            const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
            const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
            const unsigned long long key = step_key(any_safety<KSET>(D.shape, D.pcon, lx, ly, lz));
            __hip_atomic_fetch_min(&S.key[j], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
}

// Daughters from which on the bound is formed (toy detector's grid, 2^20
// points: 4 daughters 13.5 us without it and 14.5 with, 32 30.6 and 18.7, 64
// 56.4 and 31.0).
constexpr int kNearest = 8;

// The bound of the minimum from g, the |w|^2 - r^2 - delta of a daughter (in
// the tests' units; widened by more than the products' and the roots'
// rounding): from the smallest, positive ones, as above; a point inside some
// sphere (any negative one) takes |w| + r. A daughter that always passes, far
// below -r^2, bounds nothing.
__device__ __forceinline__ float nearest_bound(const VolumeRec &v, float g) {
    const bool outside = g > 0.0f;
    float b = __builtin_amdgcn_sqrtf(fmaxf(g + (outside ? v.safe_d : v.near_r2), 0.0f));
    if (!outside) b += v.near_r;
    if (v.safe_q >= 0.0f) b = fmaxf(b, __builtin_amdgcn_sqrtf(fmaxf(g + v.safe_r2, 0.0f)) + v.safe_q);
    return g >= -v.near_r2 ? fmaf(b, 0x1p-16f, b) : __builtin_inff();
}

// The safety's last queues pooled over the workgroup's W wavefronts, for
// volumes of more kinds than box, tube and cone, whose Safety takes 200 to 700
// VALU instructions for a cut solid: a batch of one wavefront's queue runs
// the code of every kind it holds in turn. As in the navigators' pooled batch,
// the workgroup's pairs are cut into batches of one kind class, dealt to the
// wavefronts; a result goes into its owner's minimum at once (an LDS minimum
// of the key, whatever the order). Queues of more than kPointPool pairs are
// run by their own wavefront. Every wavefront of the workgroup takes part.
constexpr int kPointPool = 128;
template <int W>
struct PointPool {
    int cnt[W][kClassSlots];
    unsigned char order[W][kPointPool];  // the queue's places, sorted by class
};
template <int W, bool HAS_OFFS, int KSET, typename Records>
__device__ __forceinline__ void point_pool(const Records &dau, const double *__restrict__ offs, PointScratch *scr, PointPool<W> &P, int wave, int qn, int lane) {
    constexpr int NK = kind_classes<KSET>();
    PointScratch &S = scr[wave];
    if (qn > kPointPool) {
        point_flush<HAS_OFFS, KSET>(dau, offs, S, qn, lane);
        qn = 0;
    }
    {
        const bool on0 = lane < qn, on1 = lane + 64 < qn;
        const int c0 = on0 ? kind_class<KSET>(dau[(int)(S.queue[lane] >> 10)].shape.kind) : -1;
        const int c1 = on1 ? kind_class<KSET>(dau[(int)(S.queue[lane + 64] >> 10)].shape.kind) : -1;
        int off = 0;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const unsigned long long m0 = __builtin_amdgcn_ballot_w64(c0 == c);
            const unsigned long long m1 = __builtin_amdgcn_ballot_w64(c1 == c);
            const int n0 = __popcll(m0), n = n0 + __popcll(m1);
            if (c0 == c) P.order[wave][off + lanes_below(m0)] = (unsigned char)lane;
            if (c1 == c) P.order[wave][off + n0 + lanes_below(m1)] = (unsigned char)(lane + 64);
            if (lane == c) P.cnt[wave][c] = n;
            off += n;
        }
    }
    __syncthreads();
    int cn[W][NK], nbc[NK], nb = 0;  // (uniform values)
#pragma unroll
    for (int c = 0; c < NK; ++c) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            cn[w][c] = __builtin_amdgcn_readfirstlane(P.cnt[w][c]);
            n += cn[w][c];
        }
        nbc[c] = (n + 63) >> 6;
        nb += nbc[c];
    }
    for (int b = wave; b < nb; b += W) {
        // from the last class (the costliest code) down
        int c = NK - 1, p = b;
#pragma unroll
        for (int cc = NK - 1; cc > 0; --cc)
            if (c == cc && p >= nbc[cc]) {
                p -= nbc[cc];
                c = cc - 1;
            }
        const int l = p * 64 + lane;  // the lane's pair within the class
        int own = 0, rank = 0, pre = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            int before = 0, n = 0;
#pragma unroll
            for (int cc = 0; cc < NK; ++cc) {
                if (cc < c) before += cn[w][cc];
                if (cc == c) n = cn[w][cc];
            }
            if (l >= pre && l < pre + n) {
                own = w;
                rank = before + (l - pre);
            }
            pre += n;
        }
        if (l < pre) {
            PointScratch &O = scr[own];
            const unsigned int q = O.queue[P.order[own][rank]];
            const int j = (int)(q & 1023u);
            const int k = (int)(q >> 10);
            const DaughterRec &D = dau[k];
            double wx = lds_load(&O.px[j]) - D.tr[0], wy = lds_load(&O.py[j]) - D.tr[1],
                   wz = lds_load(&O.pz[j]) - D.tr[2];
            if (HAS_OFFS) {
                wx -= offs[3 * k + 0];
                wy -= offs[3 * k + 1];
                wz -= offs[3 * k + 2];
            }
            const double *R = D.rot;
            const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
            const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
            const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
            const unsigned long long key = step_key(class_safety<KSET>(c, D.shape, D.pcon, lx, ly, lz));
            __hip_atomic_fetch_min(&O.key[j], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
}

// The tests of a wavefront's 64 points: their columns, and whether a point is
// within their range (else it takes every daughter).
struct PointTests {
    uint4v col[2];
    bool near;
};
// MODE 0: with the mother's Safety `reach`, less the bound of the nearest
// sphere; f receives the length tested with. `a` is the first block's operand,
// operand(k0) the others'.
template <int MODE, bool MOVED, typename Operand>
__device__ __forceinline__ void point_tests(const VolumeRec &v, double x, double y, double z, double reach,
                                            const uint4v &a, Operand operand, float &f, PointTests &T) {
    const int nd = v.nd;
    const double s = MODE == 0 ? v.near_s : v.cull_s;
    const bool moved = MOVED && v.moved;
    float miss = 0.0f;
    if (moved) {  // (a point outside the daughters' sphere is in none)
        x -= v.cx;
        y -= v.cy;
        z -= v.cz;
        if (!(fma(z, z, fma(y, y, x * x)) <= v.out2)) {
            x = y = z = 0.0;
            miss = kCullMiss;
        }
    }
    const float px = (float)(x * s), py = (float)(y * s), pz = (float)(z * s);
    const float pp = fmaf(pz, pz, fmaf(py, py, MOVED ? fmaf(px, px, miss) : px * px));
    CullVector split;
    cull_columns(px, py, pz, pp, 0x54005400u, split, T.col);
    f = MODE == 0 ? (float)(reach * v.near_s) : 0.0f;
    if (MODE == 0 && nd >= kNearest) {
        int g[2] = {0x7f000000, 0x7f000000};  // as integers: any negative result stays the smallest
        uint4v b = a;
        for (int k0 = 0; k0 < nd; k0 += kCullBlock) {
            if (k0 > 0) {
                b = operand(k0);
                asm volatile("" : "+v"(b));  // (waited for here, see nav_compact_core)
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float16v r = cull_product(b, T.col[c]);
#pragma unroll
                for (int i = 0; i < 16; ++i) g[c] = min(g[c], __float_as_int(r[i]));
            }
        }
        const uint2v own = __builtin_amdgcn_permlane32_swap((unsigned int)g[0], (unsigned int)g[1], false, false);
        f = fminf(f, nearest_bound(v, __int_as_float(min((int)own.x, (int)own.y))));
    }
    const float lim = kCullR + (MODE == 0 ? v.near_back : v.cull_back);
    T.near = moved || (pp <= lim * lim && f <= lim);  // (false if not a number)
    if (MODE == 0) cull_columns(split, fmaf(-f, f, pp), f, T.col);
}
// Mask of the block's daughters that pass (left: daughters from its first on).
__device__ __forceinline__ unsigned int point_mask(const uint4v &a, const PointTests &T, int left) {
    unsigned int h[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float16v g = cull_product(a, T.col[c]);
        h[c] = cull_signs<16>([&](int r) { return g[r]; });
    }
    const unsigned int m = cull_merge(h[0], h[1]);
    return T.near ? m : (left >= kCullBlock ? ~0u : (1u << left) - 1u);
}

// Safety of the points base + lane (lane < count), in scr[wave]. With POOL
// every wavefront of the workgroup calls it, one past the last point with
// count 0.
template <bool HAS_OFFS, int KSET, bool POOL, int W, typename Records>
__device__ __forceinline__ void safety_compact(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                              const Records &recs,
                                              const CullBlock *__restrict__ cul,
                                              const double *__restrict__ offs, const TracksDev &t,
                                              int64_t base, int count, PointScratch *scr, PointPool<W> *pool,
                                              int wave, int lane, double *__restrict__ out) {
    PointScratch &S = scr[wave];
    const int nd = v.nd;
    auto operand = [&](int k0) -> uint4v {
        if (!HAS_OFFS) return *reinterpret_cast<const uint4v *>(cul[k0 / kCullBlock].near[lane]);
        return cull_operand<HAS_OFFS, true>(v, dau, offs, k0, lane);
    };
    uint4v a = {};
    if (nd > 0) a = operand(0);
    const bool act = lane < count;
    const int64_t i = act ? base + lane : 0;
    const double x = t.x[i], y = t.y[i], z = t.z[i];
    lds_store(&S.px[lane], x);
    lds_store(&S.py[lane], y);
    lds_store(&S.pz[lane], z);
    const double reach = any_safety<KSET>(v.mother, v.pcon, x, y, z);
    lds_store(&S.key[lane], step_key(reach));
    int qn = 0;
    bool by_daughter = POOL && v.crowded;
    Records::ready();
    if (nd > 0 && count > 0) {
        PointTests T;
        float f;
        point_tests<0, false>(v, x, y, z, reach, a, operand, f, T);
        for (int k0 = 0; k0 < nd; k0 += kCullBlock) {
            unsigned int m = point_mask(a, T, nd - k0);
            if (!act) m = 0u;
            if (k0 + kCullBlock < nd) a = operand(k0 + kCullBlock);
            // each lane with a daughter left appends its lowest; in a crowded
            // volume, and where the queue will be too long to be pooled, the
            // lanes with the lowest lane's do: a batch then holds few daughters
            // (a lane's pairs are counted up to four). Every kind, 2^20 points:
            // 32 daughters whose spheres meet 3 % of the lines 365 to 234 us, in
            // a mother 30 times the detector's size 660 to 329.
            if (POOL) {
                const int c = __popc(m);
                int n = qn;
#pragma unroll
                for (int q = 1; q <= 4; ++q) n += __popcll(__builtin_amdgcn_ballot_w64(c >= q));
                by_daughter = by_daughter || n > kPointPool;
            }
            for (;;) {
                unsigned long long now = __builtin_amdgcn_ballot_w64(m != 0u);
                if (now == 0ull) break;
                if (qn > kPointQueue - 64) {
                    point_flush<HAS_OFFS, KSET>(recs, offs, S, qn, lane);
                    qn = 0;
                }
                if (POOL && by_daughter) {
                    const unsigned int bit =
                        (unsigned int)__builtin_amdgcn_readlane((int)(m & (0u - m)), __ffsll((long long)now) - 1);
                    now = __builtin_amdgcn_ballot_w64((m & bit) != 0u);
                    if ((m & bit) != 0u)
                        S.queue[qn + lanes_below(now)] =
                            ((unsigned int)(k0 + __builtin_ctz(bit)) << 10) | (unsigned int)lane;
                    m &= ~bit;
                } else {
                    if (m != 0u)
                        S.queue[qn + lanes_below(now)] =
                            ((unsigned int)(k0 + __builtin_ctz(m)) << 10) | (unsigned int)lane;
                    m &= m - 1u;
                }
                qn += __popcll(now);
            }
        }
    }
    if constexpr (POOL) point_pool<W, HAS_OFFS, KSET>(recs, offs, scr, *pool, wave, qn, lane);
    else point_flush<HAS_OFFS, KSET>(recs, offs, S, qn, lane);
    if (act) out[base + lane] = key_step(lds_load(&S.key[lane]));
}

// Localization of the points base + u * 64 + lane (u < U, index below `count`
// > 0 past base), as the navigator takes its tracks: a queue of 64 pairs that
// carry their points, run when it is full, each round's points requested a
// round ahead (one round per wavefront waited for its points half its time,
// and ran a batch for the one pair in 64 points that passes).
template <int U>
struct LocateScratch {
    int hit[U * 64];  // lowest daughter; 0x7fffffff none, -2 outside the mother
    unsigned int pair[kQueueCap];
    double x[kQueueCap], y[kQueueCap], z[kQueueCap];
};
template <bool HAS_OFFS, int KSET, int U>
__device__ __forceinline__ void locate_batch(const DaughterRec *__restrict__ dau, const double *__restrict__ offs,
                                             LocateScratch<U> &S, int qn, int lane) {
    if (lane < qn) {
        const unsigned int q = S.pair[lane];
        const int j = (int)(q & 1023u);
        const int k = (int)(q >> 10);
        const DaughterRec &D = dau[k];
        double wx = S.x[lane] - D.tr[0], wy = S.y[lane] - D.tr[1], wz = S.z[lane] - D.tr[2];
        if (HAS_OFFS) {
            wx -= offs[3 * k + 0];
            wy -= offs[3 * k + 1];
            wz -= offs[3 * k + 2];
        }
        const double *R = D.rot;
        const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
        const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
        const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
        if (any_contains<KSET>(D.shape, D.pcon, lx, ly, lz))
            __hip_atomic_fetch_min(&S.hit[j], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
}
template <bool HAS_OFFS, int KSET, int U, bool MOVED>
__device__ __forceinline__ void locate_compact(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                               const CullBlock *__restrict__ cul,
                                               const double *__restrict__ offs, const TracksDev &t,
                                               int64_t base, int count, LocateScratch<U> &S, int lane,
                                               int32_t *__restrict__ out) {
    struct Point {
        double x, y, z;
    };
    const int nd = v.nd;
    const double *tx = t.x + base, *ty = t.y + base, *tz = t.z + base;
    auto operand = [&](int k0) -> uint4v {
        if (!HAS_OFFS) return *reinterpret_cast<const uint4v *>(cul[k0 / kCullBlock].a[lane]);
        return cull_operand<HAS_OFFS>(v, dau, offs, k0, lane);
    };
    auto load = [&](int j) -> Point {  // (a lane past the end: the last point)
        const unsigned int ju = (unsigned int)(j < count ? j : count - 1);
        return Point{at32(tx, ju), at32(ty, ju), at32(tz, ju)};
    };
    int qn = 0;  // queue length (uniform)
    Point next = load(lane);
    uint4v first = {};
    if (nd > 0) first = operand(0);
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        if (u * 64 >= count) break;
        const int j = u * 64 + lane;
        Point p = next;
        if (U > 1 && (u + 1) * 64 < count && u + 1 < U) next = load(j + 64);
        const bool in_m = any_contains<KSET>(v.mother, v.pcon, p.x, p.y, p.z);
        lds_store(&S.hit[j], in_m ? 0x7fffffff : -2);
        const bool on = j < count && in_m;
        if (nd == 0 || __builtin_amdgcn_ballot_w64(on) == 0ull) continue;
        PointTests T;
        float f;
        point_tests<1, MOVED>(v, p.x, p.y, p.z, 0.0, first, operand, f, T);
        uint4v a = first;
        for (int k0 = 0; k0 < nd; k0 += kCullBlock) {
            if (k0 > 0) {
                a = operand(k0);
                asm volatile("" : "+v"(a));  // (waited for here, see nav_compact_core)
            }
            unsigned int m = point_mask(a, T, nd - k0);
            if (!on) m = 0u;
            // each lane with a daughter left appends its lowest, while there is room
            for (;;) {
                const unsigned long long more = __builtin_amdgcn_ballot_w64(m != 0u);
                if (more == 0ull) break;
                const int at = qn + lanes_below(more);
                if (m != 0u && at < kQueueCap) {
                    S.pair[at] = ((unsigned int)(k0 + __builtin_ctz(m)) << 10) | (unsigned int)j;
                    S.x[at] = p.x;
                    S.y[at] = p.y;
                    S.z[at] = p.z;
                    m &= m - 1u;
                }
                qn += __popcll(more);
                if (qn >= kQueueCap) {
                    locate_batch<HAS_OFFS, KSET, U>(dau, offs, S, kQueueCap, lane);
                    qn = 0;
                    // the points are read again (from an address that is not
                    // formed ahead of the batch)
                    int again = j;
                    asm volatile("" : "+v"(again));
                    p = load(again);
                }
            }
        }
    }
    if (qn > 0) locate_batch<HAS_OFFS, KSET, U>(dau, offs, S, qn, lane);
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        const int j = u * 64 + lane;
        if (j < count) {
            const int w = lds_load(&S.hit[j]);
            at32(out + base, (unsigned int)j) = w != 0x7fffffff ? w : -1;
        }
    }
}

// Both with the tests in FP64, one round of 64 points per wavefront: the pairs are
// listed daughter by daughter and read their points from the wavefront's copy.
struct ExactPoints {
    unsigned long long key[64];       // the safety's running minima, or
    int hit[64];                      // the localization's (see LocateScratch)
    unsigned int list[2 * kListCap];  // (daughter << 6) | point
    double x[64], y[64], z[64];
};
template <bool SAFETY, bool HAS_OFFS, int KSET, typename Out>
__device__ __forceinline__ void points_exact(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                             const CullBlock *__restrict__ cul, const double *__restrict__ offs,
                                             const TracksDev &t, int64_t base, int count, ExactPoints &S, int lane,
                                             Out *__restrict__ out) {
    const int nd = v.nd;
    const bool act = lane < count;
    const int64_t i = base + (act ? lane : 0);
    const double x = t.x[i], y = t.y[i], z = t.z[i];
    lds_store(&S.x[lane], x);
    lds_store(&S.y[lane], y);
    lds_store(&S.z[lane], z);
    double reach = 0.0;
    bool test = act;
    if (SAFETY) {
        reach = any_safety<KSET>(v.mother, v.pcon, x, y, z);
        lds_store(&S.key[lane], step_key(reach));
    } else {
        const bool in_m = any_contains<KSET>(v.mother, v.pcon, x, y, z);
        lds_store(&S.hit[lane], in_m ? 0x7fffffff : -2);
        test = act && in_m;
    }
    if (__builtin_amdgcn_ballot_w64(test) != 0ull) {
        ExactTrack c = exact_track(x, y, z, 0.0, 0.0, 0.0);
        if (!test) c.pp = __builtin_inf();
        int ln = 0;
        for (int g = 0;; g += 4) {
            if (g >= nd || ln > kListCap) {
                for (int e0 = 0; e0 < ln; e0 += 64) {
                    if (e0 + lane < ln) {
                        const unsigned int e = S.list[e0 + lane];
                        const int j = (int)(e & 63u), k = (int)(e >> 6);
                        const DaughterRec &D = dau[k];
                        double wx = lds_load(&S.x[j]) - D.tr[0], wy = lds_load(&S.y[j]) - D.tr[1],
                               wz = lds_load(&S.z[j]) - D.tr[2];
                        if (HAS_OFFS) {
                            wx -= offs[3 * k + 0];
                            wy -= offs[3 * k + 1];
                            wz -= offs[3 * k + 2];
                        }
                        const double *R = D.rot;
                        const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
                        const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
                        const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
                        if (SAFETY)
                            __hip_atomic_fetch_min(&S.key[j], step_key(any_safety<KSET>(D.shape, D.pcon, lx, ly, lz)),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                        else if (any_contains<KSET>(D.shape, D.pcon, lx, ly, lz))
                            __hip_atomic_fetch_min(&S.hit[j], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    }
                }
                ln = 0;
                if (g >= nd) break;
            }
            unsigned long long pass[4];
            exact_tests<SAFETY ? kNearTests : kHoldTests, HAS_OFFS, !HAS_OFFS>(c, cul, dau, offs, g, nd, x, y, z, reach, pass);
            if (((pass[0] | pass[1]) | (pass[2] | pass[3])) == 0ull) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (__builtin_amdgcn_inverse_ballot_w64(pass[q]))
                    S.list[ln + lanes_below(pass[q])] = (unsigned int)(((g + q) << 6) | lane);
                ln += __popcll(pass[q]);
            }
        }
    }
    if (!act) return;
    if (SAFETY) {
        out[base + lane] = key_step(lds_load(&S.key[lane]));
    } else {
        const int w = lds_load(&S.hit[lane]);
        out[base + lane] = w != 0x7fffffff ? w : -1;
    }
}

// ------------------------------------------ navigator safety and locate
// The navigator's other two per-track tasks (section 3), sequential form
// with every daughter evaluated (culling off; the culled kernels take the
// compacted form above).
template <bool HAS_OFFS, int KSET = kSetAll>
__device__ __forceinline__ double nav_safety(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                             const double *__restrict__ offs, double x, double y,
                                             double z) {
    double best = any_safety<KSET>(v.mother, v.pcon, x, y, z);
    const int nd = v.nd;
    for (int k = 0; k < nd; ++k) {
        const DaughterRec &D = dau[k];
        double wx = x - D.tr[0], wy = y - D.tr[1], wz = z - D.tr[2];
        if (HAS_OFFS) {
            wx -= offs[3 * k + 0];
            wy -= offs[3 * k + 1];
            wz -= offs[3 * k + 2];
        }
        const double *R = D.rot;
        const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
        const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
        const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
        best = fmin(best, any_safety<KSET>(D.shape, D.pcon, lx, ly, lz));
    }
    return best == 0.0 ? 0.0 : best;  // -0 reported as +0
}

// Daughter holding the point (lowest index), -1 for the mother's own part,
// -2 outside the mother.
template <bool HAS_OFFS, int KSET = kSetAll>
__device__ __forceinline__ int nav_locate(const VolumeRec &v, const DaughterRec *__restrict__ dau,
                                          const double *__restrict__ offs, double x, double y,
                                          double z) {
    int where = any_contains<KSET>(v.mother, v.pcon, x, y, z) ? -1 : -2;
    const int nd = v.nd;
    for (int k = 0; k < nd; ++k) {
        if (__ballot(where == -1) == 0) break;  // every lane placed
        const DaughterRec &D = dau[k];
        double wx = x - D.tr[0], wy = y - D.tr[1], wz = z - D.tr[2];
        if (HAS_OFFS) {
            wx -= offs[3 * k + 0];
            wy -= offs[3 * k + 1];
            wz -= offs[3 * k + 2];
        }
        const double *R = D.rot;
        const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
        const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
        const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
        const bool in = any_contains<KSET>(D.shape, D.pcon, lx, ly, lz);
        where = (where == -1 && in) ? k : where;
    }
    return where;
}

}  // namespace gn
