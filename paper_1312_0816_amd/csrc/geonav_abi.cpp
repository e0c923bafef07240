// C ABI of libgeonav: argument validation, the geometry handle (device copies
// of the volumes with host-derived shape constants), the batched scheduler
// (cost-sorted baskets, device-side tile expansion, a cached HIP graph), the
// launch-shape autotuner and error reporting.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <new>
#include <sstream>
#include <string>
#include <vector>

#include "geonav.h"
#include "geonav_internal.hpp"

using namespace gn;

namespace {

thread_local std::string g_last_msg;
thread_local int g_last_code = 0;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_msg = buf;
    g_last_code = code;
    return code;
}

int hip_fail(hipError_t e, const char *where) {
    return fail(GEO_ERR_HIP, "%s: %s", where, hipGetErrorString(e));
}

#define GN_HIP(call)                                      \
    do {                                                  \
        hipError_t e_ = (call);                           \
        if (e_ != hipSuccess) return hip_fail(e_, #call); \
    } while (0)

// Relative slack of the range tests at candidate hit points (see "Edges" in
// geonav_device.hpp).
constexpr double kEdgeSlack = 1e-12;

// Parameters each kind reads (the rest of par[] is ignored).
static_assert(GEO_CENSUS_SLOTS == kCensusSlots, "census layout");
static_assert(GEO_MAX_DAUGHTERS == kMaxDaughters, "daughters per volume");

int nparams(const geo_shape &s) {
    switch (s.kind) {
        case GEO_BOX:
        case GEO_TUBE: return 3;
        case GEO_CONE:
        case GEO_TUBS: return 5;
        case GEO_CONS: return 7;
        case GEO_PCON: {
            const double nz = s.par[2];
            if (!(nz >= 2 && nz <= GEO_PCON_MAX_PLANES && nz == std::floor(nz))) return -1;
            return 3 + 3 * (int)nz;
        }
        default: return 0;
    }
}

// Polycone sections: planes (z, rmin, rmax) from par[3..], validated.
int make_pcon(const double *p, PconRec &pc, double *bound_r, const char *what) {
    std::memset(&pc, 0, sizeof pc);
    const int nz = (int)p[2];
    pc.nz = nz;
    double rm = 0;
    for (int j = 0; j < nz; ++j) {
        pc.z[j] = p[3 + 3 * j];
        pc.rin[j] = p[4 + 3 * j];
        pc.rout[j] = p[5 + 3 * j];
        if (!(pc.rin[j] >= 0 && pc.rin[j] <= pc.rout[j]))
            return fail(GEO_ERR_INVALID_ARG, "%s: polycone plane %d needs 0 <= rmin <= rmax", what, j);
        if (j > 0 && !(pc.z[j] > pc.z[j - 1]))
            return fail(GEO_ERR_INVALID_ARG, "%s: polycone z must increase strictly (plane %d)", what, j);
        rm = std::max(rm, pc.rout[j]);
    }
    for (int j = 0; j + 1 < nz; ++j) {
        if (!(pc.rout[j] + pc.rout[j + 1] > 0))
            return fail(GEO_ERR_INVALID_ARG, "%s: polycone section %d has rmax 0 at both planes", what, j);
        const double h = pc.z[j + 1] - pc.z[j];
        const double bo = (pc.rout[j + 1] - pc.rout[j]) / h;
        const double bi = (pc.rin[j + 1] - pc.rin[j]) / h;
        pc.bo[j] = bo;
        pc.ao[j] = pc.rout[j] - bo * pc.z[j];
        if (pc.rin[j] > 0 || pc.rin[j + 1] > 0) {
            pc.hole_mask |= 1 << j;
            pc.bi[j] = bi;
            pc.ai[j] = pc.rin[j] - bi * pc.z[j];
        }
        pc.inv_eo[j] = 1.0 / ((pc.rout[j + 1] - pc.rout[j]) * (pc.rout[j + 1] - pc.rout[j]) + h * h);
        pc.inv_ei[j] = 1.0 / ((pc.rin[j + 1] - pc.rin[j]) * (pc.rin[j + 1] - pc.rin[j]) + h * h);
    }
    const double zm = std::max(std::fabs(pc.z[0]), std::fabs(pc.z[nz - 1]));
    pc.eps = kEdgeSlack * (zm + rm);
    auto lo2 = [&](double r) { return r > pc.eps ? (r - pc.eps) * (r - pc.eps) : 0.0; };
    auto hi2 = [&](double r) { return (r + pc.eps) * (r + pc.eps); };
    pc.rin2_0 = lo2(pc.rin[0]);
    pc.rout2_0 = hi2(pc.rout[0]);
    pc.rin2_l = lo2(pc.rin[nz - 1]);
    pc.rout2_l = hi2(pc.rout[nz - 1]);
    const double br = std::sqrt(rm * rm + zm * zm);
    pc.far2 = br * (1.0 + 1e-6) * (br * (1.0 + 1e-6));
    if (bound_r) *bound_r = br;
    return GEO_OK;
}

// Base solid of a shape record: box, tube or cone constants.
int make_base(int kind, const double *p, ShapeRec &out, double *bound_r, const char *what) {
    switch (kind) {
        case GEO_BOX:
            if (!(p[0] > 0 && p[1] > 0 && p[2] > 0))
                return fail(GEO_ERR_INVALID_ARG, "%s: box half-lengths must be > 0", what);
            out.c[0] = p[0];
            out.c[1] = p[1];
            out.c[2] = p[2];
            {
                const double br = std::sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
                const double eps = kEdgeSlack * br;
                out.c[21] = eps;
                for (int i = 0; i < 3; ++i) out.c[3 + i] = p[i] + eps;
                if (bound_r) *bound_r = br;
            }
            return GEO_OK;
        case GEO_TUBE:
            if (!(p[0] >= 0 && p[1] > 0 && p[0] <= p[1] && p[2] > 0))
                return fail(GEO_ERR_INVALID_ARG, "%s: tube needs 0 <= rmin <= rmax, rmax > 0, dz > 0",
                            what);
            out.hole = p[0] > 0 ? 1 : 0;
            out.c[0] = p[0];
            out.c[1] = p[1];
            out.c[2] = p[2];
            out.c[3] = p[0] * p[0];
            out.c[4] = p[1] * p[1];
            {
                const double br = std::sqrt(p[1] * p[1] + p[2] * p[2]);
                const double eps = kEdgeSlack * br;
                out.c[21] = eps;
                out.c[5] = p[2] + eps;
                out.c[6] = p[0] > eps ? (p[0] - eps) * (p[0] - eps) : 0.0;
                out.c[7] = (p[1] + eps) * (p[1] + eps);
                if (bound_r) *bound_r = br;
            }
            return GEO_OK;
        default: {  // GEO_CONE
            const double dz = p[0], rmin1 = p[1], rmax1 = p[2], rmin2 = p[3], rmax2 = p[4];
            if (!(dz > 0 && rmin1 >= 0 && rmin2 >= 0 && rmin1 <= rmax1 && rmin2 <= rmax2 &&
                  rmax1 + rmax2 > 0))
                return fail(GEO_ERR_INVALID_ARG,
                            "%s: cone needs dz > 0, 0 <= rmin <= rmax at both ends, rmax1 + rmax2 > 0",
                            what);
            out.hole = (rmin1 > 0 || rmin2 > 0) ? 1 : 0;
            const double bo = (rmax2 - rmax1) / (2 * dz), bi = (rmin2 - rmin1) / (2 * dz);
            out.c[0] = dz;
            out.c[1] = 0.5 * (rmax1 + rmax2);
            out.c[2] = bo;
            out.c[3] = 0.5 * (rmin1 + rmin2);
            out.c[4] = bi;
            out.c[5] = rmin1;
            out.c[6] = rmax1;
            out.c[7] = rmin2;
            out.c[8] = rmax2;
            out.c[9] = rmin1 * rmin1;
            out.c[10] = rmax1 * rmax1;
            out.c[11] = rmin2 * rmin2;
            out.c[12] = rmax2 * rmax2;
            out.c[13] = 1.0 / std::sqrt(1.0 + bo * bo);
            out.c[14] = 1.0 / std::sqrt(1.0 + bi * bi);
            out.c[15] = 1.0 / ((rmax2 - rmax1) * (rmax2 - rmax1) + 4 * dz * dz);
            out.c[16] = 1.0 / ((rmin2 - rmin1) * (rmin2 - rmin1) + 4 * dz * dz);
            {
                const double rm = std::max(rmax1, rmax2);
                const double br = std::sqrt(rm * rm + dz * dz);
                const double eps = kEdgeSlack * br;
                auto lo2 = [&](double r) { return r > eps ? (r - eps) * (r - eps) : 0.0; };
                auto hi2 = [&](double r) { return (r + eps) * (r + eps); };
                out.c[21] = eps;
                out.c[22] = dz + eps;
                out.c[23] = lo2(rmin1);
                out.c[24] = hi2(rmax1);
                out.c[25] = lo2(rmin2);
                out.c[26] = hi2(rmax2);
                if (bound_r) *bound_r = br;
            }
            return GEO_OK;
        }
    }
}

// Validate a shape and derive its device record (and, for a polycone, its
// sections in *pc, which must then be non-NULL). A segment or polycone whose
// range is a full turn (dphi == 2 pi) is stored uncut.
// The equal-radii cone (segment) of a tube (segment): the same solid.
geo_shape as_cone(const geo_shape &s) {
    geo_shape c = s;
    c.kind = s.kind == GEO_TUBE ? GEO_CONE : GEO_CONS;
    c.par[0] = s.par[2];  // dz
    c.par[1] = c.par[3] = s.par[0];  // rmin at both ends
    c.par[2] = c.par[4] = s.par[1];  // rmax at both ends
    if (s.kind == GEO_TUBS) {
        c.par[5] = s.par[3];  // phi1
        c.par[6] = s.par[4];  // dphi
    }
    return c;
}

int make_shape(const geo_shape &s, ShapeRec &out, PconRec *pc, double *bound_r, const char *what) {
    std::memset(&out, 0, sizeof out);
    const int np = nparams(s);
    if (np == 0) return fail(GEO_ERR_INVALID_ARG, "%s: unknown shape kind %d", what, s.kind);
    if (np < 0)
        return fail(GEO_ERR_INVALID_ARG, "%s: polycone needs an integral nz in 2..%d", what,
                    GEO_PCON_MAX_PLANES);
    for (int i = 0; i < np; ++i)
        if (!std::isfinite(s.par[i])) return fail(GEO_ERR_INVALID_ARG, "%s: non-finite shape parameter", what);
    const double *p = s.par;
    const bool pcon = s.kind == GEO_PCON;
    const bool seg = s.kind == GEO_TUBS || s.kind == GEO_CONS || pcon;
    const int base = s.kind == GEO_TUBS ? GEO_TUBE : s.kind == GEO_CONS ? GEO_CONE : s.kind;
    int rc;
    if (pcon) {
        if (!pc) return fail(GEO_ERR_INVALID_ARG, "%s: internal: no polycone record", what);
        rc = make_pcon(p, *pc, bound_r, what);
        out.hole = pc->hole_mask != 0;
    } else {
        rc = make_base(base, p, out, bound_r, what);
    }
    if (rc != GEO_OK || !seg) {
        out.kind = base;
        return rc;
    }
    const double two_pi = 2.0 * M_PI;
    const double phi1 = pcon ? p[0] : p[np - 2], dphi = pcon ? p[1] : p[np - 1];
    if (!(dphi > 0 && dphi <= two_pi))
        return fail(GEO_ERR_INVALID_ARG, "%s: segment needs 0 < dphi <= 2 pi", what);
    if (dphi == two_pi) {
        out.kind = pcon ? kPcon : base;
        return GEO_OK;
    }
    out.kind = pcon ? kPcons : s.kind;
    out.convex = dphi <= M_PI ? 1 : 0;
    const double phi2 = phi1 + dphi;
    out.c[17] = std::cos(phi1);
    out.c[18] = std::sin(phi1);
    out.c[19] = std::cos(phi2);
    out.c[20] = std::sin(phi2);
    return GEO_OK;
}

// What bounds a shape's Safety at a point outside its bounding sphere, |w|
// from its centre: plain, sqrt(|w|^2 + c); else |w| + q.
struct SafetyBound {
    bool plain;
    double c, q;
};
SafetyBound safety_bound(const geo_shape &s, const ShapeRec &rec) {
    const double *p = s.par;
    if (rec.kind == kBox) {
        const double b = std::min(p[0], std::min(p[1], p[2]));
        return {true, -b * b, 0};
    }
    if (rec.kind == kPcon || rec.kind == kPcons) {  // a corner of the profile
        double q = HUGE_VAL;
        for (int j = 0; j < (int)p[2]; ++j) q = std::min(q, std::hypot(p[3 + 3 * j], p[5 + 3 * j]));
        return {false, 0, q};
    }
    // tubes and cones (segments): radii at z = 0
    const bool tube = s.kind == GEO_TUBE || s.kind == GEO_TUBS;
    const double dz = tube ? p[2] : p[0];
    const double a = tube ? p[0] : 0.5 * (p[1] + p[3]), o = tube ? p[1] : 0.5 * (p[2] + p[4]);
    if (rec.kind == kTubs || rec.kind == kCons) return {false, 0, a};  // where the inner radius meets a face
    if (rec.hole) return {true, a * a, 0};
    const double slope = tube ? 0 : (p[4] - p[2]) / (2 * dz);
    const double b = std::min(dz, o / std::sqrt(1 + slope * slope));
    return {true, -b * b, 0};
}

// Surface area of the box or cylinder that holds a mother (uncut).
double mother_area(const geo_shape &s) {
    const double *p = s.par;
    double r = 0, h = 0;  // radius and height of the cylinder
    switch (s.kind) {
        case GEO_BOX: return 8 * (p[0] * p[1] + p[1] * p[2] + p[2] * p[0]);
        case GEO_TUBE:
        case GEO_TUBS: r = p[1], h = 2 * p[2]; break;
        case GEO_CONE:
        case GEO_CONS: r = std::max(p[2], p[4]), h = 2 * p[0]; break;
        default: {
            const int nz = (int)p[2];
            for (int j = 0; j < nz; ++j) r = std::max(r, p[5 + 3 * j]);
            h = p[3 * nz] - p[3];
        }
    }
    return 2 * M_PI * r * (r + h);
}

// Volume of the same.
double mother_volume(const geo_shape &s) {
    const double *p = s.par;
    switch (s.kind) {
        case GEO_BOX: return 8 * p[0] * p[1] * p[2];
        case GEO_TUBE:
        case GEO_TUBS: return 2 * M_PI * p[1] * p[1] * p[2];
        case GEO_CONE:
        case GEO_CONS: return 2 * M_PI * p[0] * std::max(p[2], p[4]) * std::max(p[2], p[4]);
    }
    const int nz = (int)p[2];
    double r = 0;
    for (int j = 0; j < nz; ++j) r = std::max(r, p[5 + 3 * j]);
    return M_PI * r * r * (p[3 * nz] - p[3]);
}

// Pairs per track that pass the tests on the matrix cores for their widening of
// r^2 alone, in units of 1 / s about the centre c with a start moved back by
// `back`, for lines through the daughters' centres in all directions (the mean
// over at most 64 of them): a line through one centre passes within r of another
// at distance d with probability r^2 / (2 d^2).
double unresolved(const DaughterRec *dau, int nd, double s, const double *c, double back) {
    const double reach = kCullR + back, s2 = s * s;
    const int step = (nd + 63) / 64;
    double sum = 0;
    int n = 0;
    for (int j = 0; j < nd; j += step, ++n) {
        const double *a = dau[j].tr;
        for (int k = 0; k < nd; ++k) {
            if (k == j) continue;
            const double *b = dau[k].tr;
            const double x = b[0] - a[0], y = b[1] - a[1], z = b[2] - a[2];
            const double u = b[0] - c[0], v = b[1] - c[1], w = b[2] - c[2];
            const double d2 = 2 * (x * x + y * y + z * z) * s2, r2 = dau[k].cull_r * dau[k].cull_r * s2;
            const double wide = r2 + 0x1p-15 * (reach * reach + (u * u + v * v + w * w) * s2);
            if (d2 > 0) sum += (std::min(d2, wide) - std::min(d2, r2)) / d2;
        }
    }
    return n > 0 ? sum / n : 0;
}

// Daughters that one round of 64 points tests at little cost.
constexpr int kRoundsFew = 11;

// How the tasks on volume r cull: the units of the tests, and what a line or a
// point meets of the daughters decides which tests and whether any.
void choose_culling(VolumeRec &r, const DaughterRec *dau, const geo_shape &mother, bool basic) {
    const double origin[3] = {0, 0, 0};
    const int blocks = (r.nd + kCullBlock - 1) / kCullBlock;
    r.cull_s = r.near_s;
    r.cull_back = r.near_back;
    // (squares and products of lengths stay normal numbers)
    if (r.nd == 0 || !(r.near_s > 0) || !(r.bound_r > 1e-20 && r.bound_r < 1e20)) return;
    double lost = unresolved(dau, r.nd, r.near_s, origin, r.near_back);
    // Daughters that the mother's units do not resolve: their own, which cost a
    // round of 64 tracks about as much as 0.04 pairs per track. The sphere is
    // taken a third larger than they need, for what offsets move.
    if (lost > 0.04 * blocks) {
        double lo[3], hi[3], c[3], big = 0, most = 0;
        for (int i = 0; i < 3; ++i) {
            lo[i] = HUGE_VAL, hi[i] = -HUGE_VAL;
            for (int k = 0; k < r.nd; ++k) {
                lo[i] = std::min(lo[i], dau[k].tr[i] - dau[k].cull_r);
                hi[i] = std::max(hi[i], dau[k].tr[i] + dau[k].cull_r);
            }
            c[i] = 0.5 * (lo[i] + hi[i]);
        }
        for (int k = 0; k < r.nd; ++k) {
            const double x = dau[k].tr[0] - c[0], y = dau[k].tr[1] - c[1], z = dau[k].tr[2] - c[2];
            big = std::max(big, std::sqrt(x * x + y * y + z * z) + dau[k].cull_r);
            most = std::max(most, dau[k].cull_r);
        }
        const double scale = 0.75 * kCullR / big;
        const double far = (std::sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]) + r.bound_r) * scale;
        if (scale > 2 * r.near_s && far <= 0x1p26) {
            r.moved = 1;
            r.cull_s = scale;
            r.cx = c[0], r.cy = c[1], r.cz = c[2];
            r.out2 = kCullR / scale * (kCullR / scale);
            r.cull_back = (float)(most * scale * (1.0 + 1e-6) + 0.25);
            lost = unresolved(dau, r.nd, scale, c, r.cull_back);
        }
    }
    // Still not resolved (daughters in clusters far apart): the tests in FP64. (The
    // toy detector in a mother 10, 20 and 30 times its size, in the mother's
    // units, 0.15, 0.59 and 1.3 pairs lost: navigator 64, 99 and 164 us at 2^22
    // tracks, in FP64 101; localization 7.9, 8.3, 11.3 us at 2^20, in FP64 9.9.)
    if (lost > 0.5 * blocks) r.exact |= kLineTasks;
    if (lost > blocks) r.exact |= kLocateTask;
    // A line through a convex mother meets a sphere inside it with the ratio of
    // their surfaces as probability, a point is in it with that of their volumes.
    // The more of the daughters (ratios of the mean daughter) a track meets, the
    // more pairs are queued, until walking all daughters in lockstep costs less.
    // The lines are where two forms crossed, for boxes, tubes and cones and for
    // more kinds (whose batches run more code), with 8, 32 and 64 daughters, 2^20
    // tracks (us: matrix cores, FP64, lockstep):
    //   navigator, 32 daughters, ratio 0.03  41  50 140; 0.06  73  66 140;
    //                                  0.15 176 119 140; 0.20 229 149 140;
    //     every kind             0.03 150 146 271; 0.06 296 219; 0.10 493 291 271;
    //   localization, ratio of surfaces 0.06 16.7 22 41; 0.10 25 21.5; 0.20 57 36; 0.30 94 54 42;
    //     every kind             0.06 38 39 71; 0.10 68 63; 0.15 112 85 73;
    //     8 daughters 0.10 11.2 11.7, every kind 19.4 26;
    //   safety (matrix cores, lockstep) 0.10 67 86; 0.20 85 86; 0.30 100 86;
    //     every kind             0.01 133 228; 0.03 235 228; 0.06 ~285 228.
    // The adjoint's lines are the navigator's.
    double met = 0, held = 0;
    for (int k = 0; k < r.nd; ++k) {
        const double rk = dau[k].cull_r;
        met += std::min(1.0, 4 * M_PI * rk * rk / mother_area(mother)) / r.nd;
        held += std::min(1.0, 4 * M_PI / 3 * rk * rk * rk / mother_volume(mother)) / r.nd;
    }
    if (met > (basic ? 0.045 : 0.027)) r.exact |= kLineTasks;
    if (held > (basic ? 0.034 : 0.026) * (r.nd > kRoundsFew ? 1 : 2)) r.exact |= kLocateTask;
    r.rounds = r.nd > kRoundsFew || held * r.nd > 0.02;
    if (met > (basic ? 0.16 : 0.08)) r.dense |= kLineTasks;
    if (held > (basic ? 0.124 : 0.044)) r.dense |= kLocateTask;
    if (met > (basic ? 0.17 : 0.04)) r.dense |= kSafetyTask;
    if (met > 0.015) r.crowded = 1;
}

int check_rotation(const double *r, const char *what) {
    for (int i = 0; i < 9; ++i)
        if (!std::isfinite(r[i])) return fail(GEO_ERR_INVALID_ARG, "%s: non-finite rotation", what);
    double worst = 0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double s = 0;
            for (int k = 0; k < 3; ++k) s += r[3 * k + i] * r[3 * k + j];
            worst = std::max(worst, std::fabs(s - (i == j ? 1.0 : 0.0)));
        }
    const double det = r[0] * (r[4] * r[8] - r[5] * r[7]) - r[1] * (r[3] * r[8] - r[5] * r[6]) +
                       r[2] * (r[3] * r[7] - r[4] * r[6]);
    if (worst > 1e-12 || det <= 0)
        return fail(GEO_ERR_INVALID_ARG, "%s: rotation not proper orthonormal (|R^T R - I| = %g, det = %g)",
                    what, worst, det);
    return GEO_OK;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_tracks(const geo_tracks &t, bool need_dir, const char *what) {
    if (t.n < 0) return fail(GEO_ERR_INVALID_ARG, "%s: n < 0", what);
    if (t.n == 0) return GEO_OK;
    const double *ps[6] = {t.x, t.y, t.z, t.ux, t.uy, t.uz};
    for (int i = 0; i < (need_dir ? 6 : 3); ++i) {
        if (!ps[i]) return fail(GEO_ERR_INVALID_ARG, "%s: NULL track array with n > 0", what);
        if (!aligned(ps[i], 8)) return fail(GEO_ERR_INVALID_ARG, "%s: track array not 8-byte aligned", what);
    }
    return GEO_OK;
}

int check_out(const void *p, size_t align, const char *what) {
    if (!p) return fail(GEO_ERR_INVALID_ARG, "%s is NULL", what);
    if (!aligned(p, align)) return fail(GEO_ERR_INVALID_ARG, "%s is misaligned", what);
    return GEO_OK;
}

int check_opt(const void *p, size_t align, const char *what) {
    if (p && !aligned(p, align)) return fail(GEO_ERR_INVALID_ARG, "%s is misaligned", what);
    return GEO_OK;
}

TracksDev to_dev(const geo_tracks &t) { return TracksDev{t.x, t.y, t.z, t.ux, t.uy, t.uz, t.n}; }

}  // namespace

// ------------------------------------------------------------ the handle
struct geo_geometry {
    int device = 0;
    int num_cus = 0;
    std::string device_name;
    int nvol = 0;
    int max_nd = 0;
    std::vector<VolumeRec> h_vols;
    VolumeRec *d_vols = nullptr;
    DaughterRec *d_dau = nullptr;
    CullBlock *d_cull = nullptr;
    CullBlock *d_shift = nullptr;    // a volume's culling blocks moved by an adjoint call's offsets
    PconRec *d_pcon = nullptr;       // polycone sections of mothers and daughters
    // kinds each volume holds (kSetBasic, kSetSeg, kSetAll) and their union:
    // the navigator kernels are specialised to carry only those
    std::vector<int> vol_kset;
    int kset = kSetBasic;
    // adjoint partial sums: kBackwardMaxBlocks x 3 x max_nd
    double *d_partial = nullptr;
    // batched state
    int tracks_per_lane = 4;
    int waves_per_simd = 0;  // hardware-scheduled until geo_autotune picks
    bool use_graph = false;  // batched kernels as two launches until geo_autotune picks
    bool any_tests = false;         // a volume has kAnyTests for its lines
    bool cull = true;               // wavefront bounding-sphere culling in the navigators
    // Basket lists are staged in a ring of mapped pinned host buffers that the
    // tile-expansion kernel reads directly (no copy node). The ring holds
    // kGroups groups of kGroup buffers; one event, recorded after the launch
    // that uses a group's last buffer, guards the whole group, so a call
    // records an event only every kGroup calls (an event record costs about
    // as much as 3% of a launch on the batched workload). Before a group is
    // refilled the host waits for its event.
    struct Stage {
        void *host = nullptr;
        void *dev = nullptr;
        size_t cap = 0;
    };
    struct StageGroup {
        hipEvent_t done = nullptr;
        bool pending = false;
    };
    static constexpr int kGroup = 4, kGroups = 4, kStages = kGroup * kGroups;
    Stage stage[kStages];
    StageGroup group[kGroups];
    int stage_next = 0;
    Tile *d_tiles = nullptr;
    int64_t tiles_cap = 0;
    unsigned int *d_cursors = nullptr;  // kQueues cursors, kQueueStride apart
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipGraphNode_t node_build = nullptr, node_nav = nullptr;
    int graph_U = 0, graph_grid = 0, graph_cull = -1, graph_mode = -1, graph_ktime = -1;
    // optional timing of the navigator kernel alone: event-record nodes
    // before and after it in the batched graph
    bool ktime = false;
    bool ktime_recorded = false;
    hipEvent_t kt_before = nullptr, kt_after = nullptr;
    std::vector<BasketRec> sorted;   // reused host scratch
    std::vector<BasketRec> joined, sort_tmp;
    std::vector<int> sort_count;
};

namespace {

void destroy_graph(geo_geometry *g) {
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    g->exec = nullptr;
    g->graph = nullptr;
    g->node_build = g->node_nav = nullptr;
    g->graph_U = g->graph_grid = 0;
    g->graph_cull = g->graph_mode = g->graph_ktime = -1;
}

// Volumes of at most this many daughters take all of them in lockstep: a
// basket through the navigator (2^22 tracks, one daughter: 41.7 us, culled
// 43.5; 3: 55.3 and 42.5), a smaller one of fewer than kBasketFew tracks (two
// daughters: 300,000 tracks 5.7 us, culled 6.8, 40,000 3.6 and 4.7; 2^20 16.9 and
// 15.0), the safety (2^20 points, 4 daughters: 13.1 us, culled 13.5).
constexpr int kBasketAll = 1, kBasketAllFew = 2, kSafetyAll = 4;
constexpr int64_t kBasketFew = (int64_t)1 << 19;

// How a call on n tracks of one volume culls.
int tests(const geo_geometry *g, int volume, int64_t n, int task) {
    const VolumeRec &v = g->h_vols[volume];
    if (!g->cull) return kNoTests;
    const int others = (v.exact & task) || (v.moved && task != kSafetyTask) ? kAnyTests : kMatrixTests;
    if (!(v.dense & task)) return others;
    if (task == kLineTasks && n <= kFewLines) return v.moved ? kAnyTests : kMatrixTests;
    return n <= (task == kLineTasks ? kFewExact : kFewPoints) ? kAnyTests : kNoTests;
}
int basket_tests(const geo_geometry *g, int volume, int64_t n) {
    const int nd = g->h_vols[volume].nd;
    return nd <= (n < kBasketFew ? kBasketAllFew : kBasketAll) ? (int)kNoTests : tests(g, volume, n, kLineTasks);
}
int batched_tests(const geo_geometry *g) { return !g->cull ? kNoTests : g->any_tests ? kAnyTests : kMatrixTests; }

const CullBlock *volume_blocks(const geo_geometry *g, int volume) {
    return g->d_cull ? g->d_cull + g->h_vols[volume].first_block : nullptr;
}

int check_device(const geo_geometry *g) {
    int dev = -1;
    GN_HIP(hipGetDevice(&dev));
    if (dev != g->device)
        return fail(GEO_ERR_INVALID_ARG, "geometry lives on device %d but device %d is current", g->device,
                    dev);
    return GEO_OK;
}

}  // namespace

// Entry points keep the C linkage of their declarations in geonav.h.

const char *geo_strerror(int status) {
    if (status != GEO_OK && status == g_last_code && !g_last_msg.empty()) return g_last_msg.c_str();
    switch (status) {
        case GEO_OK: return "success";
        case GEO_ERR_INVALID_ARG: return "invalid argument";
        case GEO_ERR_HIP: return "HIP runtime error";
        case GEO_ERR_NOMEM: return "out of memory";
        default: return "unknown status";
    }
}

int geo_geometry_create(const geo_volume_desc *v, int32_t nvol, geo_geometry **out) {
    if (!out) return fail(GEO_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (nvol <= 0 || !v) return fail(GEO_ERR_INVALID_ARG, "need nvol > 0 volumes");
    std::vector<VolumeRec> vols(nvol);
    std::vector<DaughterRec> dau;
    int nblocks = 0;  // culling blocks
    bool any_tests = false;
    // polycone sections, and which record points at each: volume index
    // (mother) or -1 - daughter index
    std::vector<PconRec> pcons;
    std::vector<int64_t> pcon_owner;
    std::vector<int> vol_kset(nvol, kSetBasic);
    auto kind_set = [](int kind) -> int {
        return kind == kTubs || kind == kCons ? kSetSeg : (kind == kPcon || kind == kPcons ? kSetAll : kSetBasic);
    };
    int max_nd = 0;
    for (int iv = 0; iv < nvol; ++iv) {
        const geo_volume_desc &d = v[iv];
        VolumeRec &r = vols[iv];
        std::memset(&r, 0, sizeof r);
        char what[64];
        snprintf(what, sizeof what, "volume %d mother", iv);
        PconRec pc;
        double mother_r = 0.0;
        int rc = make_shape(d.mother, r.mother, &pc, &mother_r, what);
        if (rc) return rc;
        r.bound_r = mother_r;
        if (r.mother.kind == kPcon || r.mother.kind == kPcons) {
            pcons.push_back(pc);
            pcon_owner.push_back(iv);
        }
        vol_kset[iv] = kind_set(r.mother.kind);
        if (d.ndaughters < 0 || d.ndaughters > GEO_MAX_DAUGHTERS)
            return fail(GEO_ERR_INVALID_ARG, "volume %d: ndaughters %d outside 0..%d", iv, d.ndaughters,
                        GEO_MAX_DAUGHTERS);
        if (d.ndaughters > 0 && (!d.daughters || !d.placements))
            return fail(GEO_ERR_INVALID_ARG, "volume %d: NULL daughter arrays", iv);
        r.nd = d.ndaughters;
        r.first = (int32_t)dau.size();
        max_nd = std::max(max_nd, r.nd);
        for (int k = 0; k < d.ndaughters; ++k) {
            DaughterRec dr;
            std::memset(&dr, 0, sizeof dr);
            snprintf(what, sizeof what, "volume %d daughter %d", iv, k);
            rc = make_shape(d.daughters[k], dr.shape, &pc, &dr.bound_r, what);
            if (rc) return rc;
            // A tube (segment) daughter is stored as the equal-radii cone
            // (segment), the same solid: the batches of queued pairs of the
            // culled navigators then hold one kind fewer, each batch running
            // every kind's code once.
            if (d.daughters[k].kind == GEO_TUBE || d.daughters[k].kind == GEO_TUBS) {
                rc = make_shape(as_cone(d.daughters[k]), dr.shape, &pc, &dr.bound_r, what);
                if (rc) return rc;
            }
            if (dr.shape.kind == kPcon || dr.shape.kind == kPcons) {
                pcons.push_back(pc);
                pcon_owner.push_back(-1 - (int64_t)dau.size());
            }
            vol_kset[iv] = std::max(vol_kset[iv], kind_set(dr.shape.kind));
            dr.cull_r = dr.bound_r * (1.0 + 1e-6) + 1e-6;
            rc = check_rotation(d.placements[k].rot, what);
            if (rc) return rc;
            for (int i = 0; i < 3; ++i)
                if (!std::isfinite(d.placements[k].tr[i]))
                    return fail(GEO_ERR_INVALID_ARG, "%s: non-finite translation", what);
            std::memcpy(dr.rot, d.placements[k].rot, sizeof dr.rot);
            std::memcpy(dr.tr, d.placements[k].tr, sizeof dr.tr);
            dau.push_back(dr);
        }
        // the culling tests' units, and the shift of a track's start: more
        // than any radius that takes part (a larger one always passes)
        const double scale = (double)kCullR / mother_r;
        r.near_s = std::isnormal(scale) ? scale : 0.0;
        double back = 0.0, safe_d = 0.0, safe_r2 = 0.0, safe_q = -1.0;
        for (int k = 0; k < r.nd; ++k) {
            const DaughterRec &dr = dau[(size_t)r.first + k];
            const double rs = dr.cull_r * r.near_s;
            if (!(rs <= (double)kCullMax)) continue;
            back = std::max(back, rs);
            const SafetyBound b = safety_bound(d.daughters[k], dr.shape);
            if (b.plain) {
                safe_d = std::max(safe_d, rs * rs + b.c * r.near_s * r.near_s);
            } else {
                safe_r2 = std::max(safe_r2, rs * rs);
                safe_q = std::max(safe_q, b.q * r.near_s);
            }
        }
        r.near_back = (float)(back * (1.0 + 1e-6) + 0.25);
        // (wider by over twice the largest widening of r^2 in the tests,
        // whatever the offsets: the centres that do not always pass have
        // coordinates of at most kCullMax)
        const double reach = kCullR + r.near_back;
        const double wide = 1.25 * 0x1p-14 * (reach * reach + 3.0 * kCullMax * kCullMax);
        r.safe_d = (float)(safe_d + wide);
        r.safe_r2 = (float)(safe_r2 + wide);
        r.safe_q = (float)(safe_q < 0 ? -1.0 : safe_q * (1 + 1e-6) + 1e-6);
        r.near_r = (float)(back * (1 + 1e-6) + 1e-6);
        r.near_r2 = (float)(back * back + wide);
        choose_culling(r, dau.data() + r.first, d.mother, vol_kset[iv] == kSetBasic);
        any_tests |= r.moved || ((r.exact | r.dense) & kLineTasks);
        r.first_block = nblocks;
        nblocks += (r.nd + kCullBlock - 1) / kCullBlock;
    }
    geo_geometry *g = new (std::nothrow) geo_geometry();
    if (!g) return fail(GEO_ERR_NOMEM, "host allocation failed");
    auto cleanup = [&](int rc) {
        geo_geometry_destroy(g);
        return rc;
    };
    hipError_t e = hipGetDevice(&g->device);
    if (e != hipSuccess) return cleanup(hip_fail(e, "hipGetDevice"));
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, g->device);
    if (e != hipSuccess) return cleanup(hip_fail(e, "hipGetDeviceProperties"));
    g->num_cus = prop.multiProcessorCount;
    g->device_name = prop.gcnArchName;
    g->nvol = nvol;
    g->max_nd = max_nd;
    g->any_tests = any_tests;
    g->h_vols = vols;
    g->vol_kset = vol_kset;
    g->kset = *std::max_element(vol_kset.begin(), vol_kset.end());
    if (hipMalloc(&g->d_vols, sizeof(VolumeRec) * nvol) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of volumes failed"));
    if (!dau.empty() && hipMalloc(&g->d_dau, sizeof(DaughterRec) * dau.size()) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of daughters failed"));
    if (nblocks > 0 && hipMalloc(&g->d_cull, sizeof(CullBlock) * (size_t)nblocks) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of culling blocks failed"));
    if (max_nd > 0 &&
        hipMalloc(&g->d_shift, sizeof(CullBlock) * (size_t)((max_nd + kCullBlock - 1) / kCullBlock)) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of the shifted culling blocks failed"));
    if (max_nd > 0 &&
        hipMalloc(&g->d_partial, sizeof(double) * 3 * (size_t)max_nd * kBackwardMaxBlocks) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of adjoint partials failed"));
    if (hipMalloc(&g->d_cursors, sizeof(unsigned int) * kQueues * kQueueStride) != hipSuccess)
        return cleanup(fail(GEO_ERR_NOMEM, "device allocation of the queue cursors failed"));
    if (!pcons.empty()) {
        if (hipMalloc(&g->d_pcon, sizeof(PconRec) * pcons.size()) != hipSuccess)
            return cleanup(fail(GEO_ERR_NOMEM, "device allocation of polycone sections failed"));
        for (size_t i = 0; i < pcons.size(); ++i) {
            const int64_t o = pcon_owner[i];
            if (o >= 0) vols[o].pcon = g->d_pcon + i;
            else dau[-1 - o].pcon = g->d_pcon + i;
        }
        e = hipMemcpy(g->d_pcon, pcons.data(), sizeof(PconRec) * pcons.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return cleanup(hip_fail(e, "hipMemcpy polycone sections"));
    }
    e = hipMemcpy(g->d_vols, vols.data(), sizeof(VolumeRec) * nvol, hipMemcpyHostToDevice);
    if (e != hipSuccess) return cleanup(hip_fail(e, "hipMemcpy volumes"));
    if (!dau.empty()) {
        e = hipMemcpy(g->d_dau, dau.data(), sizeof(DaughterRec) * dau.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) return cleanup(hip_fail(e, "hipMemcpy daughters"));
        e = launch_cull_blocks(g->d_vols, nvol, nblocks, g->d_dau, g->d_cull, nullptr);
        if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
        if (e != hipSuccess) return cleanup(hip_fail(e, "culling blocks"));
    }
    for (auto &gr : g->group) {
        e = hipEventCreateWithFlags(&gr.done, hipEventDisableTiming);
        if (e != hipSuccess) return cleanup(hip_fail(e, "hipEventCreate"));
    }
    *out = g;
    return GEO_OK;
}

int geo_geometry_destroy(geo_geometry *g) {
    if (!g) return GEO_OK;
    int dev = -1;
    (void)hipGetDevice(&dev);
    if (dev != g->device) (void)hipSetDevice(g->device);
    (void)hipDeviceSynchronize();
    destroy_graph(g);
    if (g->kt_before) (void)hipEventDestroy(g->kt_before);
    if (g->kt_after) (void)hipEventDestroy(g->kt_after);
    for (auto &gr : g->group)
        if (gr.done) (void)hipEventDestroy(gr.done);
    for (auto &st : g->stage)
        if (st.host) (void)hipHostFree(st.host);
    (void)hipFree(g->d_pcon);
    (void)hipFree(g->d_vols);
    (void)hipFree(g->d_dau);
    (void)hipFree(g->d_cull);
    (void)hipFree(g->d_shift);
    (void)hipFree(g->d_partial);
    (void)hipFree(g->d_tiles);
    (void)hipFree(g->d_cursors);
    if (dev >= 0 && dev != g->device) (void)hipSetDevice(dev);
    delete g;
    return GEO_OK;
}

int geo_shape_query(const geo_shape *s, int32_t query, geo_tracks t, void *out, hipStream_t stream) {
    if (!s) return fail(GEO_ERR_INVALID_ARG, "shape is NULL");
    if (query < GEO_CONTAINS || query > GEO_DIST_OUT) return fail(GEO_ERR_INVALID_ARG, "unknown query %d", query);
    ShapeRec rec;
    PconRec pc;
    std::memset(&pc, 0, sizeof pc);
    int rc = make_shape(*s, rec, &pc, nullptr, "shape");
    if (rc) return rc;
    rc = check_tracks(t, query >= GEO_DIST_IN, "tracks");
    if (rc) return rc;
    if (t.n == 0) return GEO_OK;
    rc = check_out(out, query == GEO_CONTAINS ? 1 : 8, "out");
    if (rc) return rc;
    hipError_t e = launch_shape_query(rec, pc, query, to_dev(t), out, stream);
    if (e != hipSuccess) return hip_fail(e, "shape query launch");
    return GEO_OK;
}

int geo_navigate_basket(const geo_geometry *g, int32_t volume, geo_tracks t, const double *offsets,
                        double *step, int32_t *hit, double *hitpt, hipStream_t stream) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (volume < 0 || volume >= g->nvol) return fail(GEO_ERR_INVALID_ARG, "volume %d out of range", volume);
    int rc = check_tracks(t, true, "tracks");
    if (rc) return rc;
    if (t.n == 0) return GEO_OK;
    if ((rc = check_out(step, 8, "step")) || (rc = check_out(hit, 4, "hit")) ||
        (rc = check_opt(hitpt, 8, "hitpt")) || (rc = check_opt(offsets, 8, "offsets")))
        return rc;
    if ((rc = check_device(g))) return rc;
    const int first = g->h_vols[volume].first;
    hipError_t e = launch_nav_basket(g->d_vols + volume, g->d_dau ? g->d_dau + first : nullptr,
                                     volume_blocks(g, volume), to_dev(t),
                                     g->h_vols[volume].nd > 0 ? offsets : nullptr, step, hit, hitpt,
                                     basket_tests(g, volume, t.n),
                                     g->vol_kset[volume], stream);
    if (e != hipSuccess) return hip_fail(e, "navigator launch");
    return GEO_OK;
}

int geo_navigate_backward(const geo_geometry *g, int32_t volume, geo_tracks t, const double *offsets,
                          const double *gstep, const double *ghit, double *g_o, double *g_d, double *g_off,
                          hipStream_t stream) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (volume < 0 || volume >= g->nvol) return fail(GEO_ERR_INVALID_ARG, "volume %d out of range", volume);
    int rc = check_tracks(t, true, "tracks");
    if (rc) return rc;
    if ((rc = check_opt(offsets, 8, "offsets")) || (rc = check_opt(gstep, 8, "gstep")) ||
        (rc = check_opt(ghit, 8, "ghit")) || (rc = check_opt(g_o, 8, "g_o")) ||
        (rc = check_opt(g_d, 8, "g_d")) || (rc = check_opt(g_off, 8, "g_off")))
        return rc;
    const int nd = g->h_vols[volume].nd;
    if (t.n == 0 && !(g_off && nd > 0)) return GEO_OK;
    if ((rc = check_device(g))) return rc;
    const int first = g->h_vols[volume].first;
    hipError_t e = launch_backward(g->d_vols + volume, g->d_dau, g->d_dau ? g->d_dau + first : nullptr,
                                   volume_blocks(g, volume), nd, to_dev(t),
                                   nd > 0 ? offsets : nullptr, gstep, ghit, g_o, g_d, g->d_partial,
                                   nd > 0 ? g_off : nullptr, tests(g, volume, t.n, kLineTasks), g->vol_kset[volume], g->d_shift, stream);
    if (e != hipSuccess) return hip_fail(e, "adjoint launch");
    return GEO_OK;
}

int geo_navigate_backward_noalloc(const geo_geometry *g, int32_t volume, geo_tracks t, const double *offsets,
                                  const double *gstep, const double *ghit, double *g_o, double *g_d,
                                  double *g_off, hipStream_t stream) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (volume < 0 || volume >= g->nvol) return fail(GEO_ERR_INVALID_ARG, "volume %d out of range", volume);
    int rc = check_tracks(t, true, "tracks");
    if (rc) return rc;
    if ((rc = check_opt(offsets, 8, "offsets")) || (rc = check_opt(gstep, 8, "gstep")) ||
        (rc = check_opt(ghit, 8, "ghit")) || (rc = check_opt(g_o, 8, "g_o")) ||
        (rc = check_opt(g_d, 8, "g_d")) || (rc = check_opt(g_off, 8, "g_off")))
        return rc;
    const int nd = g->h_vols[volume].nd;
    if (t.n == 0 && !(g_off && nd > 0)) return GEO_OK;
    if ((rc = check_device(g))) return rc;
    double *part = nullptr;
    if (g_off && nd > 0) {
        const size_t need = (size_t)backward_rows(t.n) * 3 * (size_t)nd;
        if (need > kScratchDoubles)
            return fail(GEO_ERR_INVALID_ARG,
                        "geo_navigate_backward_noalloc: %d daughters over %lld tracks need %zu partial sums, "
                        "the static buffer holds %zu (%d daughters at any track count)",
                        nd, (long long)t.n, need, kScratchDoubles, (int)(kScratchDoubles / (3 * kBackwardMaxBlocks)));
        hipError_t e = scratch_partials(&part);
        if (e != hipSuccess) return hip_fail(e, "static partial-sum buffer");
    }
    const int first = g->h_vols[volume].first;
    hipError_t e = launch_backward(g->d_vols + volume, g->d_dau, g->d_dau ? g->d_dau + first : nullptr,
                                   volume_blocks(g, volume), nd, to_dev(t),
                                   nd > 0 ? offsets : nullptr, gstep, ghit, g_o, g_d, part,
                                   nd > 0 ? g_off : nullptr, tests(g, volume, t.n, kLineTasks), g->vol_kset[volume], nullptr, stream);
    if (e != hipSuccess) return hip_fail(e, "adjoint launch");
    return GEO_OK;
}

namespace {

int point_call_checks(const geo_geometry *g, int32_t volume, const geo_tracks &t, const double *offsets,
                      const void *out, size_t out_align) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (volume < 0 || volume >= g->nvol) return fail(GEO_ERR_INVALID_ARG, "volume %d out of range", volume);
    int rc = check_tracks(t, false, "points");
    if (rc) return rc;
    if (t.n == 0) return GEO_OK;
    if ((rc = check_out(out, out_align, "out")) || (rc = check_opt(offsets, 8, "offsets"))) return rc;
    return check_device(g);
}

}  // namespace

int geo_navigate_safety(const geo_geometry *g, int32_t volume, geo_tracks t, const double *offsets,
                        double *safety, hipStream_t stream) {
    int rc = point_call_checks(g, volume, t, offsets, safety, 8);
    if (rc || t.n == 0) return rc;
    const int first = g->h_vols[volume].first;
    hipError_t e = launch_nav_safety(g->d_vols + volume, g->d_dau ? g->d_dau + first : nullptr,
                                     volume_blocks(g, volume), g->h_vols[volume].nd, to_dev(t),
                                     g->h_vols[volume].nd > 0 ? offsets : nullptr, safety,
                                     g->h_vols[volume].nd > kSafetyAll ? tests(g, volume, t.n, kSafetyTask) : (int)kNoTests,
                                     g->vol_kset[volume], stream);
    if (e != hipSuccess) return hip_fail(e, "safety launch");
    return GEO_OK;
}

int geo_locate(const geo_geometry *g, int32_t volume, geo_tracks t, const double *offsets, int32_t *where,
               hipStream_t stream) {
    int rc = point_call_checks(g, volume, t, offsets, where, 4);
    if (rc || t.n == 0) return rc;
    const int first = g->h_vols[volume].first;
    hipError_t e = launch_nav_locate(g->d_vols + volume, g->d_dau ? g->d_dau + first : nullptr,
                                     volume_blocks(g, volume), g->h_vols[volume].rounds != 0, to_dev(t),
                                     g->h_vols[volume].nd > 0 ? offsets : nullptr, where, tests(g, volume, t.n, kLocateTask),
                                     g->vol_kset[volume], stream);
    if (e != hipSuccess) return hip_fail(e, "locate launch");
    return GEO_OK;
}

// ------------------------------------------------------------- batched
namespace {

// Make the next staging buffer free and large enough for nb baskets, and the
// device tile buffer large enough for ntiles tiles.
int ensure_capacity(geo_geometry *g, int nb, int64_t ntiles, hipStream_t stream) {
    const size_t need = sizeof(BasketRec) * (size_t)nb + sizeof(int64_t) * (size_t)(nb + 1);
    if (g->stage_next % geo_geometry::kGroup == 0) {  // refilling a group: its last use is done
        geo_geometry::StageGroup &gr = g->group[g->stage_next / geo_geometry::kGroup];
        if (gr.pending) GN_HIP(hipEventSynchronize(gr.done));
        gr.pending = false;
    }
    geo_geometry::Stage &st = g->stage[g->stage_next];
    if (need > st.cap) {
        if (st.host) (void)hipHostFree(st.host);
        st.host = st.dev = nullptr;
        st.cap = 0;
        const size_t cap = std::max(need, (size_t)(1 << 16));
        if (hipHostMalloc(&st.host, cap, hipHostMallocMapped) != hipSuccess)
            return fail(GEO_ERR_NOMEM, "pinned staging allocation failed");
        GN_HIP(hipHostGetDevicePointer(&st.dev, st.host, 0));
        st.cap = cap;
    }
    if (ntiles > g->tiles_cap) {
        // the tile buffer may still be in use by a previous launch
        GN_HIP(hipStreamSynchronize(stream));
        GN_HIP(hipDeviceSynchronize());
        destroy_graph(g);
        (void)hipFree(g->d_tiles);
        g->d_tiles = nullptr;
        const int64_t cap = std::max<int64_t>(ntiles + ntiles / 4, 4096);
        if (hipMalloc(&g->d_tiles, sizeof(Tile) * (size_t)cap) != hipSuccess)
            return fail(GEO_ERR_NOMEM, "device tile allocation failed");
        g->tiles_cap = cap;
    }
    return GEO_OK;
}

// After a launch that read the current staging buffer: close its group with
// an event when it was the group's last buffer, and move on.
int advance_stage(geo_geometry *g, hipStream_t stream) {
    if (g->stage_next % geo_geometry::kGroup == geo_geometry::kGroup - 1) {
        geo_geometry::StageGroup &gr = g->group[g->stage_next / geo_geometry::kGroup];
        GN_HIP(hipEventRecord(gr.done, stream));
        gr.pending = true;
    }
    g->stage_next = (g->stage_next + 1) % geo_geometry::kStages;
    return GEO_OK;
}

int launch_batched(geo_geometry *g, const geo_basket *b, int32_t nb, const geo_tracks &all, double *step,
                   int32_t *hit, hipStream_t stream, unsigned long long *census = nullptr) {
    const int U = g->tracks_per_lane;
    const int tile_n = 64 * U;
    // Baskets of one volume that follow one another in the list and whose
    // tracks follow one another in the pool are joined, so that their tiles
    // fill whole wavefronts across the basket boundaries (results are per
    // track, so the outputs are the same): once in the order given (which
    // takes a list of many small consecutive baskets down to a few before
    // the sort), and again in the sorted order.
    auto join = [](const BasketRec &r, std::vector<BasketRec> &out) {
        BasketRec *last = out.empty() ? nullptr : &out.back();
        if (last && last->volume == r.volume && last->offset + last->n == r.offset)
            last->n += r.n;
        else
            out.push_back(r);
    };
    std::vector<BasketRec> &in = g->joined;
    in.clear();
    in.reserve((size_t)nb);
    for (int i = 0; i < nb; ++i)
        if (b[i].n > 0) join(BasketRec{b[i].volume, 0, b[i].offset, b[i].n}, in);
    if (in.empty()) return GEO_OK;
    // cost-sorted basket list (per-track cost ~ daughters + mother): a
    // stable counting sort on the daughter count, descending (O(nb), which
    // matters for tens of thousands of small baskets)
    std::vector<BasketRec> &s = g->sorted;
    std::vector<int> &cnt = g->sort_count;
    cnt.assign((size_t)g->max_nd + 2, 0);
    for (const BasketRec &r : in) ++cnt[g->max_nd - g->h_vols[r.volume].nd + 1];
    for (size_t k = 1; k < cnt.size(); ++k) cnt[k] += cnt[k - 1];
    std::vector<BasketRec> &tmp = g->sort_tmp;
    tmp.resize(in.size());
    for (const BasketRec &r : in) tmp[cnt[g->max_nd - g->h_vols[r.volume].nd]++] = r;
    s.clear();
    s.reserve(tmp.size());
    for (const BasketRec &r : tmp) join(r, s);
    const int ns = (int)s.size();
    int64_t ntiles = 0;
    for (const BasketRec &r : s) ntiles += (r.n + tile_n - 1) / tile_n;
    if (ntiles > 0x7fffffff) return fail(GEO_ERR_INVALID_ARG, "too many tiles");
    int rc = ensure_capacity(g, ns, ntiles, stream);
    if (rc) return rc;
    // stage the sorted baskets and their tile starts in the free buffer
    geo_geometry::Stage &st = g->stage[g->stage_next];
    BasketRec *hb = static_cast<BasketRec *>(st.host);
    int64_t *hs = reinterpret_cast<int64_t *>(hb + ns);
    int64_t acc = 0;
    for (int i = 0; i < ns; ++i) {
        hb[i] = s[i];
        hs[i] = acc;
        acc += (s[i].n + tile_n - 1) / tile_n;
    }
    hs[ns] = acc;

    BuildTilesArgs ba;
    ba.baskets = static_cast<const BasketRec *>(st.dev);
    ba.tile_start = reinterpret_cast<const int64_t *>(static_cast<const BasketRec *>(st.dev) + ns);
    ba.nb = ns;
    ba.tile_n = tile_n;
    ba.tiles = g->d_tiles;
    ba.cursors = g->d_cursors;
    PersistentArgs pa;
    pa.vols = g->d_vols;
    pa.dau = g->d_dau;
    pa.cul = g->d_cull;
    pa.tiles = g->d_tiles;
    pa.ntiles = (int32_t)ntiles;
    pa.cursors = g->d_cursors;
    pa.t = to_dev(all);
    pa.step = step;
    pa.hit = hit;
    pa.census = census;

    const bool persistent = g->waves_per_simd > 0;
    const int grid = batched_grid(g->waves_per_simd, g->num_cus, ntiles);
    void *bargs[] = {&ba};
    void *pargs[] = {&pa.vols, &pa.dau, &pa.cul, &pa.tiles, &pa.ntiles, &pa.cursors, &pa.t, &pa.step,
                     &pa.hit, &pa.census};
    if (census || !g->use_graph) {
        // two launches on the stream (the instrumented run always: its
        // census kernel is not the graph's)
        if (census) GN_HIP(hipMemsetAsync(census, 0, kCensusSlots * sizeof(unsigned long long), stream));
        GN_HIP(hipLaunchKernel(build_tiles_kernel(), dim3(kBuildTilesBlocks), dim3(kBlock), bargs, 0, stream));
        const bool kt = g->ktime && !census;
        if (kt) GN_HIP(hipEventRecord(g->kt_before, stream));
        GN_HIP(hipLaunchKernel(batched_kernel(U, batched_tests(g), persistent, census != nullptr, g->kset), dim3(grid),
                               dim3(kBlock), pargs, 0, stream));
        if (kt) {
            GN_HIP(hipEventRecord(g->kt_after, stream));
            g->ktime_recorded = true;
        }
        return advance_stage(g, stream);
    }
    hipKernelNodeParams kb = {};
    kb.func = const_cast<void *>(build_tiles_kernel());
    kb.gridDim = dim3(kBuildTilesBlocks);
    kb.blockDim = dim3(kBlock);
    kb.kernelParams = bargs;
    hipKernelNodeParams kn = {};
    kn.func = const_cast<void *>(batched_kernel(U, batched_tests(g), persistent, false, g->kset));
    kn.gridDim = dim3(grid);
    kn.blockDim = dim3(kBlock);
    kn.kernelParams = pargs;
    const int mode = persistent ? 1 : 0;
    bool rebuild = !g->exec || g->graph_U != U || g->graph_cull != (int)g->cull || g->graph_mode != mode ||
                   g->graph_ktime != (int)g->ktime;
    if (!rebuild) {
        // same kernels: update arguments (and the grid, which the hardware-
        // scheduled form sizes by tile count); rebuild if the update is refused
        if (hipGraphExecKernelNodeSetParams(g->exec, g->node_build, &kb) != hipSuccess ||
            hipGraphExecKernelNodeSetParams(g->exec, g->node_nav, &kn) != hipSuccess) {
            (void)hipGetLastError();
            rebuild = true;
        }
    }
    if (rebuild) {
        destroy_graph(g);
        GN_HIP(hipGraphCreate(&g->graph, 0));
        GN_HIP(hipGraphAddKernelNode(&g->node_build, g->graph, nullptr, 0, &kb));
        if (g->ktime) {
            hipGraphNode_t before = nullptr, after = nullptr;
            GN_HIP(hipGraphAddEventRecordNode(&before, g->graph, &g->node_build, 1, g->kt_before));
            GN_HIP(hipGraphAddKernelNode(&g->node_nav, g->graph, &before, 1, &kn));
            GN_HIP(hipGraphAddEventRecordNode(&after, g->graph, &g->node_nav, 1, g->kt_after));
        } else {
            GN_HIP(hipGraphAddKernelNode(&g->node_nav, g->graph, &g->node_build, 1, &kn));
        }
        GN_HIP(hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0));
        g->graph_U = U;
        g->graph_cull = (int)g->cull;
        g->graph_mode = mode;
        g->graph_ktime = (int)g->ktime;
    }
    g->graph_grid = grid;
    GN_HIP(hipGraphLaunch(g->exec, stream));
    g->ktime_recorded = g->ktime;
    return advance_stage(g, stream);
}

int validate_batched(const geo_geometry *g, const geo_basket *b, int32_t nb, const geo_tracks &all,
                     double *step, int32_t *hit, bool check_outputs) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (nb < 0) return fail(GEO_ERR_INVALID_ARG, "nb < 0");
    if (nb > 0 && !b) return fail(GEO_ERR_INVALID_ARG, "baskets is NULL");
    int rc = check_tracks(all, true, "track pool");
    if (rc) return rc;
    int64_t total = 0;
    for (int i = 0; i < nb; ++i) {
        if (b[i].volume < 0 || b[i].volume >= g->nvol)
            return fail(GEO_ERR_INVALID_ARG, "basket %d: volume %d out of range", i, b[i].volume);
        if (b[i].n < 0 || b[i].offset < 0 || b[i].offset > all.n || b[i].n > all.n - b[i].offset)
            return fail(GEO_ERR_INVALID_ARG, "basket %d: [%lld, +%lld) outside the pool of %lld", i,
                        (long long)b[i].offset, (long long)b[i].n, (long long)all.n);
        total += b[i].n;
    }
    if (total > 0 && check_outputs) {
        if ((rc = check_out(step, 8, "step")) || (rc = check_out(hit, 4, "hit"))) return rc;
    }
    return GEO_OK;
}

}  // namespace

int geo_navigate_batched(geo_geometry *g, const geo_basket *b, int32_t nb, geo_tracks all, double *step,
                         int32_t *hit, hipStream_t stream) {
    int rc = validate_batched(g, b, nb, all, step, hit, true);
    if (rc) return rc;
    if (nb == 0 || all.n == 0) return GEO_OK;
    if ((rc = check_device(g))) return rc;
    return launch_batched(g, b, nb, all, step, hit, stream);
}

int geo_navigate_batched_census(geo_geometry *g, const geo_basket *b, int32_t nb, geo_tracks all,
                                double *step, int32_t *hit, uint64_t counts[GEO_CENSUS_SLOTS], hipStream_t stream) {
    if (!counts) return fail(GEO_ERR_INVALID_ARG, "counts is NULL");
    for (int i = 0; i < GEO_CENSUS_SLOTS; ++i) counts[i] = 0;
    int rc = validate_batched(g, b, nb, all, step, hit, true);
    if (rc) return rc;
    if (nb == 0 || all.n == 0) return GEO_OK;
    if ((rc = check_device(g))) return rc;
    unsigned long long *d = nullptr;
    if (hipMalloc(&d, kCensusSlots * sizeof(unsigned long long)) != hipSuccess)
        return fail(GEO_ERR_NOMEM, "census counter allocation failed");
    rc = launch_batched(g, b, nb, all, step, hit, stream, d);
    if (rc == GEO_OK) {
        unsigned long long h[kCensusSlots];
        hipError_t e = hipMemcpyAsync(h, d, sizeof h, hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) rc = hip_fail(e, "census readback");
        else
            for (int i = 0; i < kCensusSlots; ++i) counts[i] = h[i];
    }
    (void)hipFree(d);
    return rc;
}

int geo_get_launch_config(const geo_geometry *g, int32_t *tracks_per_lane, int32_t *waves_per_simd) {
    if (!g || !tracks_per_lane || !waves_per_simd) return fail(GEO_ERR_INVALID_ARG, "NULL argument");
    *tracks_per_lane = g->tracks_per_lane;
    *waves_per_simd = g->waves_per_simd;
    return GEO_OK;
}

int geo_set_launch_config(geo_geometry *g, int32_t tracks_per_lane, int32_t waves_per_simd) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (!(tracks_per_lane == 1 || tracks_per_lane == 2 || tracks_per_lane == 4 || tracks_per_lane == 8))
        return fail(GEO_ERR_INVALID_ARG, "tracks_per_lane must be 1, 2, 4 or 8");
    if (waves_per_simd < 0 || waves_per_simd > 8)
        return fail(GEO_ERR_INVALID_ARG, "waves_per_simd must be 0 (one wavefront per tile) or 1..8");
    g->tracks_per_lane = tracks_per_lane;
    g->waves_per_simd = waves_per_simd;
    return GEO_OK;
}

int geo_get_batched_graph(const geo_geometry *g, int32_t *use_graph) {
    if (!g || !use_graph) return fail(GEO_ERR_INVALID_ARG, "NULL argument");
    *use_graph = g->use_graph ? 1 : 0;
    return GEO_OK;
}

int geo_set_batched_graph(geo_geometry *g, int32_t use_graph) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    if (use_graph != 0 && use_graph != 1) return fail(GEO_ERR_INVALID_ARG, "use_graph must be 0 or 1");
    g->use_graph = use_graph != 0;
    return GEO_OK;
}

int geo_set_culling(geo_geometry *g, int32_t enable) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    g->cull = enable != 0;
    return GEO_OK;
}

int geo_get_culling(const geo_geometry *g, int32_t *enabled) {
    if (!g || !enabled) return fail(GEO_ERR_INVALID_ARG, "NULL argument");
    *enabled = g->cull ? 1 : 0;
    return GEO_OK;
}

int geo_set_kernel_timing(geo_geometry *g, int32_t enable) {
    if (!g) return fail(GEO_ERR_INVALID_ARG, "geometry is NULL");
    int rc = check_device(g);
    if (rc) return rc;
    if (enable && !g->kt_before) {
        GN_HIP(hipEventCreate(&g->kt_before));
        GN_HIP(hipEventCreate(&g->kt_after));
    }
    g->ktime = enable != 0;
    g->ktime_recorded = false;
    return GEO_OK;
}

int geo_batched_kernel_ms(geo_geometry *g, float *ms) {
    if (!g || !ms) return fail(GEO_ERR_INVALID_ARG, "NULL argument");
    if (!g->ktime || !g->ktime_recorded)
        return fail(GEO_ERR_INVALID_ARG, "no batched call with kernel timing enabled since it was set");
    int rc = check_device(g);
    if (rc) return rc;
    GN_HIP(hipEventSynchronize(g->kt_after));
    GN_HIP(hipEventElapsedTime(ms, g->kt_before, g->kt_after));
    return GEO_OK;
}

// ------------------------------------------------------------- autotuner
namespace {

std::string tune_key(const geo_geometry *g, const geo_basket *b, int nb) {
    int64_t total = 0;
    double work = 0;
    for (int i = 0; i < nb; ++i) {
        total += b[i].n;
        work += (double)b[i].n * (g->h_vols[b[i].volume].nd + 1);
    }
    // bucket by powers of two of the basket count, track count and mean cost
    auto lg = [](double v) { return v > 1 ? (int)std::floor(std::log2(v)) : 0; };
    std::ostringstream os;
    os << g->device_name << "/cu" << g->num_cus << "/nb" << lg(nb) << "/n" << lg((double)total) << "/c"
       << lg(total > 0 ? work / total : 1);
    return os.str();
}

// The cache is a flat JSON object:
// {"key": [tracks_per_lane, waves_per_simd, use_graph], ...} (an entry of
// two numbers, from before the launch mode was tuned, reads as use_graph 0).
struct TuneEntry {
    int u, w, graph;
};
std::vector<std::pair<std::string, TuneEntry>> read_cache(const char *path) {
    std::vector<std::pair<std::string, TuneEntry>> out;
    std::ifstream f(path);
    if (!f) return out;
    std::stringstream ss;
    ss << f.rdbuf();
    const std::string s = ss.str();
    size_t pos = 0;
    while (true) {
        size_t q0 = s.find('"', pos);
        if (q0 == std::string::npos) break;
        size_t q1 = s.find('"', q0 + 1);
        if (q1 == std::string::npos) break;
        size_t lb = s.find('[', q1);
        size_t rb = s.find(']', lb == std::string::npos ? q1 : lb);
        if (lb == std::string::npos || rb == std::string::npos) break;
        int u = 0, w = 0, gr = 0;
        const std::string item = s.substr(lb + 1, rb - lb - 1);
        const int got = std::sscanf(item.c_str(), " %d , %d , %d", &u, &w, &gr);
        if (got >= 2) out.push_back({s.substr(q0 + 1, q1 - q0 - 1), TuneEntry{u, w, got == 3 ? gr : 0}});
        pos = rb + 1;
    }
    return out;
}

void write_cache(const char *path, const std::vector<std::pair<std::string, TuneEntry>> &ent) {
    std::string tmp = std::string(path) + ".tmp";
    std::ofstream f(tmp);
    if (!f) return;
    f << "{\n";
    for (size_t i = 0; i < ent.size(); ++i)
        f << "  \"" << ent[i].first << "\": [" << ent[i].second.u << ", " << ent[i].second.w << ", "
          << ent[i].second.graph << "]" << (i + 1 < ent.size() ? ",\n" : "\n");
    f << "}\n";
    f.close();
    std::rename(tmp.c_str(), path);
}

}  // namespace

int geo_autotune(geo_geometry *g, const geo_basket *b, int32_t nb, geo_tracks all, hipStream_t stream) {
    int rc = validate_batched(g, b, nb, all, nullptr, nullptr, false);
    if (rc) return rc;
    if (nb == 0 || all.n == 0) return GEO_OK;
    if ((rc = check_device(g))) return rc;
    const char *path = std::getenv("GEONAV_AUTOTUNE_CACHE");
    const std::string key = tune_key(g, b, nb);
    auto cache = path ? read_cache(path) : decltype(read_cache("")){};
    for (auto &e : cache)
        if (e.first == key && geo_set_launch_config(g, e.second.u, e.second.w) == GEO_OK &&
            geo_set_batched_graph(g, e.second.graph) == GEO_OK)
            return GEO_OK;

    double *step = nullptr;
    int32_t *hit = nullptr;
    if (hipMalloc(&step, sizeof(double) * (size_t)all.n) != hipSuccess ||
        hipMalloc(&hit, sizeof(int32_t) * (size_t)all.n) != hipSuccess) {
        (void)hipFree(step);
        return fail(GEO_ERR_NOMEM, "autotune scratch allocation failed");
    }
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    const int Us[] = {1, 2, 4, 8};
    const int Ws[] = {0, 2, 3, 4, 6, 8};
    constexpr int kNU = 4, kNW = 6;
    int bestU = g->tracks_per_lane, bestW = g->waves_per_simd;
    float tbest[kNU][kNW];
    for (auto &row : tbest)
        for (float &v : row) v = 1e30f;
    rc = GEO_OK;
    // bring the clocks up first (the GPU needs tens of milliseconds of load
    // to reach its full clock; timing from idle would favour the shapes timed
    // last), then time every shape in two passes and keep each shape's best
    {
        (void)hipEventRecord(e0, stream);
        float warm = 0;
        for (int k = 0; k < 1024 && rc == GEO_OK && warm < 50.0f; ++k) {
            rc = launch_batched(g, b, nb, all, step, hit, stream);
            if (k % 16 == 15 && rc == GEO_OK) {
                (void)hipEventRecord(e1, stream);
                if (hipEventSynchronize(e1) != hipSuccess) rc = fail(GEO_ERR_HIP, "autotune warm-up failed");
                (void)hipEventElapsedTime(&warm, e0, e1);
            }
        }
    }
    for (int pass = 0; pass < 2 && rc == GEO_OK; ++pass) {
        for (int iu = 0; iu < kNU && rc == GEO_OK; ++iu) {
            for (int iw = 0; iw < kNW && rc == GEO_OK; ++iw) {
                g->tracks_per_lane = Us[iu];
                g->waves_per_simd = Ws[iw];
                // steady state, as in a transport loop: the mean of kBurst
                // back-to-back calls after a warm-up call (which also builds
                // the graph for this shape)
                constexpr int kBurst = 6;
                rc = launch_batched(g, b, nb, all, step, hit, stream);
                (void)hipEventRecord(e0, stream);
                for (int k = 0; k < kBurst && rc == GEO_OK; ++k)
                    rc = launch_batched(g, b, nb, all, step, hit, stream);
                (void)hipEventRecord(e1, stream);
                if (rc) break;
                if (hipEventSynchronize(e1) != hipSuccess) {
                    rc = fail(GEO_ERR_HIP, "autotune timing failed");
                    break;
                }
                float ms = 0;
                (void)hipEventElapsedTime(&ms, e0, e1);
                tbest[iu][iw] = std::min(tbest[iu][iw], ms / kBurst);
            }
        }
    }
    float best = 1e30f;
    for (int iu = 0; iu < kNU; ++iu)
        for (int iw = 0; iw < kNW; ++iw)
            if (tbest[iu][iw] < best) {
                best = tbest[iu][iw];
                bestU = Us[iu];
                bestW = Ws[iw];
            }
    // then, at the best shape, the two kernels as a graph replay against two
    // launches (two passes, as above)
    const bool mode0 = g->use_graph;
    float tmode[2] = {1e30f, 1e30f};
    g->tracks_per_lane = bestU;
    g->waves_per_simd = bestW;
    for (int pass = 0; pass < 2 && rc == GEO_OK; ++pass) {
        for (int m = 0; m < 2 && rc == GEO_OK; ++m) {
            g->use_graph = m == 1;
            constexpr int kBurst = 6;
            rc = launch_batched(g, b, nb, all, step, hit, stream);
            (void)hipEventRecord(e0, stream);
            for (int k = 0; k < kBurst && rc == GEO_OK; ++k) rc = launch_batched(g, b, nb, all, step, hit, stream);
            (void)hipEventRecord(e1, stream);
            if (rc) break;
            if (hipEventSynchronize(e1) != hipSuccess) {
                rc = fail(GEO_ERR_HIP, "autotune timing failed");
                break;
            }
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            tmode[m] = std::min(tmode[m], ms / kBurst);
        }
    }
    const bool bestGraph = rc == GEO_OK ? tmode[1] < tmode[0] : mode0;
    g->use_graph = bestGraph;
    (void)hipStreamSynchronize(stream);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    (void)hipFree(step);
    (void)hipFree(hit);
    g->tracks_per_lane = bestU;
    g->waves_per_simd = bestW;
    if (rc) return rc;
    if (path) {
        bool found = false;
        const TuneEntry te{bestU, bestW, bestGraph ? 1 : 0};
        for (auto &e : cache)
            if (e.first == key) {
                e.second = te;
                found = true;
            }
        if (!found) cache.push_back({key, te});
        write_cache(path, cache);
    }
    return GEO_OK;
}

