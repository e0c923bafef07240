// Kernels of libgeonav for gfx950 and their launchers.
//
//  k_shape_query     one query of one shape over a basket (section 3.1);
//                    streaming, one lane per track, HBM-bound (the polycone
//                    and the cone segment's Safety are ALU-bound).
//  k_shape_dist      the same for the distances of large polycone baskets: the
//                    tracks that need its sections evaluated are queued.
//  k_nav_basket      the simple navigator (section 3, Fig. 1b) over one
//                    basket: culling tests on the matrix cores, the (track,
//                    daughter) pairs that pass queued in LDS and evaluated one
//                    per lane; near the copy rate over large baskets (with
//                    culling off, every lane walks every daughter).
//  k_nav_safety      the navigator's isotropic safety (section 3) per point;
//  k_nav_locate      the daughter holding each point (localization);
//  k_build_tiles     expands a host-sorted basket list into tiles of at most
//                    64 x U tracks of one volume (largest cost first);
//  k_nav_tiles       the per-track navigator over all tiles of many baskets
//                    of many volumes in one launch, one wavefront per tile;
//  k_nav_persistent  the same with a machine-sized grid whose wavefronts
//                    pull tiles from per-XCD queues;
//  k_cull_blocks     the daughters' operands of the culling tests (matrix cores
//                    and FP64), for a geometry or moved by one adjoint
//                    call's offsets;
//  k_nav_backward    adjoint of the navigator (recompute + implicit-function
//                    gradient of the surface that set the step) with
//                    per-workgroup partial sums of the offset gradient;
//  k_reduce_partials fixed-order reduction of those partials.
#include <mutex>

#include "geonav_internal.hpp"

// The build compiles this file's sections, GEONAV_PART 1 to 5, side by side.
#ifndef GEONAV_PART
#define GEONAV_PART 0
#endif
#define GN_PART(p) (GEONAV_PART == 0 || GEONAV_PART == (p))

namespace gn {

// Runs STMT with the compile-time constant KS set to the runtime kind set.
#define GN_KSET(kset, STMT)                                 \
    do {                                                    \
        if ((kset) == kSetBasic) {                          \
            constexpr int KS = kSetBasic;                   \
            STMT;                                           \
        } else if ((kset) == kSetSeg) {                     \
            constexpr int KS = kSetSeg;                     \
            STMT;                                           \
        } else {                                            \
            constexpr int KS = kSetAll;                     \
            STMT;                                           \
        }                                                   \
    } while (0)

#if GN_PART(1)
// ------------------------------------------------------------ shape queries
// A polycone's sections come by value with the arguments (`pc`, unused for
// the other kinds).
template <int KIND, int Q>
__global__ __launch_bounds__(kBlock) void k_shape_query(ShapeRec s, PconRec pc, TracksDev t,
                                                        void *out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= t.n) return;
    const double x = t.x[i], y = t.y[i], z = t.z[i];
    if (Q == 0) {
        static_cast<uint8_t *>(out)[i] = shape_contains<KIND>(s, &pc, x, y, z) ? 1 : 0;
        return;
    }
    double r;
    if (Q == 1) {
        r = shape_safety<KIND>(s, &pc, x, y, z);
    } else {
        const double ux = t.ux[i], uy = t.uy[i], uz = t.uz[i];
        int sid;
        if (Q == 2) r = shape_dist_in<KIND>(s, &pc, x, y, z, ux, uy, uz, sid);
        else r = shape_dist_out<KIND>(s, &pc, x, y, z, ux, uy, uz, sid);
    }
    static_cast<double *>(out)[i] = r;
}

// The polycone's distances, two nappe quadratics per section, are bound by
// VALU issue (4 sections: 45 FP64 instructions per nappe), and are wanted
// only for points inside (DistIn), or for points outside whose line passes
// through the bounding sphere (DistOut); the rest are 0, or misses. Each
// wavefront takes kDistRounds rounds of 64 tracks, sets what is known of each
// and queues the others with their tracks in LDS, as the navigators do, so
// that the evaluations run on full wavefronts; the results leave together,
// a whole line at a time. Shape suite (half the points inside), one lane per
// track and this: 2^24 tracks DistIn 280 and 222 us, DistOut 284 and 185 (5.1
// TB/s, the rate of a large copy), 2^21 DistIn 37 and 36, DistOut 37 and 24.
// 8 rounds: DistIn 218, DistOut 182, but two wavefronts fewer per SIMD where
// every point is inside. Rounds that nearly all need evaluating skip the
// queue (2^23 tracks, all inside: 145 and 147 us; 155 through the queue).
constexpr int kDistRounds = 4;
// lanes of a round from which on it is evaluated where it is
constexpr int kDistFull = 56;
struct DistScratch {
    double out[kDistRounds * 64];
    unsigned int at[64];  // queued tracks: place in `out`, and the track
    double x[64], y[64], z[64], ux[64], uy[64], uz[64];
};
template <int KIND, int Q>
__global__ __launch_bounds__(kBlock) void k_shape_dist(ShapeRec s, PconRec pc, TracksDev t, double *__restrict__ out) {
    constexpr bool SEG = KIND == kPcons;
    __shared__ DistScratch scr[kBlock / 64];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * (64 * kDistRounds);
    if (base >= t.n) return;
    const int count = t.n - base < 64 * kDistRounds ? (int)(t.n - base) : 64 * kDistRounds;
    DistScratch &S = scr[wave];
    const TileTracks tt = tile_tracks(t, base);
    auto load = [&](int j) -> Track {  // (a lane past the end: the last track)
        const unsigned int ju = (unsigned int)(j < count ? j : count - 1);
        return Track{at32(tt.x, ju), at32(tt.y, ju), at32(tt.z, ju), at32(tt.ux, ju), at32(tt.uy, ju), at32(tt.uz, ju)};
    };
    int qn = 0;  // queued tracks (uniform)
    auto distance = [&](const Track &p) -> double {
        int sid;
        if (Q == 2) return pcon_dist_in<SEG, true>(s, pc, p.x, p.y, p.z, p.ux, p.uy, p.uz, sid);
        return pcon_dist_out<SEG, true>(s, pc, p.x, p.y, p.z, p.ux, p.uy, p.uz, sid);
    };
    auto batch = [&]() {
        if (lane < qn)
            S.out[S.at[lane]] =
                distance(Track{S.x[lane], S.y[lane], S.z[lane], S.ux[lane], S.uy[lane], S.uz[lane]});
        qn = 0;
    };
    Track next = load(lane);
#pragma unroll 1
    for (int u = 0; u * 64 < count; ++u) {
        const int j = u * 64 + lane;
        const Track p = next;
        if ((u + 1) * 64 < count) next = load(j + 64);
        const bool inside = pcon_contains(pc, p.x, p.y, p.z) && (!SEG || wedge_in(s, p.x, p.y));
        bool want = inside;
        double known = 0.0;
        if (Q == 3) {
            // the half-line's squared distance from the origin, times |d|^2:
            // a miss by more than its rounding (or not a number: wanted)
            const double dd = fma(p.uz, p.uz, fma(p.uy, p.uy, p.ux * p.ux));
            const double pp = fma(p.z, p.z, fma(p.y, p.y, p.x * p.x));
            const double b = fmin(fma(p.z, p.uz, fma(p.y, p.uy, p.x * p.ux)), 0.0);
            const bool misses = fma(-b, b, pp * dd) > fma(64.0 * 2.220446049250313e-16, pp, pc.far2) * dd;
            known = inside ? 0.0 : kBig;
            want = !inside && !misses;
        }
        S.out[j] = known;
        bool todo = want && j < count;
        if (__popcll(__builtin_amdgcn_ballot_w64(todo)) >= kDistFull) {
            if (todo) S.out[j] = distance(p);
            continue;
        }
        for (;;) {
            const unsigned long long more = __builtin_amdgcn_ballot_w64(todo);
            if (more == 0ull) break;
            const int at = qn + lanes_below(more);
            if (todo && at < 64) {
                S.at[at] = (unsigned int)j;
                S.x[at] = p.x;
                S.y[at] = p.y;
                S.z[at] = p.z;
                S.ux[at] = p.ux;
                S.uy[at] = p.uy;
                S.uz[at] = p.uz;
                todo = false;
            }
            const int n = qn + __popcll(more);
            qn = n < 64 ? n : 64;
            if (qn == 64) batch();
        }
    }
    batch();
#pragma unroll 1
    for (int u = 0; u * 64 < count; ++u) {
        const int j = u * 64 + lane;
        if (j < count) at32(out + base, (unsigned int)j) = S.out[j];
    }
}

// Baskets of at least kDistWide tracks, which fill the chip several times
// over at kDistRounds rounds per wavefront; smaller ones one lane per track
// (2^20 tracks: DistIn 21.5 us either way, DistOut 21.9 and 16.1).
constexpr int64_t kDistWide[2] = {(int64_t)1 << 21, (int64_t)1 << 20};  // DistIn, DistOut
template <int KIND>
static bool launch_shape_pcon(const ShapeRec &s, const PconRec &pc, int query, const TracksDev &t, void *out,
                              hipStream_t st) {
    if (query < 2 || t.n < kDistWide[query - 2]) return false;
    const int64_t tile = (int64_t)kBlock * kDistRounds;
    const dim3 grid((unsigned)((t.n + tile - 1) / tile)), block(kBlock);
    double *o = static_cast<double *>(out);
    if (query == 2) hipLaunchKernelGGL((k_shape_dist<KIND, 2>), grid, block, 0, st, s, pc, t, o);
    else hipLaunchKernelGGL((k_shape_dist<KIND, 3>), grid, block, 0, st, s, pc, t, o);
    return true;
}

template <int KIND>
static hipError_t launch_shape_kind(const ShapeRec &s, const PconRec &pc, int query,
                                    const TracksDev &t, void *out, hipStream_t st) {
    const dim3 grid((unsigned)((t.n + kBlock - 1) / kBlock)), block(kBlock);
    switch (query) {
        case 0: hipLaunchKernelGGL((k_shape_query<KIND, 0>), grid, block, 0, st, s, pc, t, out); break;
        case 1: hipLaunchKernelGGL((k_shape_query<KIND, 1>), grid, block, 0, st, s, pc, t, out); break;
        case 2: hipLaunchKernelGGL((k_shape_query<KIND, 2>), grid, block, 0, st, s, pc, t, out); break;
        default: hipLaunchKernelGGL((k_shape_query<KIND, 3>), grid, block, 0, st, s, pc, t, out); break;
    }
    return hipGetLastError();
}

hipError_t launch_shape_query(const ShapeRec &s, const PconRec &pc, int query, const TracksDev &t,
                              void *out, hipStream_t st) {
    if (t.n == 0) return hipSuccess;
    switch (s.kind) {
        case kBox: return launch_shape_kind<kBox>(s, pc, query, t, out, st);
        case kTube: return launch_shape_kind<kTube>(s, pc, query, t, out, st);
        case kCone: return launch_shape_kind<kCone>(s, pc, query, t, out, st);
        case kTubs: return launch_shape_kind<kTubs>(s, pc, query, t, out, st);
        case kCons: return launch_shape_kind<kCons>(s, pc, query, t, out, st);
        case kPcon:
            if (launch_shape_pcon<kPcon>(s, pc, query, t, out, st)) return hipGetLastError();
            return launch_shape_kind<kPcon>(s, pc, query, t, out, st);
        default:
            if (launch_shape_pcon<kPcons>(s, pc, query, t, out, st)) return hipGetLastError();
            return launch_shape_kind<kPcons>(s, pc, query, t, out, st);
    }
}
#endif

#if GN_PART(2)
// ---------------------------------------------------------- basket navigator
// With culling, one wavefront takes U rounds of 64 tracks (compacted
// evaluation; more tracks per wavefront fill more lanes of each batch of
// queued pairs). What bounds it is the memory's latency as much as VALU issue
// (0.85 of the lanes' time; 4.8 TB/s of the 60 B per track on the toy
// detector, 1 GiB copies reach 5.0), so wavefronts in flight count: all are
// compiled for 5 per SIMD (75-96 VGPRs; of every kind, with 4 rounds, 12 to 36 B
// per lane spilled, 52 in the kernels of every form), which takes that nothing is
// kept live through a full queue's batch, nor an address formed ahead of it (118
// VGPRs, 4 per SIMD, before). 2^22 tracks, three sets of buffers in turn (us),
// FP64 culling tests / these tests at 4 / at 5: toy detector 84.6 / 62 / 59.4,
// every kind 112 / 87 / 83, 8 daughters 60.3 / 58.8 / 56.4, 64 131 / 89 / 85;
// 300007 tracks of every kind, one round, 19.5 / 20.5 / 15.8.
template <bool HAS_OFFS, bool HITPT, int TESTS, int KSET, int U = 1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(TESTS ? 5 : 1))) void k_nav_basket(const VolumeRec *__restrict__ vol,
                                                       const DaughterRec *__restrict__ dau,
                                                       const CullBlock *__restrict__ cul,
                                                       TracksDev t, const double *__restrict__ offs,
                                                       double *__restrict__ step,
                                                       int32_t *__restrict__ hit,
                                                       double *__restrict__ hitpt) {
    if constexpr (TESTS != kNoTests && KSET != kSetBasic) {
        // volumes of more kinds: the workgroup's wavefronts pool their last
        // flush (a wavefront past the basket's end takes part with no tracks)
        __shared__ NavScratch<U> scr[kBlock / 64];
        __shared__ unsigned short list[TESTS == kAnyTests ? kBlock / 64 : 1][TESTS == kAnyTests ? kListCap : 1];
        __shared__ PoolInfo<kBlock / 64> pool;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (uniform)
        const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * 64 * U;
        const int64_t left = t.n - base;
        const int count = left <= 0 ? 0 : (left < 64 * U ? (int)left : 64 * U);
        nav_compact_pooled<U, kBlock / 64, HAS_OFFS, HITPT, KSET, TESTS>(*vol, dau, cul, 0, offs, t, base, count, scr,
                                                                  list[TESTS == kAnyTests ? wave : 0], pool, true, wave, (int)(threadIdx.x & 63),
                                                                  step, hit, hitpt);
        return;
    }
    if constexpr (TESTS != kNoTests) {
        // (box, tube and cone only: pooling gains nothing measurable)
        __shared__ NavScratch<U> scr[kBlock / 64];
        __shared__ unsigned short list[TESTS == kAnyTests ? kBlock / 64 : 1][TESTS == kAnyTests ? kListCap : 1];
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (uniform)
        const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * 64 * U;
        if (base >= t.n) return;
        const int count = t.n - base < 64 * U ? (int)(t.n - base) : 64 * U;
        nav_compact<U, HAS_OFFS, HITPT, false, KSET, TESTS>(*vol, dau, cul, offs, t, base, count, scr[wave],
                                                            list[TESTS == kAnyTests ? wave : 0],
                                                            (vol->exact & kLineTasks) != 0, (int)(threadIdx.x & 63),
                                                            step, hit, hitpt);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= t.n) return;
    const double x = t.x[i], y = t.y[i], z = t.z[i];
    const double ux = t.ux[i], uy = t.uy[i], uz = t.uz[i];
    double best;
    int h, sid;
    nav_track<HAS_OFFS, false, false, KSET>(*vol, dau, offs, x, y, z, ux, uy, uz, best, h, sid);
    step[i] = best;
    hit[i] = h;
    if (HITPT) {
        const int64_t n = t.n;
        hitpt[i] = fma(best, ux, x);
        hitpt[n + i] = fma(best, uy, y);
        hitpt[2 * n + i] = fma(best, uz, z);
    }
}

template <int TESTS, int KSET, int U = 1>
static void launch_basket_variant(dim3 grid, const VolumeRec *vol, const DaughterRec *dau,
                                  const CullBlock *cul, const TracksDev &t, const double *offs, double *step, int32_t *hit,
                                  double *hitpt, hipStream_t st) {
    const dim3 block(kBlock);
    if (offs) {
        if (hitpt) hipLaunchKernelGGL((k_nav_basket<true, true, TESTS, KSET, U>), grid, block, 0, st, vol, dau, cul, t, offs, step, hit, hitpt);
        else hipLaunchKernelGGL((k_nav_basket<true, false, TESTS, KSET, U>), grid, block, 0, st, vol, dau, cul, t, offs, step, hit, hitpt);
    } else {
        if (hitpt) hipLaunchKernelGGL((k_nav_basket<false, true, TESTS, KSET, U>), grid, block, 0, st, vol, dau, cul, t, offs, step, hit, hitpt);
        else hipLaunchKernelGGL((k_nav_basket<false, false, TESTS, KSET, U>), grid, block, 0, st, vol, dau, cul, t, offs, step, hit, hitpt);
    }
}

// Baskets of at least kBasketWide tracks run 4 rounds per wavefront (still
// about 4096 wavefronts, several per SIMD); smaller baskets one round. (8
// rounds: toy detector 55.9 against 52.2 us at 2^22 tracks, mixed 95 against
// 77: about 60 pairs per tile, often a second batch of a few.)
constexpr int64_t kBasketWide = (int64_t)1 << 20;

hipError_t launch_nav_basket(const VolumeRec *vol, const DaughterRec *dau, const CullBlock *cul,
                             const TracksDev &t, const double *offs, double *step, int32_t *hit,
                             double *hitpt, int tests, int kset, hipStream_t st) {
    if (t.n == 0) return hipSuccess;
    const bool wide = tests != kNoTests && t.n >= kBasketWide;
    const int64_t per = (int64_t)kBlock * (wide ? 4 : 1);
    const dim3 grid((unsigned)((t.n + per - 1) / per));
#define GN_BASKET(TESTS, U) \
    GN_KSET(kset, (launch_basket_variant<TESTS, KS, U>(grid, vol, dau, cul, t, offs, step, hit, hitpt, st)))
    if (tests == kNoTests) GN_BASKET(kNoTests, 1);
    else if (tests == kAnyTests && wide) GN_BASKET(kAnyTests, 4);
    else if (tests == kAnyTests) GN_BASKET(kAnyTests, 1);
    else if (wide) GN_BASKET(kMatrixTests, 4);
    else GN_BASKET(kMatrixTests, 1);
#undef GN_BASKET
    return hipGetLastError();
}
#endif

#if GN_PART(1)
// -------------------------------------------------- safety and locate
// The safety takes one round of 64 points per wavefront (four rounds with a
// queue run when it is full: 76.1 against 75.6 us at 2^22 points of the toy
// detector before the records were in LDS, 23.7 against 22.0 at 10^6); volumes
// with segments or polycones pool their pairs over the workgroup. With TABLE
// the workgroup copies the daughters' records into its LDS first. 2^22 points,
// three sets in turn, with FP64 culling tests 110 us, now 60.5; of every kind
// 364, now 181.
template <bool HAS_OFFS, int TESTS, int KSET, bool TABLE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_nav_safety(const VolumeRec *__restrict__ vol,
                                                       const DaughterRec *__restrict__ dau,
                                                       const CullBlock *__restrict__ cul, TracksDev t,
                                                       const double *__restrict__ offs,
                                                       double *__restrict__ out) {
    if constexpr (TESTS == kAnyTests) {
        __shared__ ExactPoints scr[kBlock / 64];
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (uniform)
        const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * 64;
        if (base >= t.n) return;
        const int count = t.n - base < 64 ? (int)(t.n - base) : 64;
        points_exact<true, HAS_OFFS, KSET>(*vol, dau, cul, offs, t, base, count, scr[wave], (int)(threadIdx.x & 63),
                                           out);
        return;
    }
    if constexpr (TESTS == kMatrixTests) {
        constexpr bool POOL = KSET != kSetBasic;
        __shared__ PointScratch scr[kBlock / 64];
        __shared__ PointPool<kBlock / 64> pool;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (uniform)
        const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * 64;
        if (!POOL && !TABLE && base >= t.n) return;
        const int64_t left = t.n - base;
        const int count = left <= 0 ? 0 : (left < 64 ? (int)left : 64);
        const int lane = (int)(threadIdx.x & 63);
        if constexpr (TABLE) {
            extern __shared__ uint4v recs[];
            lds_records<KSET>(dau, vol->nd, recs);
            safety_compact<HAS_OFFS, KSET, POOL, kBlock / 64>(*vol, dau, LdsRecords<KSET>{recs}, cul, offs, t, base,
                                                              count, scr, &pool, wave, lane, out);
        } else {
            safety_compact<HAS_OFFS, KSET, POOL, kBlock / 64>(*vol, dau, GlobalRecords{dau}, cul, offs, t, base,
                                                              count, scr, &pool, wave, lane, out);
        }
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= t.n) return;
    out[i] = nav_safety<HAS_OFFS, KSET>(*vol, dau, offs, t.x[i], t.y[i], t.z[i]);
}

template <bool HAS_OFFS, int TESTS, int KSET, int U = 1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_nav_locate(const VolumeRec *__restrict__ vol,
                                                       const DaughterRec *__restrict__ dau,
                                                       const CullBlock *__restrict__ cul, TracksDev t,
                                                       const double *__restrict__ offs,
                                                       int32_t *__restrict__ out) {
    if constexpr (TESTS != kNoTests) {
        __shared__ LocateScratch<U> scr[kBlock / 64];
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // (uniform)
        const int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * (64 * U);
        if (base >= t.n) return;
        const int count = t.n - base < 64 * U ? (int)(t.n - base) : 64 * U;
        const int lane = (int)(threadIdx.x & 63);
        if constexpr (TESTS == kAnyTests) {
            static_assert(U == 1, "one round of 64 points in FP64");
            __shared__ ExactPoints exact[kBlock / 64];
            if (vol->exact & kLocateTask) {
                points_exact<false, HAS_OFFS, KSET>(*vol, dau, cul, offs, t, base, count, exact[wave], lane, out);
                return;
            }
        }
        locate_compact<HAS_OFFS, KSET, U, TESTS == kAnyTests>(*vol, dau, cul, offs, t, base, count, scr[wave], lane, out);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= t.n) return;
    out[i] = nav_locate<HAS_OFFS, KSET>(*vol, dau, offs, t.x[i], t.y[i], t.z[i]);
}

template <int TESTS, int KSET, bool TABLE = false>
static void launch_safety_variant(dim3 grid, const VolumeRec *vol, const DaughterRec *dau,
                                  const CullBlock *cul, int nd, const TracksDev &t, const double *offs,
                                  double *out, hipStream_t st) {
    const size_t lds = TABLE ? (size_t)nd * LdsRecords<KSET>::Q * 16 : 0;
    if (offs)
        hipLaunchKernelGGL((k_nav_safety<true, TESTS, KSET, TABLE>), grid, dim3(kBlock), lds, st, vol, dau, cul, t, offs, out);
    else
        hipLaunchKernelGGL((k_nav_safety<false, TESTS, KSET, TABLE>), grid, dim3(kBlock), lds, st, vol, dau, cul, t, offs, out);
}

template <int TESTS, int KSET, int U = 1>
static void launch_locate_variant(const VolumeRec *vol, const DaughterRec *dau,
                                  const CullBlock *cul, const TracksDev &t, const double *offs,
                                  int32_t *out, hipStream_t st) {
    const dim3 grid((unsigned)((t.n + kBlock * U - 1) / (kBlock * U)));
    if (offs) hipLaunchKernelGGL((k_nav_locate<true, TESTS, KSET, U>), grid, dim3(kBlock), 0, st, vol, dau, cul, t, offs, out);
    else hipLaunchKernelGGL((k_nav_locate<false, TESTS, KSET, U>), grid, dim3(kBlock), 0, st, vol, dau, cul, t, offs, out);
}

// Volumes of up to kSafetyTable daughters (20 to 24 KB of records in LDS, four
// workgroups on a CU) have them copied: faster at every count measured, 8 to
// 64 (above, and at LdsRecords), and no slower at 10,000 points (7.6 us). Larger
// volumes read the geometry's table.
constexpr int kSafetyTable = 64;

hipError_t launch_nav_safety(const VolumeRec *vol, const DaughterRec *dau, const CullBlock *cul, int nd,
                             const TracksDev &t, const double *offs, double *out, int tests,
                             int kset, hipStream_t st) {
    if (t.n == 0) return hipSuccess;
    const dim3 grid((unsigned)((t.n + kBlock - 1) / kBlock));
#define GN_SAFETY(TESTS, TABLE) \
    GN_KSET(kset, (launch_safety_variant<TESTS, KS, TABLE>(grid, vol, dau, cul, nd, t, offs, out, st)))
    if (tests == kNoTests) GN_SAFETY(kNoTests, false);
    else if (tests == kAnyTests) GN_SAFETY(kAnyTests, false);
    else if (nd <= kSafetyTable) GN_SAFETY(kMatrixTests, true);
    else GN_SAFETY(kMatrixTests, false);
#undef GN_SAFETY
    return hipGetLastError();
}

// Localizations of at least kLocateWide points in volumes of enough daughters, or whose
// points are in enough of their spheres (VolumeRec.rounds), run kLocateRounds rounds of
// 64 per wavefront, still about 3000 wavefronts; the others one round. (Toy detector,
// three sets in turn, one round / four: 2^22 points 35.4 / 29.1 us, 10^6 10.1 / 9.4; every
// kind 2^20 13.9 / 12.4. 37 us and 17.8 with FP64 culling tests. 8 daughters, one set, 2^20
// 6.0 / 7.0, 16 6.0 / 7.0; six sets, 2^21 15.8 / 15.3 and 15.5 / 14.9. 8 large daughters
// that hold 6 % of the points, 2^20 9.8 / 8.4, every kind 16.3 / 12.3.)
constexpr int64_t kLocateWide = (int64_t)3 << 18;
constexpr int kLocateRounds = 4;

hipError_t launch_nav_locate(const VolumeRec *vol, const DaughterRec *dau, const CullBlock *cul,
                             bool rounds, const TracksDev &t, const double *offs, int32_t *out, int tests,
                             int kset, hipStream_t st) {
    if (t.n == 0) return hipSuccess;
    const bool wide = t.n >= kLocateWide && rounds;
#define GN_LOCATE(TESTS, U) GN_KSET(kset, (launch_locate_variant<TESTS, KS, U>(vol, dau, cul, t, offs, out, st)))
    if (tests == kNoTests) GN_LOCATE(kNoTests, 1);
    else if (tests == kAnyTests) GN_LOCATE(kAnyTests, 1);
    else if (wide) GN_LOCATE(kMatrixTests, kLocateRounds);
    else GN_LOCATE(kMatrixTests, 1);
#undef GN_LOCATE
    return hipGetLastError();
}
#endif

#if GN_PART(3) || GN_PART(5)
// ------------------------------------------------------------------ batched
// A tile holds at most 64 * U tracks of one volume: U rounds of one track
// per lane, so the volume and its daughters are uniform over the wavefront.
// Tiles come in order of decreasing per-track cost (the host sorts the
// baskets by daughter count; k_build_tiles expands them in that order).
template <int U, int TESTS, bool COUNT, int KSET>
__device__ __forceinline__ void run_tile(const Tile &tl, const VolumeRec *__restrict__ vols,
                                         const DaughterRec *__restrict__ dau_all,
                                         const CullBlock *__restrict__ cul_all, const TracksDev &t,
                                         double *__restrict__ step, int32_t *__restrict__ hit,
                                         unsigned long long *census, int lane,
                                         NavScratch<U> *scr, unsigned short *list) {
    const VolumeRec &v = vols[tl.volume];
    const DaughterRec *dau = dau_all + v.first;
    if constexpr (TESTS != kNoTests) {
        const bool dense = TESTS == kAnyTests && (v.dense & kLineTasks);
        if (!dense || tl.count <= kFewExact) {
            const bool exact = dense ? tl.count > kFewLines : (v.exact & kLineTasks) != 0;
            nav_compact<U, false, false, COUNT, KSET, TESTS>(v, dau, cul_all + v.first_block, nullptr, t, tl.offset,
                                                             tl.count, *scr, list, exact, lane, step, hit, nullptr, census);
            return;
        }
    }
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
        const int j = u * 64 + lane;
        if (j < tl.count) {
            const int64_t i = tl.offset + j;
            const double x = t.x[i], y = t.y[i], z = t.z[i];
            const double ux = t.ux[i], uy = t.uy[i], uz = t.uz[i];
            double best;
            int h, sid;
            nav_track<false, false, COUNT, KSET>(v, dau, nullptr, x, y, z, ux, uy, uz,
                                                       best, h, sid, census);
            step[i] = best;
            hit[i] = h;
        }
    }
}

// Persistent form: a grid sized to the machine; tiles are dealt round-robin
// into kQueues queues (tile i to queue i mod kQueues, in order), each with its
// own cursor on its own 256-byte line, so the atomics that hand out tiles
// spread over kQueues addresses instead of contending on one. A wavefront
// drains the queue of its workgroup's XCD slot (blockIdx mod kQueues) first,
// then the others in turn; it exits once every queue's cursor has passed the
// queue's length, so every wavefront terminates. (Every kind, 4 rounds, 4 wavefronts
// per SIMD: compiled for 5, which spills here, 178 us, for 4 150.)
template <int U, int TESTS, bool COUNT, int KSET>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(!TESTS ? 1 : U == 1 ? 5 : 4))) void k_nav_persistent(const VolumeRec *__restrict__ vols,
                                                           const DaughterRec *__restrict__ dau_all,
                                                           const CullBlock *__restrict__ cul_all,
                                                           const Tile *__restrict__ tiles,
                                                           int32_t ntiles, unsigned int *cursors,
                                                           TracksDev t, double *__restrict__ step,
                                                           int32_t *__restrict__ hit,
                                                           unsigned long long *census) {
    const int lane = threadIdx.x & 63;
    __shared__ NavScratch<U> scr[TESTS ? kBlock / 64 : 1];
    __shared__ unsigned short list[TESTS == kAnyTests ? kBlock / 64 : 1][TESTS == kAnyTests ? kListCap : 1];
    NavScratch<U> *my = &scr[TESTS ? (threadIdx.x >> 6) : 0];
    const int wave = (int)(threadIdx.x >> 6);
    const int home = (int)(blockIdx.x % kQueues);
    for (int qq = 0; qq < kQueues; ++qq) {
        const int q = (home + qq) % kQueues;
        const unsigned int count = ntiles > q ? (unsigned int)((ntiles - q + kQueues - 1) / kQueues) : 0u;
        for (;;) {
            unsigned int id = 0;
            if (lane == 0) id = atomicAdd(&cursors[q * kQueueStride], 1u);
            id = (unsigned int)__builtin_amdgcn_readfirstlane((int)id);
            if (id >= count) break;
            run_tile<U, TESTS, COUNT, KSET>(tiles[q + kQueues * (int64_t)id], vols, dau_all, cul_all, t,
                                           step, hit, census, lane, my, list[TESTS == kAnyTests ? wave : 0]);
        }
    }
}

// Hardware-scheduled form: one wavefront per tile, workgroups dispatched in
// tile order (same parameters as the persistent form; `cursors` unused).
// Registers as in the basket navigator, 5 wavefronts per SIMD, but for tiles of 2
// rounds, which spill there (4.4 M tracks in 512 baskets: 99 at 5, 79 us at 4; every
// kind 163 and 115). (Of 4 rounds, three pools in turn, with the tile expansion: 96
// us with FP64 culling tests, 79.8 at 4 wavefronts per SIMD, 76.9 at 5.)
template <int U, int TESTS, bool COUNT, int KSET>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(!TESTS ? 1 : U == 2 ? 4 : 5))) void k_nav_tiles(const VolumeRec *__restrict__ vols,
                                                      const DaughterRec *__restrict__ dau_all,
                                                      const CullBlock *__restrict__ cul_all,
                                                      const Tile *__restrict__ tiles, int32_t ntiles,
                                                      unsigned int *cursors, TracksDev t,
                                                      double *__restrict__ step,
                                                      int32_t *__restrict__ hit,
                                                      unsigned long long *census) {
    (void)cursors;
    __shared__ NavScratch<U> scr[TESTS ? kBlock / 64 : 1];
    __shared__ unsigned short list[TESTS == kAnyTests ? kBlock / 64 : 1][TESTS == kAnyTests ? kListCap : 1];
    const int wave = (int)(threadIdx.x >> 6);
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kBlock / 64) + wave));
    if constexpr (TESTS != kNoTests && !COUNT && KSET != kSetBasic) {
        // volumes of more kinds: the workgroup's wavefronts pool their last
        // flush when their four tiles belong to one volume (work of about
        // the same length: tiles of one volume come together in the cost
        // order); a wavefront past the last tile takes part with no tracks
        __shared__ PoolInfo<kBlock / 64> pool;
        const int w0 = (int)blockIdx.x * (kBlock / 64);
        bool shared = w0 + kBlock / 64 <= ntiles;
        for (int q = 1; shared && q < kBlock / 64; ++q) shared = tiles[w0 + q].volume == tiles[w0].volume;
        Tile tl;
        tl.volume = 0;
        tl.count = 0;
        tl.offset = 0;
        if (w < ntiles) tl = tiles[w];
        const VolumeRec &v = vols[tl.volume];
        if (TESTS == kAnyTests && (v.dense & kLineTasks)) {  // (all four of a shared workgroup)
            if (w < ntiles)
                run_tile<U, TESTS, false, KSET>(tl, vols, dau_all, cul_all, t, step, hit, nullptr,
                                                (int)(threadIdx.x & 63), &scr[wave], list[TESTS == kAnyTests ? wave : 0]);
            return;
        }
        nav_compact_pooled<U, kBlock / 64, false, false, KSET, TESTS>(v, dau_all, cul_all + v.first_block, v.first, nullptr, t, tl.offset,
                                                               tl.count, scr, list[TESTS == kAnyTests ? wave : 0], pool, shared, wave,
                                                               (int)(threadIdx.x & 63), step, hit, nullptr);
        return;
    }
    if (w >= ntiles) return;
    run_tile<U, TESTS, COUNT, KSET>(tiles[w], vols, dau_all, cul_all, t, step, hit, census,
                                   (int)(threadIdx.x & 63), &scr[TESTS ? wave : 0], list[TESTS == kAnyTests ? wave : 0]);
}

template <bool PERSISTENT, int U, int TESTS, bool COUNT, int KSET>
static const void *pick_mode() {
    if constexpr (PERSISTENT) return reinterpret_cast<const void *>(&k_nav_persistent<U, TESTS, COUNT, KSET>);
    else return reinterpret_cast<const void *>(&k_nav_tiles<U, TESTS, COUNT, KSET>);
}

template <bool PERSISTENT, int TESTS, bool COUNT, int KSET>
static const void *pick_u(int U) {
    switch (U) {
        case 1: return pick_mode<PERSISTENT, 1, TESTS, COUNT, KSET>();
        case 2: return pick_mode<PERSISTENT, 2, TESTS, COUNT, KSET>();
        case 4: return pick_mode<PERSISTENT, 4, TESTS, COUNT, KSET>();
        default: return pick_mode<PERSISTENT, 8, TESTS, COUNT, KSET>();
    }
}

// The census variants (instrumentation, not timed) exist for the full kind
// set only.
template <bool PERSISTENT>
static const void *pick_kernel(int tracks_per_lane, int tests, bool count, int kset) {
    const void *k = nullptr;
    if (count) {
        k = tests ? pick_u<PERSISTENT, kAnyTests, true, kSetAll>(tracks_per_lane)
                  : pick_u<PERSISTENT, kNoTests, true, kSetAll>(tracks_per_lane);
    } else if (tests == kAnyTests) {
        GN_KSET(kset, (k = pick_u<PERSISTENT, kAnyTests, false, KS>(tracks_per_lane)));
    } else if (tests) {
        GN_KSET(kset, (k = pick_u<PERSISTENT, kMatrixTests, false, KS>(tracks_per_lane)));
    } else {
        GN_KSET(kset, (k = pick_u<PERSISTENT, kNoTests, false, KS>(tracks_per_lane)));
    }
    return k;
}

const void *persistent_kernel(int tracks_per_lane, int tests, bool count, int kset);
#endif

#if GN_PART(5)
const void *persistent_kernel(int tracks_per_lane, int tests, bool count, int kset) {
    return pick_kernel<true>(tracks_per_lane, tests, count, kset);
}
#endif

#if GN_PART(3)
// Expands the (cost-sorted) basket list into tiles of at most tile_n tracks:
// basket b owns tiles [tile_start[b], tile_start[b + 1]). The baskets are
// split into one contiguous run per wavefront (ceil(nb / waves) baskets, so
// a few hundred baskets spread over as many wavefronts); within its run a
// wavefront reads up to 64 basket records at once, lane j taking record j
// (mapped host memory: one round trip per 64), then writes each basket's
// tiles 64 at a time. Also resets the persistent kernel's queue cursors.
__global__ __launch_bounds__(kBlock) void k_build_tiles(BuildTilesArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    const int nwaves = gridDim.x * (kBlock / 64);
    if (blockIdx.x == 0 && threadIdx.x < kQueues) a.cursors[threadIdx.x * kQueueStride] = 0u;
    const int run = (a.nb + nwaves - 1) / nwaves;
    const int b0 = wave * run;
    const int b1 = b0 + run < a.nb ? b0 + run : a.nb;
    for (int base = b0; base < b1; base += 64) {
        const int b = base + lane;
        int vol = 0;
        int64_t off = 0, n = 0, first = 0, last = 0;
        if (b < b1) {
            const BasketRec bk = a.baskets[b];
            vol = bk.volume;
            off = bk.offset;
            n = bk.n;
            first = a.tile_start[b];
            last = a.tile_start[b + 1];
        }
        const int m = b1 - base < 64 ? b1 - base : 64;
        for (int i = 0; i < m; ++i) {
            const int v_i = __shfl(vol, i);
            const int64_t off_i = __shfl(off, i), n_i = __shfl(n, i);
            const int64_t f_i = __shfl(first, i), l_i = __shfl(last, i);
            for (int64_t c = lane; c < l_i - f_i; c += 64) {
                const int64_t o = c * a.tile_n;
                const int64_t left = n_i - o;
                Tile tl;
                tl.volume = v_i;
                tl.count = (int32_t)(left < a.tile_n ? left : a.tile_n);
                tl.offset = off_i + o;
                a.tiles[f_i + c] = tl;
            }
        }
    }
}

const void *batched_kernel(int tracks_per_lane, int tests, bool persistent, bool count, int kset) {
    return persistent ? persistent_kernel(tracks_per_lane, tests, count, kset)
                      : pick_kernel<false>(tracks_per_lane, tests, count, kset);
}

const void *build_tiles_kernel() { return reinterpret_cast<const void *>(&k_build_tiles); }

int batched_grid(int waves_per_simd, int num_cus, int64_t ntiles) {
    // persistent: 4 SIMDs per CU and kBlock / 64 = 4 wavefronts per workgroup,
    // so num_cus * waves_per_simd workgroups give waves_per_simd per SIMD;
    // hardware-scheduled: one wavefront per tile
    if (waves_per_simd > 0) return num_cus * waves_per_simd;
    return (int)((ntiles + kBlock / 64 - 1) / (kBlock / 64));
}
#endif

#if GN_PART(4)
// ------------------------------------------------------------------ adjoint
// Culling blocks from the daughter records, one wavefront each. HAS_OFFS false:
// block blockIdx.x of the geometry's table, which is of the last volume whose
// first block is not past it (the blocks run through the volumes in order; one
// grid dimension, whose limit no geometry reaches, and no workgroup without
// work where the volumes' counts differ). HAS_OFFS true: one volume's (vols),
// moved by this call's daughter offsets, into a buffer of its own (for the
// adjoint's forward). The tests' centre T + offset is rounded once more than
// the T of the evaluation, far inside the culling radius's enlargement of 1e-6
// relative + 1e-6.
template <bool HAS_OFFS>
__global__ __launch_bounds__(64) void k_cull_blocks(const VolumeRec *__restrict__ vols, int nvol,
                                                    const DaughterRec *__restrict__ dau_all,
                                                    const double *__restrict__ offs, CullBlock *__restrict__ out) {
    const int block = (int)blockIdx.x, lane = (int)threadIdx.x;
    int lo = 0;
    if (!HAS_OFFS) {
        for (int hi = nvol; hi - lo > 1;) {
            const int mid = lo + (hi - lo) / 2;
            if (vols[mid].first_block <= block) lo = mid;
            else hi = mid;
        }
    }
    const VolumeRec &v = vols[lo];
    const int k0 = (block - (HAS_OFFS ? 0 : v.first_block)) * kCullBlock;
    *reinterpret_cast<uint4v *>(out[block].a[lane]) = cull_operand<HAS_OFFS>(v, dau_all + v.first, offs, k0, lane);
    *reinterpret_cast<uint4v *>(out[block].near[lane]) =
        cull_operand<HAS_OFFS, true>(v, dau_all + v.first, offs, k0, lane);
    if (lane < kCullBlock) exact_row<HAS_OFFS>(v, dau_all + v.first, offs, k0 + lane, out[block].exact[lane]);
}

hipError_t launch_cull_blocks(const VolumeRec *vols, int nvol, int nblocks, const DaughterRec *dau, CullBlock *out,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_cull_blocks<false>, dim3(nblocks), dim3(64), 0, st, vols, nvol, dau, nullptr, out);
    return hipGetLastError();
}

// For each track: recompute the forward step keeping the surface that set it,
// take that surface's normal n (mother frame) at the hit point and, by the
// implicit-function theorem on the surface equation,
//   ds/dp = -n / (n.d),  ds/dd = s ds/dp,  ds/d delta_hit = n / (n.d).
// With phi = gstep s + ghit . (p + s d) and c = gstep + ghit . d:
//   g_p = ghit + c ds/dp,  g_d = s ghit + c ds/dd,  g_delta_hit += c ds/d delta.
// The offset gradient of the workgroup's tracks is summed per daughter in a
// fixed lane order into the workgroup's row of `partial`, accumulated over
// the workgroup's passes in LDS when lds_acc (3 nd doubles; else in the row
// itself) and written once. With TABLE the forward's culling operands are
// read from `cul`: the volume's, or with offsets those k_cull_blocks moved.
//
// Row b of the partial sums is that of the passes (of 256 tracks) b, b + rows,
// b + 2 rows, ..., added in that order, whatever the tests and U: the sums' bits do
// not depend on them. A workgroup takes U passes at a time: each wavefront
// navigates its 64 tracks of all of them in one go, so that a batch of queued pairs
// holds U times as many, then the passes are differentiated one by one. They are U
// >> log_each rows' first 1 << log_each passes, or one row's next U (log_each 2).
template <bool HAS_OFFS, int TESTS, int KSET, bool TABLE, int U>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(TESTS ? 4 : 1))) void k_nav_backward(
    const VolumeRec *__restrict__ vol, const DaughterRec *__restrict__ dau,
    const CullBlock *__restrict__ cul, TracksDev t, const double *__restrict__ offs,
    const double *__restrict__ gstep,
    const double *__restrict__ ghit, double *__restrict__ g_o, double *__restrict__ g_d,
    double *__restrict__ partial, bool lds_acc, int rows, int log_each) {
    __shared__ double s_g[3][kBlock];
    __shared__ NavScratch<U> scr[TESTS ? kBlock / 64 : 1];
    __shared__ unsigned short list[TESTS == kAnyTests ? kBlock / 64 : 1][TESTS == kAnyTests ? kListCap : 1];
    // [3 nd] doubles of the row's accumulator when lds_acc, then 4 nd + nd + 1
    // ints (see below)
    extern __shared__ double s_dyn[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nd = vol->nd;
    const int nj = 3 * nd;
    int *s_bins = reinterpret_cast<int *>(s_dyn + (lds_acc ? nj : 0));
    const int64_t n = t.n;
    const int npass = (int)((n + kBlock - 1) / kBlock);  // (n < 2^39)
    // `u`: the pass's place among those navigated together
    auto differentiate = [&](int pass, int u, double *acc_row) {
        const int64_t base = (int64_t)pass * kBlock;
        const int64_t i = base + tid;
        int h = -2;
        double gdx = 0.0, gdy = 0.0, gdz = 0.0;
        if constexpr (TESTS != kNoTests) {
            // the forward steps and hits of the next U passes by the
            // compacted navigator
            const int64_t wbase = base + wave * 64;
            if (u == 0 && wbase < n) {
                // (a row's passes are `rows` passes apart)
                const Rounds rounds = log_each == 0   ? Rounds{kBlock, 2 * kBlock}
                                      : log_each == 1 ? Rounds{rows * kBlock, kBlock}
                                                      : Rounds{rows * kBlock, 2 * rows * kBlock};
                const int64_t most = (U == 1 ? 0 : rounds.at(U - 1)) + 64;
                const int cnt = (int)(n - wbase < most ? n - wbase : most);
                nav_core<U, HAS_OFFS, false, KSET, TESTS, true, true, TABLE, U == 1>(
                    *vol, dau, cul, offs, t, wbase, cnt, scr[wave], list[TESTS == kAnyTests ? wave : 0],
                    (vol->exact & kLineTasks) != 0, lane, nullptr, rounds);
            }
        }
        if (i < n) {
            const double x = t.x[i], y = t.y[i], z = t.z[i];
            const double ux = t.ux[i], uy = t.uy[i], uz = t.uz[i];
            double best;
            int sid;
            if constexpr (TESTS != kNoTests) {
                // the step, the winner and the surface that set its step, as
                // the compacted navigator left them
                best = key_step(lds_load(&scr[wave].key[u * 64 + lane]));
                const int v = lds_load(&scr[wave].hit[u * 64 + lane]);
                h = hit_index(v);
                sid = hit_surface(v);
            } else {
                nav_track<HAS_OFFS, true, false, KSET>(*vol, dau, offs, x, y, z, ux, uy, uz, best,
                                                       h, sid);
            }
            const bool finite = best < kBig;
            const double s = finite ? best : 0.0;
            const double hx = fma(s, ux, x), hy = fma(s, uy, y), hz = fma(s, uz, z);
            double nx, ny, nz;
            if (h < 0) {
                surface_normal(vol->mother, vol->pcon, sid, hx, hy, hz, nx, ny, nz);
            } else {
                const DaughterRec &D = dau[h];
                double wx = hx - D.tr[0], wy = hy - D.tr[1], wz = hz - D.tr[2];
                if (HAS_OFFS) {
                    wx -= offs[3 * h + 0];
                    wy -= offs[3 * h + 1];
                    wz -= offs[3 * h + 2];
                }
                const double *R = D.rot;
                const double lx = fma(R[6], wz, fma(R[3], wy, R[0] * wx));
                const double ly = fma(R[7], wz, fma(R[4], wy, R[1] * wx));
                const double lz = fma(R[8], wz, fma(R[5], wy, R[2] * wx));
                double mx, my, mz;
                surface_normal(D.shape, D.pcon, sid, lx, ly, lz, mx, my, mz);
                // back to the mother frame: n = R m
                nx = fma(R[2], mz, fma(R[1], my, R[0] * mx));
                ny = fma(R[5], mz, fma(R[4], my, R[3] * mx));
                nz = fma(R[8], mz, fma(R[7], my, R[6] * mx));
            }
            const double nd_ = fma(nz, uz, fma(ny, uy, nx * ux));
            const bool ok = finite && best > 0.0 && nd_ != 0.0;
            const double inv = ok ? -1.0 / nd_ : 0.0;
            const double dsx = nx * inv, dsy = ny * inv, dsz = nz * inv;  // ds/dp
            const double gs = gstep ? gstep[i] : 0.0;
            double ghx = 0.0, ghy = 0.0, ghz = 0.0;
            if (ghit) {
                ghx = ghit[i];
                ghy = ghit[n + i];
                ghz = ghit[2 * n + i];
            }
            const double c = fma(ghz, uz, fma(ghy, uy, fma(ghx, ux, gs)));
            if (g_o) {
                g_o[i] = fma(c, dsx, ghx);
                g_o[n + i] = fma(c, dsy, ghy);
                g_o[2 * n + i] = fma(c, dsz, ghz);
            }
            if (g_d) {
                const double cs = c * s;
                g_d[i] = fma(cs, dsx, s * ghx);
                g_d[n + i] = fma(cs, dsy, s * ghy);
                g_d[2 * n + i] = fma(cs, dsz, s * ghz);
            }
            gdx = -c * dsx;
            gdy = -c * dsy;
            gdz = -c * dsz;
        }
        if (partial) {
            // Offset gradient of the workgroup's tracks per daughter: a
            // stable counting sort of the contributions by hit daughter,
            // then each (daughter, component) sums its run in track order,
            // the order of a plain scan over the workgroup's tracks.
            int *cnt = s_bins;           // [4][nd]: per-wavefront counts
            int *run = s_bins + 4 * nd;  // [nd + 1]: start of each daughter's run
            // each wavefront clears its own row (the other wavefronts last
            // read it before the barrier that ended the previous pass), then
            // counts its tracks per daughter and ranks each among the
            // earlier lanes with the same daughter
            for (int k = lane; k < nd; k += 64) cnt[wave * nd + k] = 0;
            int rank = 0;
            unsigned long long rem = __builtin_amdgcn_ballot_w64(h >= 0);
            while (rem != 0ull) {
                const int k = __builtin_amdgcn_readlane(h, __ffsll((long long)rem) - 1);
                const unsigned long long m = __builtin_amdgcn_ballot_w64(h == k);
                if (h == k) rank = lanes_below(m);
                if (lane == 0) cnt[wave * nd + k] = __popcll(m);
                rem &= ~m;
            }
            __syncthreads();
            // every wavefront forms the runs itself (an exclusive scan of the
            // daughters' totals, 64 daughters a pass, lane = daughter) and
            // its own offset within each run; wavefront 0 publishes the runs
            int pos = 0;
            int carry = 0;
            for (int k0 = 0; k0 < nd; k0 += 64) {
                const int k = k0 + lane;
                int tot = 0, below = 0;
                if (k < nd) {
#pragma unroll
                    for (int w = 0; w < kBlock / 64; ++w) {
                        const int c = cnt[w * nd + k];
                        tot += c;
                        below += w < wave ? c : 0;
                    }
                }
                int incl = tot;
                for (int dlt = 1; dlt < 64; dlt <<= 1) {
                    const int v = __shfl_up(incl, dlt);
                    if (lane >= dlt) incl += v;
                }
                const int start = carry + incl - tot;
                if (wave == 0 && k < nd) run[k] = start;
                // a lane whose daughter falls in this pass takes its offset
                const int off = __shfl(start + below, (h - k0) & 63);
                if (h >= k0 && h < k0 + 64) pos = off + rank;
                carry += __shfl(incl, 63);
            }
            if (wave == 0 && lane == 0) run[nd] = carry;
            if (h >= 0) {
                s_g[0][pos] = gdx;
                s_g[1][pos] = gdy;
                s_g[2][pos] = gdz;
            }
            __syncthreads();
            for (int j = tid; j < nj; j += kBlock) {
                const int k = j / 3, comp = j - 3 * k;
                double acc = 0.0;
                for (int q = run[k]; q < run[k + 1]; ++q) acc += s_g[comp][q];
                acc_row[j] += acc;
            }
            __syncthreads();
        }
    };
    // A row of partial sums starts at zero; each of its entries j is thread
    // (j mod kBlock)'s alone.
    auto start = [&](double *acc_row) {
        if (partial)
            for (int j = tid; j < nj; j += kBlock) acc_row[j] = 0.0;
    };
    auto finish = [&](int row) {
        if (partial && lds_acc)
            for (int j = tid; j < nj; j += kBlock) partial[(size_t)row * nj + j] = s_dyn[j];
    };
    auto acc_of = [&](int row) { return lds_acc || !partial ? s_dyn : partial + (size_t)row * nj; };
    // U >> log_each rows of 1 << log_each passes, one after the other; or one row
    // with all its passes
    const bool whole = U == 1 || log_each == 2;
    int row = (int)blockIdx.x * (whole ? 1 : U >> log_each);
    double *acc_row = acc_of(row);
    start(acc_row);
    for (int pass = row, u = 0, q = 0;;) {
        if (pass < npass) differentiate(pass, u, acc_row);
        u = (u + 1) % U;
        pass += rows;
        if (whole ? pass < npass : ++q < 1 << log_each) continue;
        finish(row);
        if (whole || u == 0 || ++row >= rows) return;
        acc_row = acc_of(row);
        start(acc_row);
        pass = row;
        q = 0;
    }
}

// out[j] = sum over workgroups b of partial[b][j], in a fixed order.
__global__ __launch_bounds__(kBlock) void k_reduce_partials(const double *__restrict__ partial,
                                                            int nblocks, int nj,
                                                            double *__restrict__ out) {
    __shared__ double s[kBlock];
    const int j = blockIdx.x;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kBlock) acc += partial[(size_t)b * nj + j];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[j] = s[0];
}

constexpr int kBackwardLdsAcc = 256;

template <int TESTS, int KSET, int U>
static void launch_backward_variant(int rows, int nd, const VolumeRec *vol, const DaughterRec *dau,
                                    const CullBlock *cul, const TracksDev &t, const double *offs, const double *gstep,
                                    const double *ghit, double *g_o, double *g_d, double *part,
                                    const CullBlock *shifted, hipStream_t st) {
    // the offset-gradient sort's counts and runs; the row's accumulator in
    // LDS up to kBackwardLdsAcc daughters (6 KB)
    const bool lds_acc = part && nd <= kBackwardLdsAcc;
    const int64_t npass = (t.n + kBlock - 1) / kBlock;
    if (!part && U > 1) rows = (int)npass;  // (no sums: the passes in order)
    const int log_each = U == 1 || npass <= rows ? 0 : npass <= 2 * (int64_t)rows ? 1 : 2;
    const int own = U >> log_each, nblocks = (rows + own - 1) / own;
    const size_t dyn = (lds_acc ? sizeof(double) * 3 * (size_t)nd : 0) + sizeof(int) * (size_t)(5 * nd + 1);
    if (offs && TESTS && shifted)
        hipLaunchKernelGGL((k_nav_backward<true, TESTS, KSET, TESTS != kNoTests, U>), dim3(nblocks), dim3(kBlock), dyn, st, vol,
                           dau, shifted, t, offs, gstep, ghit, g_o, g_d, part, lds_acc, rows, log_each);
    else if (offs)
        hipLaunchKernelGGL((k_nav_backward<true, TESTS, KSET, false, U>), dim3(nblocks), dim3(kBlock), dyn, st, vol,
                           dau, cul, t, offs, gstep, ghit, g_o, g_d, part, lds_acc, rows, log_each);
    else
        hipLaunchKernelGGL((k_nav_backward<false, TESTS, KSET, true, U>), dim3(nblocks), dim3(kBlock), dyn, st, vol,
                           dau, cul, t, offs, gstep, ghit, g_o, g_d, part, lds_acc, rows, log_each);
}

// Passes that a workgroup takes at a time: kBackwardRounds from the sizes on
// at which the fuller batches gain more than the fewer workgroups lose, for
// volumes of box, tube and cone, and sooner where a batch runs more kinds'
// code. (us, one pass / four: toy detector 600k tracks 35.9 / 36.2, 2^20 50.1 / 46.1;
// every kind 350k 47.2 / 47.2, 400k 50 / 48. Every daughter walked: one pass.)
constexpr int kBackwardRounds = 4;
static bool backward_wide(int64_t n, int kset) {
    return n >= (kset == kSetBasic ? (int64_t)5 << 17 : (int64_t)11 << 15);
}

hipError_t launch_backward(const VolumeRec *vol, const DaughterRec *dau_all, const DaughterRec *dau,
                           const CullBlock *cul, int nd,
                           const TracksDev &t, const double *offs, const double *gstep,
                           const double *ghit, double *g_o, double *g_d, double *partial,
                           double *g_off, int tests, int kset, CullBlock *shift_buf, hipStream_t st) {
    const int rows = backward_rows(t.n);
    double *part = (g_off && nd > 0) ? partial : nullptr;
    if (t.n > 0 || part) {
        const CullBlock *shifted = nullptr;
        if (tests && offs && shift_buf && nd > 0 && t.n > 0) {
            // (the kernel takes the geometry's daughter table)
            hipLaunchKernelGGL(k_cull_blocks<true>, dim3((nd + kCullBlock - 1) / kCullBlock), dim3(64), 0, st, vol, 1,
                               dau_all, offs, shift_buf);
            shifted = shift_buf;
        }
        const bool wide = backward_wide(t.n, kset);
#define GN_BACKWARD(TESTS, U) \
    GN_KSET(kset, (launch_backward_variant<TESTS, KS, U>(rows, nd, vol, dau, cul, t, offs, gstep, ghit, g_o, g_d, \
                                                        part, shifted, st)))
        if (tests == kMatrixTests && wide) GN_BACKWARD(kMatrixTests, kBackwardRounds);
        else if (tests == kMatrixTests) GN_BACKWARD(kMatrixTests, 1);
        else if (tests == kAnyTests && wide) GN_BACKWARD(kAnyTests, kBackwardRounds);
        else if (tests == kAnyTests) GN_BACKWARD(kAnyTests, 1);
        else GN_BACKWARD(kNoTests, 1);
#undef GN_BACKWARD
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (part) {
        hipLaunchKernelGGL(k_reduce_partials, dim3(3 * nd), dim3(kBlock), 0, st, part, rows, 3 * nd,
                           g_off);
        return hipGetLastError();
    }
    return hipSuccess;
}

// ------------------------------------------------ allocation-free adjoint
// The offset gradient's per-workgroup partial sums for the adjoint entry
// point that allocates nothing: a file-scope device array, one copy per GPU
// the library runs on, held until the process ends. In host code the name
// `scratch` is a host-side stand-in, not a device address: host code uses
// only the address hipGetSymbolAddress returns for the current device,
// looked up at the first call on each device and kept.
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t scratch_partials(double **out) {
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
#endif

}  // namespace gn
